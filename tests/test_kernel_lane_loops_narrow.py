"""Walk-length tracking adds no per-entry loop over the active lanes to the
narrow path either (narrow_scores, a function of its own in the assembly,
where pruned runs spend nearly all their time): as
test_kernel_lane_loops.py checks for the alignment kernel, but at every depth,
since the function's loops start at its scores.  Pinned on per-entry LDS
maxima put into record_entry, which fails."""
import re

import pytest

from paper_2206_13574_amd import asm_check, build

_SRC = [s for s in build.sources() if s.endswith("gwfa_kernels.hip")][0]


def _counts(text):
    out = {}
    for name, lines in asm_check._functions(text):
        m = re.search(r"narrow_scoresILi(\d+)ELi(\d)E", name)
        if m:
            out[(int(m.group(1)), int(m.group(2)))] = len(asm_check.lane_loops(lines))
    return out


@pytest.fixture(scope="module")
def counts():
    return _counts(asm_check.device_asm(_SRC))


def test_every_instantiation_is_checked(counts):
    assert sorted(counts) == [(b, m) for b in (64, 128, 256, 512) for m in (0, 1, 3)]


def test_tracked_instantiations_add_no_lane_loops(counts):
    for (block, mode), n in counts.items():
        assert n <= counts[(block, 0)], (block, mode, n, counts[(block, 0)])


def test_checker_flags_per_entry_atomics(tmp_path):
    src = open(_SRC).read()
    new = """        lmax.x = max(lmax.x, i + W);
        lmax.y = max(lmax.y, i);"""
    assert new in src
    src = src.replace(new, """        atomicMax(&S.amax, i + W);
        atomicMax(&S.imax, i);""")
    p = tmp_path / "gwfa_kernels.hip"
    p.write_text(src)
    c = _counts(asm_check.device_asm(str(p)))
    assert all(c[(b, m)] > c[(b, 0)] for b in (64, 128, 256, 512) for m in (1, 3))
