"""GPU parity on tandem repeats, where several diagonals of one wavefront match
the query over hundreds of bases and their runs are continued together.

A start window over a vertex whose label repeats a unit of 17 to 40 bases puts
the runs' lanes a unit apart, two to four of them in a wave; the query follows
the window's first, a middle or its last unit, exactly or with errors early
on, so that a run cut short changes the distance.  Bar: as the narrow
wavefronts' tests, bit for bit against the oracle at every width."""
import numpy as np
import pytest

from tests.test_gpu_narrow import G, _compare, _dna  # noqa: F401 (G: fixture)

pytestmark = pytest.mark.gpu


def repeat_case(rng, unit, n, errs):
    """(case, window): n start offsets, a label of repeats of `unit` bases."""
    u = _dna(rng, unit)
    labels = [(u * (900 // unit))[:850], _dna(rng, 120), _dna(rng, 90)]
    edges = [(0, 1), (0, 2), (1, 2)]
    j0 = int(rng.integers(0, 200))
    j = j0 + int(rng.choice([0, (n - 1) // 2, n - 1]))
    q = list(labels[0][j:] + labels[1][:100])
    for _ in range(errs):
        p = int(rng.integers(0, 20))
        q[p] = "ACGT"[("ACGT".index(q[p]) + 1) % 4]
    return (labels, edges, "".join(q).encode(), 0), (j0, j0 + n - 1)


@pytest.mark.parametrize("lanes", [64, 128, 256, 512])
def test_runs_of_repeats_are_continued_whole(G, lanes):  # noqa: F811
    gw, ctx = G
    rng = np.random.default_rng(8600)
    both = [repeat_case(rng, unit, n, errs) for unit in (17, 20, 23, 24, 30, 31, 33, 40) for n in (40, 48, 64, 130)
            for errs in (0, 1, 3)]
    cases, windows = [b[0] for b in both], [b[1] for b in both]
    ctx.config(lanes=lanes, groups=len(cases))
    try:
        for a_diff in (0, 100000):
            print(f"[gpu-repeats] lanes {lanes}: {len(cases)} repeats, a_diff={a_diff}", flush=True)
            _compare(gw, ctx, cases, a_diff, windows)
    finally:
        ctx.config()
