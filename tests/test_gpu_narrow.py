"""GPU parity of wavefronts around the sizes where one wave hands a score to
the whole workgroup: lists of 48 and 64 entries, 64 and 128 crossing
candidates (hub vertices of such out-degrees, reached at once or again
through a cycle), and free start windows of such lengths.

Bar: distance, end, number of scores and sum |F_s| equal the oracle's
transcription of Algorithms 1-4, bit for bit, at every width of workgroup;
traced walks spell a string at the reported distance."""
import numpy as np
import pytest

import oracle as O
from paper_2206_13574_amd import synth
from tests.test_gpu_parity import check_path, reads_of, union_graph

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G(gpu_lib):
    ctx = gpu_lib.Context(0)
    yield gpu_lib, ctx
    ctx.close()


def _dna(rng, n):
    return "".join("ACGT"[x] for x in rng.integers(0, 4, size=n))


def hub_case(rng, deg, cyclic):
    """A vertex with `deg` out-edges whose targets meet again, three times
    over (cyclic: the last one leads back to the first); a query along one
    walk with errors."""
    labels, edges, walk, hub = [_dna(rng, 70)], [], [0], 0
    for _ in range(3):
        first = len(labels)
        labels += [_dna(rng, int(rng.integers(1, 40))) for _ in range(deg)] + [_dna(rng, 33)]
        join = len(labels) - 1
        edges += [(hub, first + j) for j in range(deg)] + [(first + j, join) for j in range(deg)]
        walk += [first + int(rng.integers(0, deg)), join]
        hub = join
    if cyclic:
        edges.append((hub, 0))
        walk += walk[:3]
    q = list("".join(labels[v] for v in walk))
    for _ in range(max(2, len(q) // 25)):
        p, kind = int(rng.integers(0, len(q))), int(rng.integers(0, 3))
        if kind == 0:
            q[p] = _dna(rng, 1)
        elif kind == 1:
            q.insert(p, _dna(rng, 1))
        else:
            del q[p]
    return labels, edges, "".join(q).encode(), 0


def _compare(gw, ctx, cases, a_diff, windows=None):
    g, base = union_graph(cases)
    graph = gw.Graph.of(ctx, g)
    seq, off = reads_of([c[2] for c in cases])
    vs = np.asarray([c[3] + b for c, b in zip(cases, base)], np.int32)
    o = gw.opts(prune=gw.PRUNE_HEURISTIC if a_diff else gw.PRUNE_NONE, a_diff=a_diff)
    kw = {}
    if windows is not None:
        kw = dict(start_off=np.asarray([w[0] for w in windows], np.int32),
                  start_hi=np.asarray([w[1] for w in windows], np.int32))
    try:
        res, paths = gw.align(ctx, graph, seq, off, vs, o, path_cap=4 * int(off[-1]) + 64 * len(cases), **kw)
    finally:
        graph.close()
    for i, (labels, edges, q, v_s) in enumerate(cases):
        j0, j1 = windows[i] if windows is not None else (0, -1)
        ref = O.gwf((labels, edges), q, v_s, a_diff=a_diff, j0=j0, j1=j1)
        got = (int(res[i]["status"]), int(res[i]["dist"]), int(res[i]["end_v"]) - base[i], int(res[i]["end_off"]),
               int(res[i]["n_scores"]), int(res[i]["work"]))
        assert got == (0, ref["dist"], ref["end_v"], ref["end_j"], ref["dist"] + 1, ref["work"]), (i, a_diff)
        if windows is None and a_diff == 0:
            check_path(g, q, int(vs[i]), res[i], paths[i])


@pytest.mark.parametrize("lanes", [64, 128, 256, 512])
def test_hubs_around_the_narrow_limits(G, lanes):
    gw, ctx = G
    ctx.config(lanes=lanes)
    rng = np.random.default_rng(8100)
    cases = [hub_case(rng, deg, cyc) for deg in (1, 2, 3, 15, 16, 31, 32, 47, 48, 49, 61, 62, 63, 64, 65, 127, 128, 129,
                                                 200) for cyc in (False, True)]
    for a_diff in (0, 1, 12, 40, 100000):
        print(f"[gpu-narrow] lanes {lanes}: {len(cases)} hub graphs, a_diff={a_diff}", flush=True)
        _compare(gw, ctx, cases, a_diff)


@pytest.mark.parametrize("lanes", [64, 256])
def test_start_windows_around_the_narrow_limits(G, lanes):
    gw, ctx = G
    ctx.config(lanes=lanes)
    rng = np.random.default_rng(8200)
    cases, windows = [], []
    for n in (1, 2, 31, 32, 33, 46, 47, 48, 49, 50, 62, 63, 64, 65, 66, 128, 200):
        labels, edges, q, v_s = hub_case(rng, 5, False)
        labels[0] = _dna(rng, 210)
        cases.append((labels, edges, labels[0][n:].encode() + q[70:], v_s))
        j0 = int(rng.integers(0, 210 - n + 1))
        windows.append((j0, j0 + n - 1))
    for a_diff in (0, 12, 100000):
        print(f"[gpu-narrow] lanes {lanes}: {len(cases)} start windows, a_diff={a_diff}", flush=True)
        _compare(gw, ctx, cases, a_diff, windows)


@pytest.mark.parametrize("a_diff", [40, 1024, 1025])
def test_pruned_queries_that_outgrow_the_first_tier(G, a_diff):
    """Pruned runs up to a lag of 1,024 start on small arenas (lists of 4,096
    entries, also before a score is pruned); a query that outgrows them is run
    again on the configured ones.  The results do not depend on the tier."""
    gw, ctx = G
    ctx.config(lanes=64)
    rng = np.random.default_rng(8300)
    cases = [hub_case(rng, 2200, False), hub_case(rng, 5, False)]
    ctx.stats(reset=True)
    _compare(gw, ctx, cases, a_diff)
    assert ctx.stats()["reruns"] > 0


@pytest.mark.parametrize("lanes", [64, 256, 512])
def test_hubs_around_the_merge_limits(G, lanes):
    """Crossing sets of as many entries as the merge ranks in LDS (256 or
    1,024), one fewer and one more, exact: lists of several thousand entries
    with few neighbours among them, in parts written by each wave."""
    gw, ctx = G
    ctx.config(lanes=lanes)
    rng = np.random.default_rng(8400)
    print(f"[gpu-narrow] lanes {lanes}: merge limits", flush=True)
    _compare(gw, ctx, [hub_case(rng, deg, False) for deg in (255, 256, 257, 511, 1023, 1024, 1025)], 0)


@pytest.mark.parametrize("lanes", [64, 128, 256, 512])
def test_start_windows_around_whole_batches(G, lanes):
    """Wide lists whose parts hold one, two and three groups of 64 entries, one
    or two fewer and one more: first, middle and last batches of a wave, full
    and of a few candidates.  With the number of workgroups given the exact
    batch keeps the width asked for."""
    gw, ctx = G
    rng = np.random.default_rng(8500)
    cases, windows = [], []
    for b in (1, 2, 3):
        for n in (lanes * b + d for d in (-2, -1, 0, 1)):
            labels, edges, q, v_s = hub_case(rng, 5, False)
            labels[0] = _dna(rng, 1700)
            cases.append((labels, edges, labels[0][n:].encode() + q[70:], v_s))
            j0 = int(rng.integers(0, 1700 - n + 1))
            windows.append((j0, j0 + n - 1))
    ctx.config(lanes=lanes, groups=len(cases))
    try:
        for a_diff in (0, 100000):
            print(f"[gpu-narrow] lanes {lanes}: {len(cases)} whole batches, a_diff={a_diff}", flush=True)
            _compare(gw, ctx, cases, a_diff, windows)
    finally:
        ctx.config()


def test_batches_around_the_widening_limits(G):
    """Exact batches small enough to be resident at more lanes per query are
    launched with more: the same results at every size."""
    gw, ctx = G
    g = synth.bubble_graph(90, 5000, snp_gap=50, indel_gap=300, indel_arm=(1, 20))
    r = synth.sample_reads(g, 91, 3600, lambda rng, n: rng.integers(50, 400, size=n), 0.04)
    graph = gw.Graph.of(ctx, g)
    try:
        ctx.config(lanes=64, groups=300)           # a given number of workgroups: no widening
        ref, _ = gw.align(ctx, graph, r.seq, r.off, r.v_start)
        ctx.config(lanes=64)
        for n in (1, 767, 768, 769, 1023, 1024, 1025, 2303, 2304, 2305, 3600):
            print(f"[gpu-narrow] {n} queries", flush=True)
            s = r.subset(np.arange(n))
            res, paths = gw.align(ctx, graph, s.seq, s.off, s.v_start)
            for f in ("status", "dist", "end_v", "end_off", "n_scores", "work"):
                assert np.array_equal(res[f], ref[f][:n]), (n, f)
            for i in range(0, n, 97):
                check_path(g, s.read(i), int(s.v_start[i]), res[i], paths[i])
    finally:
        graph.close()
