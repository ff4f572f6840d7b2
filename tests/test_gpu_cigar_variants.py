"""The base-level alignment's variants (packed query, walk string and rows in
LDS with 256 or 512 lanes, or in memory) give the same operations: the
variant follows from the longest query and the largest distance of a batch,
so the same reads are aligned alone and beside a read that changes it.
Every CIGAR spells its query and its walk and costs the walk's edit distance
(at most the reported distance, which it equals for exact runs)."""
import numpy as np
import pytest

import oracle as O
from paper_2206_13574_amd import synth
from tests import refs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G(gpu_lib):
    ctx = gpu_lib.Context(0)
    ctx.config(lanes=64)
    yield gpu_lib, ctx
    ctx.close()


@pytest.fixture(scope="module")
def setting(G):
    """A graph of structural bubbles, reads of many lengths and error rates
    (none to every base), a very noisy one and a very long one."""
    g = synth.bubble_graph(95, 400_000, sv_gap=4000, sv_arm=(50, 800))
    lens = [1, 2, 31, 32, 33, 63, 64, 65, 127, 500, 1000, 3001]
    r = synth.sample_reads(g, 96, 60, lambda rng, n: np.resize(lens, n), lambda rng, n: rng.choice([0.0, 0.02, 0.1, 0.4], n))
    noisy = synth.sample_reads(g, 97, 1, 9000, 0.15)
    long_ = synth.sample_reads(g, 98, 1, 330_000, 0.001)
    return g, r, noisy, long_


def _run(gw, ctx, g, reads, o):
    seq = np.concatenate([x.seq for x in reads])
    off = np.concatenate([[0], np.cumsum(np.concatenate([np.diff(x.off) for x in reads]))]).astype(np.int64)
    vs = np.concatenate([x.v_start for x in reads])
    graph = gw.Graph.of(ctx, g)
    try:
        batch = gw.upload_reads(ctx, seq, off, vs)
        out = gw.alloc_out(ctx, len(vs), int(off[-1]) + 64 * len(vs))
        gw.step_dev(ctx, graph, batch, out, o)
        res, path, _ = gw.fetch(out, len(vs))
        ops, coff, clen = gw.cigar_dev(ctx, graph, batch, out)
    finally:
        graph.close()
    cig = []
    for i in range(len(vs)):
        q = seq[off[i]:off[i + 1]].tobytes()
        assert res[i]["status"] == 0 and clen[i] >= 0
        c = ops[coff[i]:coff[i] + clen[i]]
        t = O.spell_walk(g, path[res[i]["path_off"]:res[i]["path_off"] + res[i]["path_len"]], int(res[i]["end_off"]))
        cost = refs.cigar_cost(q, t, c)
        assert cost <= res[i]["dist"]
        if len(q) <= 1000:
            assert cost == O.ed_global(q, t)
        cig.append(c)
    return res, cig


@pytest.mark.parametrize("mode", ["exact", "pruned"])
def test_variants_agree(G, setting, mode):
    gw, ctx = G
    g, r, noisy, long_ = setting
    o = gw.opts() if mode == "exact" else gw.opts(prune=gw.PRUNE_HEURISTIC, a_diff=60)
    res, alone = _run(gw, ctx, g, [r], o)
    print(f"[gpu-cigar] {mode}: alone, distances up to {res['dist'].max()}", flush=True)
    assert res["dist"].max() < 1024
    more = [[r, noisy]] if mode == "exact" else [[r, noisy], [r, long_], [r, noisy, long_]]
    for reads in more:
        res2, cig = _run(gw, ctx, g, reads, o)
        print(f"[gpu-cigar] {mode}: beside {[int(x.off[-1]) for x in reads[1:]]} bases, distances {res2['dist'][r.n:]}",
              flush=True)
        assert np.array_equal(res2["dist"][:r.n], res["dist"])
        for a, b in zip(alone, cig):
            assert np.array_equal(a, b)
