"""The library's counters (gwfa_stats): kept per workgroup over its queries and
added up on several lines when a workgroup ends, they equal the sums over the
result records for fewer, as many and more queries than workgroups."""
import pytest

from paper_2206_13574_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,groups", [(1, 0), (63, 64), (64, 64), (65, 64), (700, 129), (700, 3)])
def test_counters_are_the_sums_over_the_results(gpu_lib, n, groups):
    gw = gpu_lib
    g = synth.bubble_graph(88, 4000, snp_gap=60, indel_gap=300, indel_arm=(1, 20))
    r = synth.sample_reads(g, 89, n, 200, 0.03)
    ctx = gw.Context(0)
    ctx.config(lanes=64, groups=groups, dir_log2_max=12, list_cap=4096)
    graph = gw.Graph.of(ctx, g)
    try:
        for _ in range(2):
            ctx.stats(reset=True)
            res, _ = gw.align(ctx, graph, r.seq, r.off, r.v_start)
            st = ctx.stats()
            assert (res["status"] == 0).all()
            assert st["entries"] == int(res["work"].sum())
            assert st["scores"] == int(res["n_scores"].sum())
            assert st["reruns"] == 0
        assert ctx.stats(reset=True)["scores"] == int(res["n_scores"].sum())
        assert all(v == 0 for v in ctx.stats().values())
    finally:
        graph.close()
        ctx.close()
