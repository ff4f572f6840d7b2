"""The host-buffer entry point around the sizes where it changes how data
moves: inputs up to 1 MiB go through pinned memory in one copy, results and
first walks up to 64 KiB come back in one; calls of different sizes in a row
share one workspace; overflowing queries are re-run before the results are
fetched again."""
import numpy as np
import pytest

from paper_2206_13574_amd import synth
from tests.test_gpu_parity import check_path

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("small", [False, True], ids=["default", "overflowing"])
def test_sizes_around_the_staging_limits(gpu_lib, small):
    gw = gpu_lib
    g = synth.bubble_graph(92, 30_000, snp_gap=80, indel_gap=400, indel_arm=(1, 20))
    r = synth.sample_reads(g, 93, 2600, lambda rng, n: rng.integers(300, 560, size=n), 0.02)
    ctx = gw.Context(0)
    graph = gw.Graph.of(ctx, g)
    try:
        ref, _ = gw.align(ctx, graph, r.seq, r.off, r.v_start)
        if small:
            ctx.config(lanes=64, groups=64, dir_log2_max=10, list_cap=1024, dir_factor=1)
        ctx.stats(reset=True)
        # 1,008 results are 64,512 bytes; 64,000 bytes of a few walks; 1 MiB of
        # inputs lies between 2,200 and 2,600 reads
        for n in (1, 2, 500, 1007, 1008, 1023, 1024, 1025, 2200, 2600, 3, 1):
            s = r.subset(np.arange(n))
            cap = int(s.off[-1]) + 64 * n
            code, res, path, need = gw.align_host(ctx, graph, s.seq, s.off, s.v_start, gw.opts(), path_cap=cap)
            print(f"[gpu-host] {n} reads, {int(s.off[-1])} bases, {need} ids", flush=True)
            assert code == gw.OK and need == int(res["path_len"].sum())
            for f in ("status", "dist", "end_v", "end_off", "n_scores", "work"):
                assert np.array_equal(res[f], ref[f][:n]), (n, f)
            for i in range(0, n, 53):
                check_path(g, s.read(i), int(s.v_start[i]), res[i],
                           path[res[i]["path_off"]:res[i]["path_off"] + res[i]["path_len"]])
            code, res2, _, need2 = gw.align_host(ctx, graph, s.seq, s.off, s.v_start, gw.opts(), path_cap=need - 1)
            assert code == gw.ERR_PATH_CAP and need2 >= 1 and np.array_equal(res2["dist"], res["dist"])
        bad = r.subset(np.arange(40))
        for at in (0, 4095, 4096, len(bad.seq) - 1):
            seq = bad.seq.copy()
            seq[at] = ord("N")
            assert gw.align_host(ctx, graph, seq, bad.off, bad.v_start, gw.opts())[0] == gw.ERR_ALPHABET
    finally:
        graph.close()
        ctx.close()
