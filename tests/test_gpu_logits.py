"""GPU: batch logits of the pruning network are the alignment kernel's own, bit
for bit: with the threshold set to an entry's logit, the kernel drops exactly
the entries whose batch logit is below it."""
import numpy as np
import pytest

from paper_2206_13574_amd import synth, train_prune

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G(gpu_lib):
    ctx = gpu_lib.Context(0)
    yield gpu_lib, ctx
    ctx.close()


def test_decisions_at_an_entry_s_own_logit(G):
    gw, ctx = G
    torch = ctx.torch
    W = train_prune.load()
    ctx.mlp_load(W["w_bf16"], W["scale"])
    bits = torch.from_numpy(np.ascontiguousarray(W["w_bf16"]).view(np.int16).copy()).to(ctx.tdev)
    g = synth.bubble_graph(61, 4000, snp_gap=60, indel_gap=300, indel_arm=(1, 20))
    r = synth.sample_reads(g, 62, 40, lambda rng, n: rng.integers(300, 600, size=n), 0.06)
    graph = gw.Graph.of(ctx, g)
    gate, period, tau, close = 4, 2, W["tau"], 0
    rng = np.random.default_rng(63)
    try:
        for step in range(60):
            ctx.stats(reset=True)
            o = gw.opts(prune=gw.PRUNE_LEARNED, keep_threshold=float(tau), mlp_gate=gate, mlp_period=period,
                        traceback=False)
            _, d, produced = gw.align_dump(ctx, graph, r.seq, r.off, r.v_start, o)
            st = ctx.stats()
            f = torch.from_numpy(d["feat"]).to(ctx.tdev)
            out = torch.empty(len(d["feat"]), dtype=torch.float32, device=ctx.tdev)
            gw.mlp_logits_dev(ctx, f, W["scale"], bits, out)
            z = out.cpu().numpy()
            key = d["read"].astype(np.int64) << 32 | d["score"]
            _, inv, cnt = np.unique(key, return_inverse=True, return_counts=True)
            a = d["i"] + d["W"]
            amax = np.full(len(cnt), -1, np.int64)
            np.maximum.at(amax, inv, a)
            run = (cnt[inv] >= gate) & (d["score"] % period == 0)
            drop = run & (z < np.float32(tau)) & (a != amax[inv])
            assert produced == len(z) and int(run.sum()) == st["mlp_evals"], step
            assert int(drop.sum()) == st["pruned"], (step, tau, int(drop.sum()), st["pruned"])
            # next: the logit of an entry that any threshold meets (score 2, before anything is dropped)
            first = np.flatnonzero(run & (d["score"] == period) & (a != amax[inv]))
            close += int((z[first] == np.float32(tau)).sum())
            tau = z[rng.choice(first)]
    finally:
        graph.close()
    assert close > 20          # entries that stood at the threshold itself
