"""The work a user of this library has it do, as cases that can be timed and
whose outputs can be compared: alignments of reads to sequence graphs through
each entry point, mode and size range, base-level alignment of the walks, and
training and inference of the pruning network.

A case is a dict of plain values.  `prepare` makes what a program holds before
the call (graph uploaded once, reads and output buffers on the device, the
context configured from the tuner's table), `run` is one call.

Outputs of alignments are the result records' deterministic fields, as views
of the result buffer.  The order in which walks are placed in the path buffer
and the choice among equally good walks at a bubble are not determined by the
inputs, so walks come back only where the graph has one best walk per read
(graphs of structural bubbles), in read order.
"""
import math

import numpy as np
import torch

from paper_2206_13574_amd import calibrate_prune, gwfa, synth, train_prune, tune

# Graphs: the shapes of the repository's workloads, plus a graph of structural
# bubbles alone (large alternative arms, as assembly-level variation graphs
# have), where every read has one best walk.  `tuned` names the tuner's entry.
SHAPES = {
    "dag5k": dict(seed=101, backbone_len=5_000, snp_gap=100, indel_gap=500, indel_arm=(1, 20), tuned="cfg1"),
    "dag1m": dict(seed=201, backbone_len=1_000_000, snp_gap=1000, indel_gap=5000, indel_arm=(1, 50),
                  sv_gap=100_000, sv_arm=(1000, 10000), tuned="cfg2"),
    "loops500k": dict(seed=301, backbone_len=500_000, loop_sites=200, loop_unit=(10, 200), tuned="cfg3"),
    "dag10m": dict(seed=401, backbone_len=10_000_000, snp_gap=100, indel_gap=500, indel_arm=(1, 20), tuned="cfg4"),
    "sv1m": dict(seed=501, backbone_len=1_000_000, sv_gap=5000, sv_arm=(200, 2000), tuned="none"),
}
A_DIFF = 50        # Algorithm 4's lag on reads of this length
N_PARAM = gwfa.MLP_N


def listed():
    return [
        # one read from host memory: an interactive query, or a loop over reads
        dict(name="one_read", kind="one", shape="sv1m", mode="exact", len=1000, err_lo=0.01, err_hi=0.01),
        # a handful of reads against a gene-sized graph
        dict(name="gene_50x1k", kind="batch", shape="dag5k", mode="exact", walks=True, reads=50, len=1000, half=0,
             sigma=0.0, err_lo=0.01, err_hi=0.01),
        # short reads seeded inside vertices, with end vertices and free end gaps, distances only
        dict(name="short_seeded", kind="seeded", shape="dag1m", mode="exact", walks=False, reads=20_011, len=200,
             half=50, sigma=0.0, err_lo=0.001, err_hi=0.03),
        # long reads against a 1 Mb DAG, exact with walks
        dict(name="dag1m_exact", kind="batch", shape="dag1m", mode="exact", walks=True, reads=20_000, len=10_000,
             half=0, sigma=0.5, err_lo=0.001, err_hi=0.05),
        # the same with Algorithm 4, and with the trained network
        dict(name="dag1m_heuristic", kind="batch", shape="dag1m", mode="heuristic", walks=True, reads=20_000,
             len=10_000, half=0, sigma=0.5, err_lo=0.001, err_hi=0.05),
        # long noisy reads against the 10 Mb graph, a captured launch
        dict(name="dag10m_exact", kind="plan", shape="dag10m", mode="exact", walks=True, reads=3_001, len=20_000,
             half=10_000, sigma=0.0, err_lo=0.01, err_hi=0.10),
        dict(name="dag10m_learned", kind="batch", shape="dag10m", mode="learned", walks=True, reads=8_009, len=20_000,
             half=10_000, sigma=0.0, err_lo=0.01, err_hi=0.10),
        # very long reads through tandem-repeat loops (a cyclic graph), distances only
        dict(name="loops_exact", kind="batch", shape="loops500k", mode="exact", walks=False, reads=500, len=100_000,
             half=0, sigma=0.0, err_lo=0.01, err_hi=0.01),
        # a file's worth of reads from host memory to results in host memory
        dict(name="host_batch", kind="host", shape="sv1m", mode="heuristic", walks=True, reads=2_003, len=10_000,
             half=0, sigma=0.5, err_lo=0.001, err_hi=0.05),
        # CIGARs of a finished batch
        dict(name="cigar", kind="cigar", shape="sv1m", mode="heuristic", walks=True, reads=4_001, len=8_000, half=0,
             sigma=0.5, err_lo=0.01, err_hi=0.08),
        # one training step of the pruning network (the trainer's batch), and scoring a dump's records
        dict(name="mlp_train", kind="train", samples=32_768),
        dict(name="mlp_logits", kind="logits", samples=1_000_003),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["one", "gene", "seeded", "dag1m", "dag10m", "loops", "host", "cigar", "train", "logits"])
    mode = rng.choice(["exact", "heuristic", "learned"])
    if kind == "train":
        return dict(kind="train", samples=_log(rng, 1_000, 200_000))
    if kind == "logits":
        return dict(kind="logits", samples=_log(rng, 1_000, 1_000_000))
    err = rng.uniform(0.002, 0.05)
    if kind == "one":
        return dict(kind="one", shape=rng.choice(["sv1m", "dag5k"]), mode="exact", len=_log(rng, 100, 4_000),
                    err_lo=err, err_hi=err)
    if kind == "gene":
        return dict(kind=rng.choice(["batch", "plan"]), shape="dag5k", mode=mode, walks=rng.random() < 0.5,
                    reads=_log(rng, 3, 300), len=_log(rng, 200, 2_000), half=0, sigma=0.3, err_lo=0.0, err_hi=err)
    if kind == "seeded":
        return dict(kind="seeded", shape="dag1m", mode=mode, walks=rng.random() < 0.5, reads=_log(rng, 500, 20_000),
                    len=_log(rng, 100, 600), half=0, sigma=0.2, err_lo=0.0, err_hi=err)
    if kind == "dag1m":
        return dict(kind=rng.choice(["batch", "plan"]), shape="dag1m", mode=mode, walks=rng.random() < 0.7,
                    reads=_log(rng, 200, 20_000), len=_log(rng, 1_000, 10_000), half=0, sigma=0.5, err_lo=0.0,
                    err_hi=err)
    if kind == "dag10m":
        return dict(kind="batch", shape="dag10m", mode=mode, walks=rng.random() < 0.7, reads=_log(rng, 300, 3_000),
                    len=_log(rng, 3_000, 20_000), half=1_000, sigma=0.0, err_lo=0.0, err_hi=err)
    if kind == "loops":
        return dict(kind="batch", shape="loops500k", mode=mode, walks=False, reads=_log(rng, 50, 500),
                    len=_log(rng, 10_000, 100_000), half=0, sigma=0.0, err_lo=0.0, err_hi=0.01)
    if kind == "host":
        return dict(kind="host", shape="sv1m", mode="heuristic", walks=True, reads=_log(rng, 10, 2_000),
                    len=_log(rng, 500, 10_000), half=0, sigma=0.5, err_lo=0.0, err_hi=err)
    return dict(kind="cigar", shape="sv1m", mode="heuristic", walks=True, reads=_log(rng, 20, 4_000),
                len=_log(rng, 500, 8_000), half=0, sigma=0.5, err_lo=0.0, err_hi=0.08)


# --------------------------------------------------------------------------
# reads
# --------------------------------------------------------------------------
_graphs = {}


def _graph(shape):
    if shape not in _graphs:
        a = {k: v for k, v in SHAPES[shape].items() if k not in ("seed", "tuned")}
        _graphs[shape] = synth.bubble_graph(SHAPES[shape]["seed"], **a)
    return _graphs[shape]


def _lengths(case, n, rng):
    if case.get("sigma"):
        x = rng.lognormal(math.log(case["len"]), case["sigma"], size=n)
        return np.clip(np.round(x), case["len"] / 10, case["len"] * 5).astype(np.int64)
    h = case.get("half", 0)
    return rng.integers(case["len"] - h, case["len"] + h + 1, size=n)


def _sample(g, lens, errs, seed, inside):
    """Reads along random forward walks with sequencing errors, drawn on the
    GPU: (ascii, offsets, start vertex, start offset, last vertex), numpy.
    inside: the read starts anywhere inside its start vertex, else at its
    first base.  Loops are passed 1 to 30 times.  A read that meets the end
    of the graph ends there."""
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(seed)
    n = len(lens)
    lab = torch.from_numpy(np.diff(g.seg_off)).to(dev)
    base_of = torch.from_numpy(g.seg_off).to(dev)
    loop = np.zeros(g.n_vtx, bool)
    loop[g.edge_src[g.edge_src == g.edge_dst]] = True
    keep = g.edge_src != g.edge_dst
    order = np.argsort(g.edge_src[keep], kind="stable")
    dst = torch.from_numpy(np.append(g.edge_dst[keep][order], 0).astype(np.int64)).to(dev)
    first = np.zeros(g.n_vtx + 1, np.int64)
    first[1:] = np.cumsum(np.bincount(g.edge_src[keep], minlength=g.n_vtx))
    first = torch.from_numpy(first).to(dev)
    loop = torch.from_numpy(loop).to(dev)
    # starts whose read fits before the end of the backbone (most of the time)
    pos = torch.from_numpy(g.pos).to(dev)
    last = int(g.pos[-1]) + int(g.seg_off[-1] - g.seg_off[-2])
    need = torch.from_numpy(np.asarray(lens, np.int64)).to(dev)
    u = torch.rand(n, generator=gen, device=dev, dtype=torch.float64)
    start_pos = (u * (last - 1.2 * need.double()).clamp(min=1.0)).long()
    v = (torch.searchsorted(pos, start_pos, right=True) - 1).clamp(min=0)
    v_start = v.clone()
    skip = (torch.rand(n, generator=gen, device=dev) * lab[v]).long() if inside else torch.zeros_like(v)
    laps = torch.where(loop[v], torch.randint(1, 31, (n,), generator=gen, device=dev), torch.ones_like(v))
    left, at, segs, takes = need.clone(), skip.clone(), [], []
    v_end = v.clone()
    step = 0
    while True:
        take = torch.minimum(lab[v] - at, left)
        segs.append(base_of[v] + at)
        takes.append(take)
        v_end = torch.where(take > 0, v, v_end)
        left = left - take
        step += 1
        if step % 32 == 0 and not bool((left > 0).any()):
            break
        at = torch.zeros_like(v)
        again = laps > 1
        deg = first[v + 1] - first[v]
        pick = first[v] + (torch.rand(n, generator=gen, device=dev) * deg).long()
        new = torch.where(deg > 0, dst[pick], v)
        left = torch.where(~again & (deg == 0), torch.zeros_like(left), left)
        nlaps = torch.where(loop[new], torch.randint(1, 31, (n,), generator=gen, device=dev), torch.ones_like(v))
        laps = torch.where(again, laps - 1, nlaps)
        v = torch.where(again, v, new)
    segs, takes = torch.stack(segs, 1), torch.stack(takes, 1)
    ref = torch.from_numpy(g.seq).to(dev)
    acgt = torch.tensor([65, 67, 71, 84], dtype=torch.uint8, device=dev)
    code = torch.zeros(256, dtype=torch.uint8, device=dev)
    code[acgt.long()] = torch.arange(4, dtype=torch.uint8, device=dev)
    e = torch.from_numpy(np.asarray(errs, np.float32)).to(dev)
    seqs, counts = [], []
    per = max(1, int(3e7 / max(float(need.double().mean()), 1.0)))     # reads spelled at a time
    for a in range(0, n, per):
        s, t = segs[a:a + per].reshape(-1), takes[a:a + per].reshape(-1)
        rid = torch.repeat_interleave(torch.arange(takes[a:a + per].shape[0], device=dev),
                                      takes[a:a + per].sum(1))
        ends = torch.cumsum(t, 0)
        tot = int(ends[-1])
        shift = torch.repeat_interleave(s - (ends - t), t)
        c = code[ref[shift + torch.arange(tot, device=dev)].long()]
        bad = torch.rand(tot, generator=gen, device=dev) < e[a:a + per][rid]
        what = torch.randint(0, 3, (tot,), generator=gen, device=dev, dtype=torch.uint8)
        other = torch.randint(1, 4, (tot,), generator=gen, device=dev, dtype=torch.uint8)
        c = torch.where(bad & (what == 0), (c + other) & 3, c)
        cnt = torch.where(bad & (what == 1), 2, torch.where(bad & (what == 2), 0, 1))
        b = torch.repeat_interleave(acgt[c.long()], cnt)
        ins = (torch.cumsum(cnt, 0) - 1)[bad & (what == 1)]
        b[ins] = acgt[torch.randint(0, 4, (len(ins),), generator=gen, device=dev)]
        seqs.append(b.cpu())
        counts.append(torch.zeros(takes[a:a + per].shape[0], dtype=torch.int64, device=dev)
                      .index_add_(0, rid, cnt.long()).cpu())
    off = np.zeros(n + 1, np.int64)
    off[1:] = np.cumsum(torch.cat(counts).numpy())
    return (torch.cat(seqs).numpy(), off, v_start.int().cpu().numpy(), skip.int().cpu().numpy(),
            v_end.int().cpu().numpy())


# --------------------------------------------------------------------------
# what a program keeps: one context with its working memory, the graph
# uploaded to it, and the pruning network
# --------------------------------------------------------------------------
_held = {}


def _context(case):
    key = (case["shape"], case["mode"], case["kind"])
    if key not in _held:
        _held.clear()      # a process holds one context's working memory at a time
        ctx = gwfa.Context(0)
        tuned = SHAPES[case["shape"]]["tuned"]
        cfg = tune.best_config(tuned)
        if case["mode"] != "exact":
            cfg["lanes"] = tune.best_lanes(tuned, case["mode"])
        if case["kind"] == "seeded":
            cfg["lanes"] = 64          # wavefronts of short reads are small
        ctx.config(**cfg)
        W = train_prune.load()
        ctx.mlp_load(W["w_bf16"], W["scale"])
        _held[key] = (ctx, gwfa.Graph.of(ctx, _graph(case["shape"])))
    return _held[key]


def _opts(case):
    walks = bool(case.get("walks", True))
    more = dict(query_end_free=10, walk_end_free=True) if case["kind"] == "seeded" else {}
    if case["mode"] == "heuristic":
        return gwfa.opts(prune=gwfa.PRUNE_HEURISTIC, a_diff=A_DIFF, traceback=walks, **more)
    if case["mode"] == "learned":
        W = train_prune.load()
        tau = calibrate_prune.load().get(SHAPES[case["shape"]]["tuned"], W)["tau"]
        return gwfa.opts(prune=gwfa.PRUNE_LEARNED, keep_threshold=float(tau), mlp_gate=W["gate"],
                         mlp_period=W["period"], traceback=walks, **more)
    return gwfa.opts(traceback=walks, **more)


def _features(n, gen, dev):
    """Trace-record features of 1 kb reads (log1p of the integer quantities
    the alignment kernel forms) and labels (few positives)."""
    def ints(hi):
        return torch.randint(0, hi, (n,), generator=gen, device=dev).float()
    lag, front = ints(300), ints(1000)
    f = torch.stack([torch.log1p(lag), torch.log1p(ints(80)), torch.log1p(1 + ints(2)), torch.log1p(lag // 2),
                     torch.log1p(ints(120)), (2 * ints(2) - 1) * torch.log1p(ints(25)), front / 1000,
                     torch.log1p(1000 - front)], 1).contiguous()
    y = (torch.rand(n, generator=gen, device=dev) < 0.3 * torch.exp(-lag / 20)).to(torch.uint8)
    return f, y


def _params(gen, dev):
    """Weights and Adam moments in the middle of a training run."""
    w = torch.zeros(N_PARAM, device=dev)
    for a, b, s in ((0, 512, 0.5), (576, 4672, 0.18), (4736, 4800, 0.125)):
        w[a:b] = s * torch.randn(b - a, generator=gen, device=dev)
    m1 = 1e-3 * torch.randn(N_PARAM, generator=gen, device=dev)
    m2 = 1e-5 * (0.1 + torch.rand(N_PARAM, generator=gen, device=dev))
    return w, m1, m2


SCALE = np.array([0.17, 0.23, 0.7, 0.2, 0.2, 0.3, 1.0, 0.14], np.float32)
POS_WEIGHT, LR, STEP0 = 8.0, 2e-3, 1000


def prepare(case, seed):
    kind, dev = case["kind"], torch.device("cuda")
    if kind in ("train", "logits"):
        if "ctx" not in _held:
            _held.clear()
            _held["ctx"] = gwfa.Context(0)
        ctx = _held["ctx"]
        gen = torch.Generator(device=dev).manual_seed(seed)
        f, y = _features(case["samples"], gen, dev)
        w, m1, m2 = _params(gen, dev)
        wb = torch.zeros(N_PARAM, dtype=torch.int16, device=dev)
        gwfa.mlp_cast_dev(ctx, w, wb)
        return dict(kind=kind, ctx=ctx, f=f, y=y, w=w, m1=m1, m2=m2, wb=wb, grad=torch.zeros(N_PARAM, device=dev),
                    loss=torch.zeros(1, device=dev), z=torch.zeros(case["samples"], device=dev), step=STEP0)
    rng = np.random.default_rng(seed)
    n = case.get("reads", 1)
    lens = _lengths(case, n, rng)
    errs = rng.uniform(case["err_lo"], case["err_hi"], size=n)
    g = _graph(case["shape"])
    seq, off, vs, j0, ve = _sample(g, lens, errs, seed, inside=kind == "seeded")
    ctx, graph = _context(case)
    o = _opts(case)
    s = dict(kind=kind, shape=case["shape"], ctx=ctx, graph=graph, o=o, n=n)
    if kind in ("one", "host"):
        s.update(seq=seq, off=off, vs=vs, cap=int(off[-1]) // 4 + 64 * n, walks=np.zeros(32 * n + 64, np.int32))
        return s
    s["batch"] = gwfa.upload_reads(ctx, seq, off, vs)
    s["out"] = gwfa.alloc_out(ctx, n, int(off[-1]) // 4 + 64 * n if o.traceback else 0)
    if kind == "seeded":
        lab = np.diff(g.seg_off)[vs]
        s["at"] = [torch.from_numpy(np.ascontiguousarray(x, np.int32)).to(dev)
                   for x in (ve, j0, np.minimum(j0 + 8, lab))]
    elif kind == "plan":
        s["plan"] = gwfa.Plan(ctx, graph, s["batch"], s["out"], o)
    elif kind == "cigar":
        gwfa.step_dev(ctx, graph, s["batch"], s["out"], o)
        s["ops"] = np.zeros(n * case["len"] // 2 + 64, np.int32)
    return s


def _fields(res, n):
    """dist, end_v, end_off, status | n_scores, work | start_off, clip"""
    x = res.view(torch.int32)[:16 * n].view(n, 16)
    return [x[:, 0:4], x[:, 7:10], x[:, 14:16]]


def _in_order(words, offs, lens, into):
    """The variable-length outputs of all reads, in read order, in the
    caller's buffer (zeros after them)."""
    parts = [words[a:a + k] for a, k in zip(offs.tolist(), lens.tolist()) if k > 0]
    if parts:
        np.concatenate(parts, out=into[:sum(map(len, parts))])
    return into


def run(s):
    kind, ctx = s["kind"], s["ctx"]
    if kind == "train":
        s["step"] += 1
        gwfa.mlp_grad_dev(ctx, s["f"], s["y"], SCALE, s["wb"], s["grad"], s["loss"], pos_weight=POS_WEIGHT)
        gwfa.mlp_adam_dev(ctx, s["w"], s["m1"], s["m2"], s["grad"], s["wb"], s["step"], LR)
        return dict(grad=s["grad"], loss=s["loss"], master=s["w"], m1=s["m1"], m2=s["m2"],
                    weights=s["wb"].view(torch.bfloat16))
    if kind == "logits":
        gwfa.mlp_logits_dev(ctx, s["f"], SCALE, s["wb"], s["z"])
        return s["z"]
    graph, o, n = s["graph"], s["o"], s["n"]
    if kind == "one":
        code, res, walk = gwfa.align_one(ctx, graph, s["seq"], int(s["vs"][0]), o)
        out = [code] + [int(res[k]) for k in ("dist", "end_v", "end_off", "status", "n_scores", "work")]
        if s["shape"] == "sv1m":
            s["walks"][:len(walk)] = walk
            out.append(s["walks"])
        return out
    if kind == "host":
        code, res, path, _ = gwfa.align_host(ctx, graph, s["seq"], s["off"], s["vs"], o, path_cap=s["cap"])
        return [code] + [res[k] for k in ("dist", "end_v", "end_off", "status", "path_len", "n_scores", "work")] + \
            [_in_order(path, res["path_off"], res["path_len"], s["walks"])]
    if kind == "cigar":
        ops, coff, clen = gwfa.cigar_dev(ctx, graph, s["batch"], s["out"])
        return [_in_order(ops.view(np.int32), coff, clen, s["ops"]), clen]
    if kind == "plan":
        gwfa.pack_dev(ctx, s["batch"], s["out"].err)
        s["plan"].launch()
        s["plan"].finish()
    elif kind == "seeded":
        gwfa.step_dev(ctx, graph, s["batch"], s["out"], o, v_end=s["at"][0], start_off=s["at"][1],
                      start_hi=s["at"][2])
    else:
        gwfa.step_dev(ctx, graph, s["batch"], s["out"], o)
    return _fields(s["out"].res, n)


def work(case):
    """Inputs read once and outputs written once; the network's products."""
    if case["kind"] in ("train", "logits"):
        n = case["samples"]
        mac = 8 * 64 + 64 * 64 + 64
        if case["kind"] == "logits":
            return dict(bytes=n * (32 + 4) + 2 * N_PARAM, flops=2 * mac * n)
        return dict(bytes=n * 33 + N_PARAM * (2 + 2 + 4 + 6 * 4), flops=2 * (2 * mac + 64 * 64 + 64) * n)
    n = case.get("reads", 1)
    bases = n * case["len"]
    s = SHAPES[case["shape"]]
    # a read touches its own stretch of the graph: packed labels along it
    graph = min(bases, s["backbone_len"]) / 4
    if case["kind"] == "cigar":
        # packed reads, walks and results in; about two operations per error out
        ops = 2 * bases * (case["err_lo"] + case["err_hi"]) / 2 + n
        return dict(bytes=bases / 4 + graph + 64 * n + 4 * ops + 12 * n, flops=0)
    return dict(bytes=bases * 1.5 + graph + 64 * n, flops=0)


# --------------------------------------------------------------------------
# the network in 64 bits (activations rounded to bfloat16 where the network
# is defined to)
# --------------------------------------------------------------------------
def _bf(x):
    return x.to(torch.float32).to(torch.bfloat16).double()


def _forward(f, wb):
    w = wb.view(torch.bfloat16).double()
    w1, b1, w2, b2, w3, b3 = (w[0:512].view(64, 8), w[512:576], w[576:4672].view(64, 64), w[4672:4736],
                              w[4736:4800], w[4800])
    x = _bf(f * torch.from_numpy(SCALE).to(f.device))
    a1 = x @ w1.T + b1
    h1 = _bf(a1.clamp(min=0))
    a2 = h1 @ w2.T + b2
    h2 = _bf(a2.clamp(min=0))
    return x, a1, h1, a2, h2, h2 @ w3 + b3, w2, w3


def exact(case, seed):
    if case["kind"] not in ("train", "logits"):
        return None            # whole numbers: the same for every correct run
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(seed)
    f, y = _features(case["samples"], gen, dev)
    w, m1, m2 = _params(gen, dev)
    wb = w.to(torch.bfloat16).view(torch.int16)
    x, a1, h1, a2, h2, z, w2, w3 = _forward(f, wb)
    if case["kind"] == "logits":
        return z
    n, pos = case["samples"], y != 0
    sp = torch.nn.functional.softplus
    loss = torch.where(pos, POS_WEIGHT * sp(-z), sp(z)).mean().view(1)
    dz = torch.where(pos, POS_WEIGHT * (torch.sigmoid(z) - 1), torch.sigmoid(z)) / n
    g2 = torch.where(a2 > 0, dz[:, None] * w3, torch.zeros_like(a2))
    g1 = torch.where(a1 > 0, g2 @ w2, torch.zeros_like(a1))
    grad = torch.cat([(g1.T @ x).reshape(-1), g1.sum(0), (g2.T @ h1).reshape(-1), g2.sum(0), h2.T @ dz,
                      dz.sum().view(1)])
    t = STEP0 + 1
    m1, m2 = 0.9 * m1.double() + 0.1 * grad, 0.999 * m2.double() + 0.001 * grad * grad
    master = w.double() - LR * (m1 / (1 - 0.9 ** t)) / ((m2 / (1 - 0.999 ** t)).sqrt() + 1e-8)
    return dict(grad=grad, loss=loss, master=master, m1=m1, m2=m2, weights=master)
