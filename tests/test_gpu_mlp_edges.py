"""Gradient and logits of the pruning network at the edges of the kernels'
tiles: 16 samples a step, 64 a workgroup or wave, 16,384 in one pass of the
gradient's workgroups; rows of 8, 9 and 16 floats, aligned or not.

Weights and inputs are small integers (and eighths), so that every sum of
the forward pass is exact in float32 and every activation a bfloat16 value:
logits are equal, and the gradient differs from the float64 reference only
by float32 arithmetic of the loss (about 10 rounding errors a sample, 6e-8
each) and of its sums, which average out: 5e-6 of the gradient's norm."""
import numpy as np
import pytest

from oracle import mlp_ref as M

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G(gpu_lib):
    ctx = gpu_lib.Context(0)
    yield gpu_lib, ctx
    ctx.close()


def _case(n, stride, lead, seed):
    rng = np.random.default_rng(seed)
    w = np.zeros(M.N_PARAM)
    w[M.O_W1:M.O_B1] = rng.integers(-1, 2, 512)
    w[M.O_B1:M.O_W2] = rng.integers(-1, 3, 64)
    W2 = np.zeros((64, 64))
    for j in range(64):
        W2[j, rng.choice(64, 4, replace=False)] = rng.choice([-1.0, 1.0, 0.5], 4)
    w[M.O_W2:M.O_B2] = W2.ravel()
    w[M.O_B2:M.O_W3] = rng.integers(-1, 2, 64)
    w[M.O_W3:M.O_B3] = rng.choice([-1.0, 1.0], 64) / 8
    w[M.O_B3] = 0.25
    buf = rng.normal(size=lead + n * stride).astype(np.float32)      # what lies between the rows is not read
    f = buf[lead:].reshape(n, stride)
    f[:, :8] = rng.integers(-4, 5, size=(n, 8))
    return w, buf, f[:, :8].copy(), (rng.random(n) < 0.3).astype(np.uint8)


SCALE = np.full(8, 0.5, np.float32)
SIZES = [1, 15, 16, 17, 63, 64, 65, 255, 256, 257, 1023, 16383, 16384, 16385, 40001]


def _bits(ctx, w):
    return ctx.torch.from_numpy(M.bf16_bits(w).view(np.int16).copy()).to(ctx.tdev)


@pytest.mark.parametrize("stride,lead", [(8, 0), (9, 0), (16, 0), (8, 1), (12, 2)])
def test_gradient_at_the_tile_edges(G, stride, lead):
    gw, ctx = G
    torch = ctx.torch
    for n in SIZES:
        w, buf, f, y = _case(n, stride, lead, 7000 + n)
        tf = torch.from_numpy(buf).to(ctx.tdev)[lead:].view(n, stride)
        grad = torch.full((M.N_PARAM,), 7.0, dtype=torch.float32, device=ctx.tdev)
        loss = torch.full((1,), 7.0, dtype=torch.float32, device=ctx.tdev)
        gw.mlp_grad_dev(ctx, tf, torch.from_numpy(y).to(ctx.tdev), SCALE, _bits(ctx, w), grad, loss, pos_weight=3.0)
        torch.cuda.synchronize()
        l_ref, g_ref = M.loss_and_grad(w, M.inputs(f, SCALE), y, 3.0)
        g = grad.cpu().numpy().astype(np.float64)
        rel = np.linalg.norm(g - g_ref) / np.linalg.norm(g_ref)
        print(f"[gpu-mlp] n={n} stride={stride}: gradient {rel:.1e}, loss {float(loss.item()):.6f} {l_ref:.6f}", flush=True)
        assert rel <= 5e-6 and abs(float(loss.item()) - l_ref) <= 5e-6 * l_ref


def test_gradient_of_no_samples_is_zero(G):
    gw, ctx = G
    torch = ctx.torch
    grad = torch.full((M.N_PARAM,), 7.0, dtype=torch.float32, device=ctx.tdev)
    loss = torch.full((1,), 7.0, dtype=torch.float32, device=ctx.tdev)
    gw.mlp_grad_dev(ctx, torch.zeros((1, 8), device=ctx.tdev), torch.zeros(1, dtype=torch.uint8, device=ctx.tdev),
                    SCALE, _bits(ctx, np.zeros(M.N_PARAM)), grad, loss, n=0)
    torch.cuda.synchronize()
    assert not grad.any() and not loss.any()


@pytest.mark.parametrize("stride,lead", [(8, 0), (9, 0), (16, 0), (8, 1), (12, 2)])
def test_logits_at_the_tile_edges(G, stride, lead):
    gw, ctx = G
    torch = ctx.torch
    for n in SIZES + [262143, 262144, 262209]:
        w, buf, f, _ = _case(n, stride, lead, 8000 + n)
        tf = torch.from_numpy(buf).to(ctx.tdev)[lead:].view(n, stride)
        out = torch.full((n + 64,), 7.0, dtype=torch.float32, device=ctx.tdev)
        gw.mlp_logits_dev(ctx, tf, SCALE, _bits(ctx, w), out, n=n)
        torch.cuda.synchronize()
        z = out.cpu().numpy()
        zr, _ = M.forward(w, M.inputs(f, SCALE))
        assert np.array_equal(z[:n], zr.astype(np.float32)), (n, stride)
        assert (z[n:] == 7.0).all()
