"""GPU: weights that are not finite reach the samples whose inputs they
multiply, and no others: batch logits and the gradient against numpy with the
same rules (a product of zero and infinity is not a number, a ReLU of that is 0)."""
import numpy as np
import pytest

from oracle import mlp_ref as M
from tests.test_gpu_mlp_edges import SCALE, G, _case  # noqa: F401 (G: fixture)

pytestmark = pytest.mark.gpu
INF = float("inf")


def _bits(ctx, w):
    """The bfloat16 values w, infinities among them."""
    u = (np.asarray(w, np.float32).view(np.uint32) >> 16).astype(np.uint16)
    return ctx.torch.from_numpy(u.view(np.int16).copy()).to(ctx.tdev)


def _layers(w, x):
    W1, b1, W2, b2, W3, b3 = M.unpack(w)
    with np.errstate(all="ignore"):
        a1 = (x[:, None, :] * W1[None]).sum(-1) + b1
        h1 = np.fmax(a1, 0.0)
        a2 = (h1[:, None, :] * W2[None]).sum(-1) + b2
        h2 = np.fmax(a2, 0.0)
        return (h2 * W3).sum(-1) + b3


@pytest.mark.parametrize("at", [0, 3, 511, 520])
def test_logits_of_infinite_weights(G, at):  # noqa: F811
    """One first-layer weight (520: a bias) infinite: where its input is positive
    the unit is, where it is negative the unit is 0."""
    gw, ctx = G
    torch = ctx.torch
    for value in (INF, -INF):
        for n in (1, 16, 17, 64, 1000):
            w, _, f, _ = _case(n, 8, 0, 7100 + n)
            w[at] = value
            unit = at // 8 if at < 512 else at - 512
            w[M.O_W2 + unit:M.O_B2:64] = 1.0        # no zero meets the infinite unit
            w[M.O_W3:M.O_B3] = 0.125
            out = torch.full((n,), 7.0, dtype=torch.float32, device=ctx.tdev)
            gw.mlp_logits_dev(ctx, torch.from_numpy(f).to(ctx.tdev), SCALE, _bits(ctx, w), out)
            z = out.cpu().numpy()
            assert np.array_equal(z, _layers(w, M.inputs(f, SCALE)).astype(np.float32), equal_nan=True), (value, n)


@pytest.mark.parametrize("n", [1, 15, 16, 17, 63, 64, 65])
def test_gradient_of_an_infinite_weight_no_sample_meets(G, n):  # noqa: F811
    """Unit 5 of layer 1 is off for every sample (a positive bias, a negative
    input), so its infinite weight into unit 7 of layer 2 turns that unit off as
    well and meets no gradient: the gradient is finite, as without the two
    units, whatever the rows that fill up the last tile hold."""
    gw, ctx = G
    torch = ctx.torch
    w, _, f, y = _case(n, 8, 0, 7200 + n)
    f[:, 0] = -2.0 - np.abs(f[:, 0])
    W1, b1, W2, b2, W3, b3 = [a.copy() for a in M.unpack(w)]
    W1[5], b1[5] = 0.0, 1.0
    W1[5, 0] = 4.0
    W2[7], b2[7], W2[:, 5] = 0.0, -1.0, 0.0
    grads = []
    for value in (0.0, INF):
        W2[7, 5] = value
        grad = torch.full((M.N_PARAM,), 7.0, dtype=torch.float32, device=ctx.tdev)
        loss = torch.full((1,), 7.0, dtype=torch.float32, device=ctx.tdev)
        gw.mlp_grad_dev(ctx, torch.from_numpy(f).to(ctx.tdev), torch.from_numpy(y).to(ctx.tdev), SCALE,
                        _bits(ctx, np.concatenate([W1.ravel(), b1, W2.ravel(), b2, W3, [b3]])), grad, loss,
                        pos_weight=3.0)
        grads.append(np.append(grad.cpu().numpy(), loss.cpu().numpy()))
    assert np.isfinite(grads[0]).all() and np.array_equal(grads[0], grads[1])
