"""GPU: weights that are not finite reach the samples whose inputs they
multiply, and no others: batch logits against numpy with the same
rules (a product of zero and infinity is not a number, a ReLU of that is 0)."""
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
