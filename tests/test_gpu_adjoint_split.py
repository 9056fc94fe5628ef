"""The differentiable update over all pairs at the edges of its split: fewer
rows than a wave, remainders of waves and chunks, one and many chunks, both
types, the widths with the update and dS in one pass and in two, against the
formulas in FP64."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def exact(X, S, h, G):
    dx = X[:, None, :, :] - S[:, :, None, :]                       # b m n d
    w = np.exp(-(dx ** 2).sum(3) / (2 * h * h))
    W = w.sum(2)
    delta = (w[..., None] * dx).sum(2) / W[..., None]
    gdx = (G[:, :, None, :] * dx).sum(3) - (G * delta).sum(2)[..., None]
    beta = w * gdx / (h * h * W[..., None])
    dS = (beta[..., None] * dx).sum(2)
    dX = ((w / W[..., None])[..., None] * G[:, :, None, :] - beta[..., None] * dx).sum(1)
    return S + delta, dS, dX


# rounding of a few hundred terms of weight <= 1 whose exponents stay under 32:
# 32 eps each on the scale of the array's largest value, and room for the sums
TOL = {torch.float32: 2e-5, torch.float64: 1e-13}


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("d", [1, 3, 8, 13, 16, 32, 33, 64])
@pytest.mark.parametrize("nb,n,m", [(1, 1, 1), (2, 63, 65), (1, 129, 64), (3, 257, 31), (1, 700, 513), (1, 40, 1001)])
def test_split(dtype, d, nb, n, m):
    from paper_2112_13891_amd import api
    rng = np.random.default_rng(1000 * d + n)
    h = 0.6 * np.sqrt(d)
    X = rng.standard_normal((nb, n, d))
    S = rng.standard_normal((nb, m, d)) * 0.8
    G = rng.standard_normal((nb, m, d))
    Xt, St, Gt = (torch.tensor(a, dtype=dtype, device="cuda") for a in (X, S, G))
    want = exact(*(t.cpu().numpy().astype(np.float64) for t in (Xt, St)), h, Gt.cpu().numpy().astype(np.float64))
    S1 = api.forward_update(Xt, St, h)
    dS, dX = api.step_adjoint(Xt, St, h, Gt)
    for name, got, ref in zip(("S'", "dS", "dX"), (S1, dS, dX), want):
        scale = max(np.abs(ref).max(), np.abs(G).max())
        err = np.abs(got.cpu().numpy() - ref).max() / scale
        assert err < TOL[dtype], (name, err)
    again = api.step_adjoint(Xt, St, h, Gt)
    assert torch.equal(again[0], dS) and torch.equal(again[1], dX)
