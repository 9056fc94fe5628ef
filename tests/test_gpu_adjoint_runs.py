"""The FP32 differentiable form over pivot runs against the FP64 autograd
reference: sizes from which the runs are used, dimensions padded and exact,
seeds that are the points and seeds that are not, several clouds, data with
nothing to leave out, and what is added into the caller's arrays."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2112_13891_amd import api  # noqa: E402

DEV = "cuda:0"


def _ref(X, S, h, G):
    """S', dL/dS and dL/dX of one update in FP64 (the whole matrix, on the GPU)."""
    X, S, G = X.double(), S.double(), G.double()
    q = (S * S).sum(1)[:, None] + (X * X).sum(1)[None, :] - 2.0 * (S @ X.T)   # FP64: 1e-13 of |x|^2
    w = torch.exp(-q.clamp_(min=0.0) / (2 * h * h))
    p = w / w.sum(1, keepdim=True)
    new = p @ X
    beta = p * (G @ X.T - (G * new).sum(1, keepdim=True)) / (h * h)
    dS = beta @ X - beta.sum(1, keepdim=True) * S
    dX = p.T @ G + beta.T @ S - beta.sum(0)[:, None] * X
    return new, dS, dX


def _cloud(seed, n, d, k, spread=3.0, sigma=0.4):
    g = torch.Generator(device=DEV).manual_seed(seed)
    c = spread * torch.randn(k, d, generator=g, device=DEV)
    y = torch.randint(0, k, (n,), generator=g, device=DEV)
    return (c[y] + sigma * torch.randn(n, d, generator=g, device=DEV)).contiguous()


def _close(got, ref, what):
    # sums of a few thousand FP32 terms, each with some ulps of exp2 and of its
    # distance: 1e-5 of the largest entry is ten times their worst case
    err = (got.double() - ref).abs().max().item() / ref.abs().max().item()
    assert err < 1e-5, (what, err)


# nb n m above 2^27
@pytest.mark.parametrize("nb,n,m,d,k", [(1, 12000, 12000, 3, 15), (2, 8192, 8192, 16, 20), (1, 16385, 8200, 13, 7),
                                        (3, 7001, 6500, 8, 12), (1, 11700, 11700, 32, 30), (1, 11700, 11700, 4, 1),
                                        (1, 150001, 900, 16, 40)])
def test_runs_update_and_adjoint(nb, n, m, d, k):
    X = torch.stack([_cloud(10 * n + d + b, n, d, k) for b in range(nb)])
    same = m == n
    S = X if same else torch.stack([_cloud(7 * m + d + b, m, d, k) + 0 for b in range(nb)])
    if not same:   # seeds near the points: a subset, moved a little
        S = (X[:, :m] + 0.3 * torch.sin(torch.arange(m * d, device=DEV, dtype=torch.float32).view(m, d))).contiguous()
    G = torch.randn(nb, m, d, device=DEV, generator=torch.Generator(device=DEV).manual_seed(1))
    new = api.forward_update(X, S, 1.0)
    dS, dX = api.step_adjoint(X, S, 1.0, G)
    for b in range(nb):
        rn, rS, rX = _ref(X[b], S[b], 1.0, G[b])
        _close(new[b], rn, "update")
        _close(dS[b], rS, "dS")
        _close(dX[b], rX, "dX")


def test_runs_nothing_left_out_and_accumulates():
    """A bandwidth as wide as the data: every pair counts.  The gradients are
    added to what the arrays hold, also where dS is dX (S is X)."""
    X = _cloud(3, 11700, 6, 1, sigma=1.0)
    G = torch.randn(11700, 6, device=DEV, generator=torch.Generator(device=DEV).manual_seed(2))
    rn, rS, rX = _ref(X, X, 2.0, G)
    _close(api.forward_update(X, X, 2.0), rn, "update")
    both = torch.full_like(X, 0.25)
    api.step_adjoint_accumulate(X, X, 2.0, G, both, both)
    _close(both, rS + rX + 0.25, "dS + dX")


def test_runs_repeat_bitwise():
    X = _cloud(5, 12000, 16, 20)
    G = torch.randn(12000, 16, device=DEV, generator=torch.Generator(device=DEV).manual_seed(3))
    a = api.step_adjoint(X, X, 1.0, G)
    b = api.step_adjoint(X, X, 1.0, G)
    assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
    assert torch.equal(api.forward_update(X, X, 1.0), api.forward_update(X, X, 1.0))


def test_runs_non_finite_point():
    """A point that is not finite reaches every seed, as without runs."""
    X = _cloud(6, 12000, 16, 20)
    X[500, 2] = float("nan")
    assert int(torch.isfinite(api.forward_update(X, X.clone(), 1.0)).all(1).sum()) == 0


@pytest.mark.parametrize("nb,n,m,d", [(2, 8192, 8192, 16), (1, 12000, 11500, 3)])   # nb n m above 2^27: both over runs
def test_planned_calls_same_bits(nb, n, m, d):
    X = torch.stack([_cloud(31 + b, n, d, 12) for b in range(nb)])
    S = X if m == n else X[:, :m].contiguous()
    G = torch.randn(nb, m, d, device=DEV, generator=torch.Generator(device=DEV).manual_seed(4))
    plan = api.points_plan(X, 1.0)
    assert plan is not None
    assert torch.equal(api.forward_update(X, S, 1.0, plan), api.forward_update(X, S, 1.0))
    out = [(torch.zeros_like(S), torch.zeros_like(X)) for _ in range(2)]
    for (dS, dX), p in zip(out, (plan, None)):
        api.step_adjoint_accumulate(X, S, 1.0, G, dS, dX, p)
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
    with pytest.raises(api.MeanShiftError, match="plan"):
        api.forward_update(X, S, 2.0, plan)
    with pytest.raises(api.MeanShiftError, match="plan"):
        api.forward_update(X[:, :-1].contiguous(), S, 1.0, plan)
    with pytest.raises(ValueError, match="plan"):
        api.forward_update(X, S, 1.0, plan.data)


@pytest.mark.parametrize("d,bad", [(16, [float("inf")]), (16, [float("inf"), float("-inf")]), (3, [float("inf")]),
                                   (8, [3e38, 3e38]), (8, [3e30, 3e30])])
def test_runs_infinite_point_shares_a_run(d, bad):
    """Points that are not finite lie in one run with far points; neither may
    be left out.  An infinite coordinate makes that coordinate of every update of
    its cloud NaN (0 inf) and with it all gradients, as over all pairs, and
    leaves the other cloud alone; a finite one whose distance
    overflows weighs nothing, and the far points beside it keep their weight."""
    X = torch.stack([_cloud(6, 8200, d, 20), _cloud(7, 8200, d, 20)])
    X[0, 100:140] += 400.0 * torch.arange(1, 41, device=DEV, dtype=torch.float32)[:, None]   # far, one by one
    clean = X.clone()
    for i, v in enumerate(bad):
        X[0, 500 + i, 1] = v
    S = clean.clone()
    G = torch.randn(2, 8200, d, device=DEV, generator=torch.Generator(device=DEV).manual_seed(5))
    new = api.forward_update(X, S, 1.0)
    dS, dX = api.step_adjoint(X, S, 1.0, G)
    rn, rS, rX = _ref(clean[1], S[1], 1.0, G[1])
    _close(new[1], rn, "update")
    _close(dS[1], rS, "dS")
    _close(dX[1], rX, "dX")
    keep = torch.ones(8200, dtype=torch.bool, device=DEV)
    keep[500:500 + len(bad)] = False
    rn, rS, rX = _ref(clean[0][keep], S[0], 1.0, G[0])
    if not np.isfinite(bad).all():
        assert not torch.isfinite(new[0][:, 1]).any()
        other = [k for k in range(d) if k != 1]
        _close(new[0][:, other], rn[:, other], "update")
        assert not torch.isfinite(dS[0]).any() and not torch.isfinite(dX[0]).any()
        return
    _close(new[0], rn, "update")
    if max(bad) < 1e38:   # else g.dx overflows in FP32, in every form
        _close(dS[0], rS, "dS")
        _close(dX[0][keep], rX, "dX")


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("d,k,m", [(16, 15, 8200), (16, 9, 8300), (32, 31, 8200)])
def test_runs_not_finite_in_the_second_half(d, k, m, bad):
    """A point with a coordinate that is not finite counts for every seed and
    every gradient of its cloud, also by a coordinate in the second half of a
    distance: finite where the all-pairs form (FP64) is."""
    X = torch.stack([_cloud(6, 8200, d, 20), _cloud(7, 8200, d, 20)])
    S = torch.cat([X, X], 1)[:, :m].contiguous()
    X[0, 500, k] = bad
    G = torch.randn(2, m, d, device=DEV, generator=torch.Generator(device=DEV).manual_seed(5))
    new = api.forward_update(X, S, 1.0)
    dS, dX = api.step_adjoint(X, S, 1.0, G)
    ref = api.forward_update(X.double(), S.double(), 1.0)
    rS, rX = api.step_adjoint(X.double(), S.double(), 1.0, G.double())
    for a, b in ((new, ref), (dS, rS), (dX, rX)):
        assert torch.equal(torch.isfinite(a), torch.isfinite(b))
        assert not torch.isfinite(b[0]).all() and torch.isfinite(b[1]).all()


@pytest.mark.parametrize("nb,n,m,d,values", [(2, 16384, 8192, 32, 7), (1, 16384, 16384, 16, 7), (2, 16384, 8192, 13, 2),
                                             (1, 32768, 8192, 8, 2)])
def test_runs_repeated_points_keep_the_sums(nb, n, m, d, values):
    """Points of few values, all within reach: additions of equal terms round
    the same way, by about 7e-9 of the sum each, so that a lane's error grows
    with its additions in a row.  256 rows and a few folds in a row make at most
    2e-6 of a sum and of W, 4e-6 of an update; all 2,048 of a wave were 1.5e-5."""
    g = torch.Generator(device=DEV).manual_seed(n + d)
    V = 4.0 * torch.randn(values, d, device=DEV, generator=g)
    X = V[torch.randint(values, (nb, n), device=DEV, generator=g)].contiguous()
    h = 3.0 * d ** 0.5
    S = X[:, torch.randint(n, (m,), device=DEV, generator=g)] + 0.2 * h * torch.randn(nb, m, d, device=DEV, generator=g)
    G = torch.randn(nb, m, d, device=DEV, generator=g)
    new = api.forward_update(X, S, h)
    dS, dX = api.step_adjoint(X, S, h, G)
    ref = api.forward_update(X.double(), S.double(), h)
    rS, rX = api.step_adjoint(X.double(), S.double(), h, G.double())
    assert ((new - S) - (ref - S.double())).norm() <= 4e-6 * (ref - S.double()).norm()
    assert (dS - rS).norm() <= 3e-6 * G.norm() and (dX - rX).norm() <= 1e-6 * G.norm()


# either side of the lines between the two forms: points of the least cloud,
# tiles of the smaller side, more seeds than points, pairs
@pytest.mark.parametrize("nb,n,m,d", [(2, 8192, 8192, 8), (3, 8300, 8195, 5), (2, 8191, 8191, 8), (1, 8192, 20000, 3),
                                      (1, 65536, 8192, 16), (1, 65536, 8191, 16), (16, 2048, 4096, 16),
                                      (16, 2047, 4200, 16), (32, 2100, 2100, 29), (300, 500, 500, 16),
                                      (4100, 129, 130, 16), (70000 // 2, 33, 62, 3)])
def test_lines_between_runs_and_all_pairs(nb, n, m, d):
    X = _cloud(n + d, nb * n, d, 12).view(nb, n, d)
    S = _cloud(n + d, nb * m, d, 12).view(nb, m, d) if m != n else X
    G = torch.randn(nb, m, d, device=DEV, generator=torch.Generator(device=DEV).manual_seed(6))
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    new = api.forward_update(X, S, 1.0)
    dS, dX = api.step_adjoint(X, S, 1.0, G)
    torch.cuda.synchronize()
    # no more memory than a few hundred copies of the rows' partial sums
    assert free - torch.cuda.mem_get_info()[0] < (1 << 29) + 64 * 4 * (nb * (n + m) * d)
    for b in sorted({0, nb // 2, nb - 1}):
        rn, rS, rX = _ref(X[b], S[b], 1.0, G[b])
        _close(new[b], rn, "update")
        # the rounding of a distance q/2 is the weight's times q/2: without a
        # point within 3 h a seed's own gradient is off by more than its sums
        s64, x64 = S[b].double(), X[b].double()
        near = ((s64 * s64).sum(1)[:, None] + (x64 * x64).sum(1) - 2.0 * s64 @ x64.T).min(1)[0] < 9.0
        assert int(near.sum()) * 2 > m
        _close(dS[b][near], rS[near], "dS")
        _close(dX[b], rX, "dX")
