"""The wide step by a screen of the pairs (padded d = 64, 128, 256): parity with
the FP64 oracle over padded and exact dimensions, both kernels, remainders of
words, seed tiles and lists; every pair within reach; seeds far from all points;
rows that are not finite; the cosine metric; and the same results where the
fixed scratch of ms_step_noalloc is too small for the screen."""
import numpy as np
import pytest

from parity import ragged_check

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2112_13891_amd import api  # noqa: E402

DEV = "cuda:0"


def _gpu(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def embed(seed, n, d, k):
    rng = np.random.default_rng(seed)
    C = 4.0 * rng.standard_normal((k, d))
    X = C[rng.integers(0, k, n)] + 0.5 * rng.standard_normal((n, d))
    far = rng.random(n) < 0.05
    X[far] = rng.uniform(-12.0, 12.0, (int(far.sum()), d))
    return np.ascontiguousarray(X, dtype=np.float32)


@pytest.mark.parametrize("d,n,m", [(33, 64, 1), (64, 65, 31), (63, 1, 1), (100, 1000, 33), (128, 16384, 64),
                                   (128, 16385, 32), (129, 3001, 97), (200, 2047, 16), (256, 20000, 130)])
@pytest.mark.parametrize("kernel", ["gaussian", "flat"])
def test_screen_step(orc, d, n, m, kernel):
    X = embed(n + d, n, d, max(1, min(20, n // 50)))
    S0 = X[np.random.default_rng(m).choice(n, m, replace=False)]
    h = 1.5 * np.sqrt(d / 32.0) * (1.0 if kernel == "gaussian" else 2.0)
    S, conv, it, sh = api.step(_gpu(X), _gpu(S0), h, kernel=kernel, n_iter=3)
    torch.cuda.synchronize()
    ref, ost, oit, osh = orc.step(X, S0.astype(np.float64), h, kernel, tol=1e-3, n_iter=3)
    ragged_check(orc, X, S0, h, kernel, 3, S.cpu().numpy(), it.cpu().numpy(), conv.cpu().numpy(), ref, oit, ost)


@pytest.mark.parametrize("d", [64, 128, 250])
@pytest.mark.parametrize("metric", ["euclidean", "cosine"])
def test_screen_all_near(d, metric):
    """One cluster: every pair is kept; and the list of a seed spans segments."""
    rng = np.random.default_rng(d)
    X = (3.0 + 0.3 * rng.standard_normal((40000, d))).astype(np.float32)
    S0 = np.ascontiguousarray(X[:70])
    h = 1.0 if metric == "euclidean" else 0.3
    a = api.step(_gpu(X), _gpu(S0), h, n_iter=2, metric=metric)
    b = api.step(_gpu(X), _gpu(S0), h, n_iter=2, metric=metric, plain=True)
    # two FP32 orders of the same sums of 40,000 terms
    assert float((a[0] - b[0]).abs().max() / b[0].abs().max()) < 5e-6
    assert torch.equal(a[2], b[2])


def test_screen_far_and_nonfinite():
    X = embed(5, 5000, 128, 10)
    S0 = np.ascontiguousarray(X[:40])
    S0[1] += 1000.0        # no point within reach: W = 0
    S0[2, 7] = np.nan
    S0[3, 9] = np.inf
    a = api.step(_gpu(X), _gpu(S0), 3.0, n_iter=2)
    b = api.step(_gpu(X), _gpu(S0), 3.0, n_iter=2, plain=True)
    assert torch.equal(a[1], b[1]) and torch.equal(a[2], b[2])
    ok = torch.ones(40, dtype=torch.bool, device=DEV)
    ok[1:4] = False
    assert float((a[0][ok] - b[0][ok]).abs().max()) < 1e-4
    # a row that is not finite reaches every seed, also as the first row
    for row, v in ((3000, np.inf), (0, np.nan), (4999, 3e30), (0, -np.inf)):
        Y = X.copy()
        Y[row, 5] = v
        a = api.step(_gpu(Y), _gpu(X[:40]), 3.0, n_iter=1)
        b = api.step(_gpu(Y), _gpu(X[:40]), 3.0, n_iter=1, plain=True)
        assert torch.equal(a[1], b[1]) and torch.equal(a[2], b[2]), (row, v)


@pytest.mark.parametrize("d,n,m", [(128, 40000, 64), (64, 90000, 64), (8, 520000, 64), (8, 400000, 64)])
def test_scratch_without_room(d, n, m):
    """More than the fixed scratch holds for the newer forms, not for the plain one."""
    X = embed(n, n, d, 30)
    S0 = np.ascontiguousarray(X[:m])
    h = 1.5 * np.sqrt(max(d, 8) / 32.0)
    try:
        a = api.step(_gpu(X), _gpu(S0), h, n_iter=1, noalloc=True, plain=True)
    except api.MeanShiftError:
        pytest.skip("the plain form does not fit either")
    b = api.step(_gpu(X), _gpu(S0), h, n_iter=1, noalloc=True)
    assert float((a[0] - b[0]).abs().max() / a[0].abs().max()) < 5e-6


def test_screen_fit_matches_plain():
    X = embed(11, 6000, 96, 6)
    X = X[np.abs(X).max(1) < 11.0]
    r = [api.fit(_gpu(X), 2.6, n_initial=64, rng_seed=3, plain=p) for p in (False, True)]
    assert r[0].modes.shape == r[1].modes.shape
    assert float((r[0].modes - r[1].modes).abs().max()) < 1e-3
    assert torch.equal(r[0].labels, r[1].labels)


@pytest.mark.parametrize("n,d,B", [(20001, 100, 256), (1500, 40, 512)])
def test_screen_fit_counts_each_pair_once(n, d, B):
    """The mask launch has a grid of points x seed tiles; each iteration's
    active seeds x points are counted once, whatever its second dimension."""
    X = embed(n + d, n, d, 12)
    g = api.fit(_gpu(X), 1.5 * np.sqrt(d / 32.0), n_initial=B, rng_seed=4, trace=True)
    assert (g.drawn_status != 2).all()
    assert g.pairs == int(g.drawn_iters.astype(np.int64).sum()) * n


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_screen_bound_at_the_worst_rounding(d, sign):
    """Pairs at the edge of a flat window, far from the first row, with every
    factor of the bf16 product rounded the same way as far as it goes: down
    from 1 + 2^-8 (the product is short by 2^-7 of |s|^2 + |x|^2, nearly the
    whole allowance) or up from 1 + 3 2^-8."""
    n, m = 4000, 96
    rng = np.random.default_rng(d)
    mag = 64.0 * (1.0 + (2.0 ** -8 if sign > 0 else 3.0 * 2.0 ** -8))
    X = np.zeros((n, d), np.float32)
    X[1:] = mag
    # neighbours differ in a few coordinates by the next binade's equally bad value
    for i in range(1, n):
        X[i, rng.choice(d, rng.integers(0, 6), replace=False)] *= 0.5
    S0 = np.ascontiguousarray(X[1:m + 1])
    # the window: the pairs that differ in at most 4 coordinates, in or just out
    for h in (0.5 * mag * 2.0, 0.5 * mag * 2.0 * (1 - 1e-6), 0.5 * mag):
        a = api.step(_gpu(X), _gpu(S0), h, kernel="flat", n_iter=1)
        b = api.step(_gpu(X), _gpu(S0), h, kernel="flat", n_iter=1, plain=True)
        assert torch.equal(a[1], b[1]) and torch.equal(a[2], b[2])
        # two orders of sums of up to 4,000 terms of FP32
        assert float((a[0] - b[0]).abs().max()) < 1e-5 * mag


@pytest.mark.parametrize("n,d,m", [(66382, 64, 4), (76426, 33, 40), (120001, 128, 12), (115371, 200, 1)])
def test_repeated_points_keep_the_sums(n, d, m):
    """Points of seven values, all within reach: the additions of equal terms
    round the same way, so that the error of a sum grows with the number of
    additions in a row.  One update against FP64, within 1.5 times the error of
    the form that evaluates every pair in short chunks, and 1e-6 h."""
    rng = np.random.default_rng(n + d)
    X = (4.0 * rng.standard_normal((7, d)))[rng.integers(0, 7, n)].astype(np.float32)
    h = 3.0 * np.sqrt(d)
    S0 = X[rng.choice(n, m, replace=False)] + (0.1 * h * rng.standard_normal((m, d))).astype(np.float32)
    val, cnt = np.unique(X, axis=0, return_counts=True)
    val, S64 = val.astype(np.float64), S0.astype(np.float64)
    w = cnt * np.exp(-0.5 * ((S64[:, None] - val[None]) ** 2).sum(-1) / h ** 2)
    ref = (w @ val) / w.sum(1, keepdims=True)
    err = []
    for plain in (False, True):
        S, conv, it, sh = api.step(_gpu(X), _gpu(S0), h, n_iter=1, plain=plain)
        err.append(np.abs(S.cpu().numpy() - ref).max() / h)
    assert err[0] <= 1.5 * err[1] + 1e-6, err


@pytest.mark.parametrize("value", [1.6e9, 1e12, -1e16])
@pytest.mark.parametrize("n,d,m,kernel", [(1, 64, 1, "gaussian"), (3001, 33, 97, "gaussian"), (5000, 128, 64, "flat")])
def test_column_of_one_large_value(n, d, m, kernel, value):
    """A column that holds one value throughout adds nothing to any distance,
    however large it is against h: the results are those without the column."""
    X = embed(n, n, d, 5)
    X[:, d // 2] = value
    S0 = X[np.random.default_rng(m).choice(n, m, replace=False)]
    h = 1.5 * np.sqrt(d / 32.0) * (1.0 if kernel == "gaussian" else 2.0)
    S, conv, it, sh = api.step(_gpu(X), _gpu(S0), h, kernel=kernel, n_iter=2)
    X[:, d // 2] = 0.0
    S0[:, d // 2] = 0.0
    R, rconv, rit, rsh = api.step(_gpu(X), _gpu(S0), h, kernel=kernel, n_iter=2)
    assert torch.equal(conv, rconv) and torch.equal(it, rit)
    assert (S[:, d // 2] == value).all()
    S[:, d // 2] = 0.0
    assert (S - R).abs().max().item() <= 1e-5 * h
