"""GPU parity of the seed form over pivot runs (5 <= d <= 32) against the FP64
oracle: padded and exact dimensions, both kernels, seeds below and above the
count from which they are ordered, clusters with outliers far from every pivot
(whose runs are left out by their distance bound alone), duplicated points
(pivots at one place), one pivot only, and data with nothing to leave out."""
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


def embed(seed, n, d, k=30, out=0.05):
    rng = np.random.default_rng(seed)
    C = 6.0 * rng.standard_normal((k, d))
    X = C[rng.integers(0, k, n)] + 0.5 * rng.standard_normal((n, d))
    far = rng.random(n) < out
    X[far] = rng.uniform(-20.0, 20.0, (int(far.sum()), d))
    return np.ascontiguousarray(X, dtype=np.float32)


def _check(orc, X, S0, h, kernel, n_iter, sample, precision="fp32"):
    S, conv, it, sh = api.step(_gpu(X), _gpu(S0), h, kernel=kernel, n_iter=n_iter, precision=precision)
    torch.cuda.synchronize()
    ref, ost, oit, osh = orc.step(X, S0[sample].astype(np.float64), h, kernel, tol=1e-3, n_iter=n_iter)
    ragged_check(orc, X, S0[sample], h, kernel, n_iter, S.cpu().numpy()[sample], it.cpu().numpy()[sample],
                 conv.cpu().numpy()[sample], ref, oit, ost)


# seeds x points x padded d x updates above 2^28: the runs are used
@pytest.mark.parametrize("d,n,m", [(5, 40001, 2000), (8, 40000, 2049), (13, 30000, 700), (16, 20011, 2500),
                                   (29, 20000, 500), (32, 16384, 2100)])
@pytest.mark.parametrize("kernel", ["gaussian", "flat"])
@pytest.mark.parametrize("precision", ["fp32", "bf16"])
def test_runs_step(orc, d, n, m, kernel, precision):
    X = embed(n + d, n, d)
    S0 = X[np.random.default_rng(m).choice(n, m, replace=False)]
    sample = np.random.default_rng(1).choice(m, 64, replace=False)
    _check(orc, X, S0, 1.2, kernel, 2, sample, precision)


def test_runs_far_seeds(orc):
    """Seeds between the clusters and among the outliers, not on points."""
    X = embed(7, 40000, 16)
    rng = np.random.default_rng(2)
    S0 = np.ascontiguousarray(X[:1500] + rng.uniform(-4.0, 4.0, (1500, 16)), dtype=np.float32)
    S, conv, it, sh = api.step(_gpu(X), _gpu(S0), 1.2, n_iter=1)
    P, pconv, pit, psh = api.step(_gpu(X), _gpu(S0), 1.2, n_iter=1, plain=True)
    torch.cuda.synchronize()
    # against the plain FP32 form, which evaluates every pair: the same seeds
    # fail (every weight 0), the others move alike (1e-4 h, the parity bound)
    assert torch.equal(conv == 2, pconv == 2)
    ok = conv != 2
    assert (S - P)[ok].abs().max().item() < 1e-4 * 1.2


def test_runs_duplicates_and_single_pivot(orc):
    rng = np.random.default_rng(5)
    base = embed(11, 40, 8, out=0.0)
    X = np.ascontiguousarray(np.repeat(base, 1000, axis=0)[rng.permutation(40000)])   # pivots at one place
    S0 = np.ascontiguousarray(X[:2100] + 0.1 * rng.standard_normal((2100, 8)), dtype=np.float32)
    _check(orc, X, S0, 1.2, "gaussian", 2, np.arange(40))
    X = embed(12, 300, 32)                                                             # one pivot, m n D > 2^28
    S0 = np.ascontiguousarray(np.repeat(X, 60, axis=0) + 0.1, dtype=np.float32)
    _check(orc, X, S0, 1.2, "gaussian", 2, np.arange(0, len(S0), 300))


def test_runs_nothing_left_out(orc):
    """One broad blob whose every pair counts."""
    rng = np.random.default_rng(6)
    X = np.ascontiguousarray(rng.standard_normal((20000, 16)), dtype=np.float32)
    for m in (900, 2100):
        S0 = X[:m] * np.float32(1.5)
        _check(orc, X, S0, 3.0, "gaussian", 1, np.arange(0, m, 50))


def test_runs_repeats_bitwise_and_non_finite():
    X = _gpu(embed(9, 50000, 16))
    for m in (600, 3000):
        a = api.step(X, X[:m].clone(), 1.2, n_iter=3)
        b = api.step(X, X[:m].clone(), 1.2, n_iter=3)
        assert all(torch.equal(u.nan_to_num(), v.nan_to_num()) if u.is_floating_point() else torch.equal(u, v)
                   for u, v in zip(a, b))
    for bad in (float("nan"), float("inf")):
        Y = X.clone()
        Y[777, 3] = bad   # seen by every seed, as without runs: every seed fails
        S, conv, it, sh = api.step(Y, X[1000:1600].clone(), 1.2, n_iter=2)
        torch.cuda.synchronize()
        assert int((conv != 2).sum()) == 0


@pytest.mark.parametrize("d", [8, 32])
def test_dense_rows(orc, d):
    """Few pairs: every tile is evaluated, in the rows' order."""
    for n, m in ((1, 1), (64, 3), (65, 65), (1000, 300)):
        X = embed(n + d, n, d, k=5)
        S0 = np.ascontiguousarray(X[:m])
        _check(orc, X, S0, 1.2, "gaussian", 2, np.arange(m))


@pytest.mark.parametrize("d,ncl,n_each,m,few", [(2, 40, 40000, 30, 3), (3, 40, 40000, 20, 2), (8, 30, 40000, 40, 2),
                                                (16, 45, 32000, 10, 3)])
def test_batched_both_sides_of_the_line(d, ncl, n_each, m, few):
    """A batched step that is large enough for the tile form against the same
    clouds in a small call, which runs over their pivot runs."""
    X = np.concatenate([embed(100 + c, n_each - 7 * c, d, 20, 0.0) for c in range(ncl)])
    off = np.concatenate([[0], np.cumsum([n_each - 7 * c for c in range(ncl)])])
    rng = np.random.default_rng(d)
    S0 = np.concatenate([X[off[c] + rng.choice(n_each - 7 * c, m, replace=False)] for c in range(ncl)])
    so = np.arange(ncl + 1) * m
    Xg, Sg = _gpu(X), _gpu(S0)
    a = api.step_batched(Xg, off, Sg, so, 1.2, n_iter=2)
    b = api.step_batched(Xg[:off[few]].contiguous(), off[:few + 1], Sg[:so[few]].contiguous(), so[:few + 1], 1.2,
                         n_iter=2)
    k = few * m
    assert torch.equal(a[1][:k], b[1]) and torch.equal(a[2][:k], b[2])
    # two FP32 orders of sums over a cluster of 2,000 points, coordinates up to 30
    assert float((a[0][:k] - b[0]).abs().max()) < 1e-4


@pytest.mark.parametrize("d,n,m,k", [(16, 30001, 511, 1), (16, 30001, 512, 2), (16, 20000, 2050, 3), (32, 20000, 514, 1),
                                     (32, 16385, 2061, 2), (29, 30000, 1001, 4)])
@pytest.mark.parametrize("kernel", ["gaussian", "flat"])
def test_runs_many_tiles_in_reach(orc, d, n, m, k, kernel):
    """Few clusters: a seed per wave from 512 seeds on, remainders of a workgroup's four."""
    X = embed(n + d + k, n, d, k)
    S0 = X[np.random.default_rng(m).choice(n, m, replace=False)]
    sample = np.concatenate([np.arange(8), np.random.default_rng(1).choice(m, 24, replace=False), np.arange(m - 8, m)])
    _check(orc, X, S0, 1.2, kernel, 2, sample)


@pytest.mark.parametrize("d", [3, 16, 32])
def test_cosine_all_within_reach(d):
    """Directions with every pair within reach: a small call and one above its line."""
    rng = np.random.default_rng(d)
    X = rng.standard_normal((30000, d)).astype(np.float32)
    S0 = np.ascontiguousarray(X[:1500])
    a = api.step(_gpu(X), _gpu(S0), 0.4, n_iter=2, metric="cosine")
    b = api.step(_gpu(X), _gpu(S0[:5]), 0.4, n_iter=2, metric="cosine")
    p = api.step(_gpu(X), _gpu(S0), 0.4, n_iter=2, metric="cosine", plain=True)
    assert float((a[0] - p[0]).abs().max()) < 1e-5 and float((a[0][:5] - b[0]).abs().max()) < 1e-5


@pytest.mark.parametrize("d,ncl,n_each,m,n_iter,few", [(2, 40, 40000, 30, 1, 2), (3, 40, 40000, 20, 1, 2),
                                                       (8, 30, 40000, 200, 3, 1), (16, 1500, 100, 60, 2, 20),
                                                       (29, 1500, 100, 60, 2, 20)])
def test_batched_calls_that_keep_the_tile_form(d, ncl, n_each, m, n_iter, few):
    """Calls for which the index or a workgroup per seed costs more than it
    saves, against their first clouds alone, which run over their pivot runs;
    and both against an explicit launch shape, which always takes the tiles."""
    c = np.random.default_rng(d).uniform(0.0, 30.0, (20, d))
    rng = np.random.default_rng(d + 1)
    sizes = n_each - rng.integers(0, 9, ncl)
    off = np.concatenate([[0], np.cumsum(sizes)])
    X = (c[rng.integers(0, 20, off[-1])] + 0.5 * rng.standard_normal((off[-1], d))).astype(np.float32)
    S0 = np.concatenate([X[a + rng.choice(k, m, replace=False)] for a, k in zip(off[:-1], sizes)])
    so = np.arange(ncl + 1) * m
    Xg, Sg = _gpu(X), _gpu(S0)
    a = api.step_batched(Xg, off, Sg, so, 1.2, n_iter=n_iter)
    tiles = api.step_batched(Xg, off, Sg, so, 1.2, n_iter=n_iter, tile_R=1, tile_chunk=1024, tile_grid=2048)
    for u, v in zip(a, tiles):
        torch.testing.assert_close(u, v, rtol=0, atol=0, equal_nan=True)   # R never changes the bits
    b = api.step_batched(Xg[:off[few]].contiguous(), off[:few + 1], Sg[:so[few]].contiguous(), so[:few + 1], 1.2,
                         n_iter=n_iter)
    k = few * m
    assert torch.equal(a[2][:k], b[2])
    # two FP32 orders of sums over a cluster of 2,000 points, coordinates up to 30
    assert float((a[0][:k] - b[0]).abs().max()) < 1e-4


@pytest.mark.parametrize("d,n,m,k", [(16, 30001, 1279, 1), (16, 30001, 1280, 2), (32, 20000, 831, 2),
                                     (32, 20000, 833, 1), (13, 30000, 1501, 4)])
@pytest.mark.parametrize("kernel", ["gaussian", "flat"])
def test_runs_many_tiles_in_reach_at_the_line(orc, d, n, m, k, kernel):
    """Either side of the seeds from which each wave takes one of its own."""
    test_runs_many_tiles_in_reach(orc, d, n, m, k, kernel)
