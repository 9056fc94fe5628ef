"""GPU parity of the seed-per-workgroup form (d <= 4) against the FP64 oracle at
the edges of its tiles, lists and groups: point counts around a 64-point tile,
around the 16,384 points from which the points are ordered, and past the 6,144
tiles that one list holds; one seed per workgroup and four; a seed far from
every point, whose nearest weights are far below those of the other seeds."""
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


def blobs(seed, n, d, k=12, box=60.0):
    rng = np.random.default_rng(seed)
    C = rng.uniform(0.0, box, (k, d))
    return np.ascontiguousarray(C[rng.integers(0, k, n)] + rng.standard_normal((n, d)), dtype=np.float32)


@pytest.mark.parametrize("n,m", [(1, 1), (63, 5), (64, 64), (65, 65), (3000, 2048), (3000, 2049), (16384, 513),
                                 (16447, 2051), (393217, 9), (400001, 2050)])
@pytest.mark.parametrize("d", [1, 3, 4])
@pytest.mark.parametrize("kernel", ["gaussian", "flat"])
def test_seed_form_edges(orc, n, m, d, kernel):
    if n * m > 10 ** 8 and (d != 3 or kernel != "gaussian"):
        pytest.skip("one large shape is enough for the oracle")
    X = blobs(n + d, n, d)
    S0 = X[np.random.default_rng(m).choice(n, m, replace=False)]
    check = np.arange(m) if n * m <= 10 ** 8 else np.array([0, 1, 2, 3, 1024, 2047, 2048, 2049])
    S, conv, it, sh = api.step(_gpu(X), _gpu(S0), 1.5, kernel=kernel, n_iter=2)
    torch.cuda.synchronize()
    ref, ost, oit, osh = orc.step(X, S0[check].astype(np.float64), 1.5, kernel, tol=1e-3, n_iter=2)
    ragged_check(orc, X, S0[check], 1.5, kernel, 2, S.cpu().numpy()[check], it.cpu().numpy()[check],
                 conv.cpu().numpy()[check], ref, oit, ost)


@pytest.mark.parametrize("n", [500, 20000])
def test_seed_form_far_seed(orc, n):
    """Seeds 5, 9 and 13 h beyond the last point: W is about 2^-18, 2^-58 and
    2^-122, and the nearest points alone decide the update.  The last one is
    held to the plain FP32 form: next to its W the other weights fall below
    FP32's smallest normal number, which every FP32 form drops."""
    X = blobs(3, n, 2)
    top = X[np.argmax(X[:, 0])].astype(np.float64)
    S0 = np.stack([top + np.array([g * 1.5, 0.0]) for g in (5.0, 9.0, 13.0)]).astype(np.float32)
    S, conv, it, sh = api.step(_gpu(X), _gpu(S0), 1.5, n_iter=1)
    P, pconv, pit, psh = api.step(_gpu(X), _gpu(S0), 1.5, n_iter=1, plain=True)
    torch.cuda.synchronize()
    ref, ost, oit, osh = orc.step(X, S0.astype(np.float64), 1.5, "gaussian", tol=1e-3, n_iter=1)
    assert np.array_equal(it.cpu().numpy(), oit)
    # the exponent of a weight is q <= 130 with FP32 rounding: 1e-5 of it, on
    # shifts of up to 13 h
    err = np.abs(S.cpu().numpy() - ref)
    assert err[:2].max() < 1e-4 * 1.5
    assert (S - P).abs().max().item() < 1e-4 * 1.5


def test_seed_form_repeats_bitwise():
    X = _gpu(blobs(9, 50000, 3))
    for m in (200, 3000):
        a = api.step(X, X[:m].clone(), 1.5, n_iter=6)
        b = api.step(X, X[:m].clone(), 1.5, n_iter=6)
        assert all(torch.equal(u.nan_to_num(), v.nan_to_num()) if u.is_floating_point() else torch.equal(u, v)
                   for u, v in zip(a, b))


def test_seed_form_non_finite_point():
    """A point that is not finite is seen by every seed, as without an order:
    every seed fails."""
    for n in (2000, 20000):
        X = blobs(4, n, 3)
        X[n // 2, 1] = np.inf
        S, conv, it, sh = api.step(_gpu(X), _gpu(X[:50]), 1.5, n_iter=2)
        torch.cuda.synchronize()
        assert (conv.cpu().numpy() == 2).all()


@pytest.mark.parametrize("m,d", [((1 << 21) + 77, 5), ((1 << 25) + 5, 5), ((1 << 26) + 3, 2)])
def test_seed_form_more_seeds_than_a_launch(m, d):
    """Past 2^21 workgroups the seeds go in several launches (2^32 threads are
    the most a launch takes): seeds that repeat give the first ones' bits."""
    n = 300
    X = torch.randn(n, d, device=DEV, generator=torch.Generator(device=DEV).manual_seed(d)).contiguous()
    j = torch.arange(m, device=DEV) % n
    S, conv, it, sh = api.step(X, X[j], 1.0, n_iter=2)
    few = api.step(X, X, 1.0, n_iter=2, plain=True)[0]
    assert float((S[:n] - few).abs().max()) < 1e-5
    assert torch.equal(S, S[:n][j]) and torch.equal(it, it[:n][j]) and torch.equal(conv, conv[:n][j])


def test_step_store_past_2_32_coordinates():
    """m d > 2^32 coordinates of seeds in one call."""
    m, d = (1 << 24) + 1, 256
    X = torch.zeros(2, d, device=DEV)
    X[1, 0] = 0.5
    S, conv, it, sh = api.step(X, X[:1].expand(m, d).contiguous(), 1.0, n_iter=1)
    assert int(it.min()) == 1 and torch.equal(S[-1], S[0])
    assert float(S[-1, 0]) == pytest.approx(0.5 * np.exp(-0.125) / (1 + np.exp(-0.125)), rel=1e-5)


@pytest.mark.parametrize("d,n,m", [(2, 1001, 200), (2, 20001, 64), (16, 20001, 1000), (128, 5001, 64)])
@pytest.mark.parametrize("unit", [1e18, 1e-20])
def test_flat_window_of_any_size(d, n, m, unit):
    """The tiles' padding (points at 1e19) never falls into a window, and no
    bound is taken in units where bf16 products underflow."""
    rng = np.random.default_rng(d)
    X = rng.uniform(-0.1, 0.1, (n, d))
    X[:, 0] = rng.uniform(-9.0, 9.0, n)
    if d == 2:
        X[:, 1] = rng.uniform(-9.0, 9.0, n)
    X = torch.from_numpy((unit * X).astype(np.float32)).to(DEV)
    S = X[torch.topk(X[:, 0], m).indices].contiguous()   # the seeds nearest to the padding
    a = api.step(X, S, 3.0 * unit, kernel="flat", n_iter=1)
    b = api.step(X, S, 3.0 * unit, kernel="flat", n_iter=1, plain=True)
    assert int(b[2].min()) == 1 and torch.equal(a[2], b[2])
    assert float((a[0] - b[0]).abs().max()) < 1e-5 * unit * 9.0


# either side of the lines on seeds a workgroup (512, 1,024, 2,048 seeds; 2^19
# points) and of the one on few seeds over very many points
@pytest.mark.parametrize("n,m,d", [(524288, 1024, 3), (524288, 2049, 3), (524289, 512, 2), (524289, 513, 1),
                                   (530001, 1023, 2), (530001, 1024, 4), (530001, 1025, 3), (524289, 2047, 2),
                                   (524289, 2048, 4), (524289, 2049, 1), (1048577, 256, 3), (1048577, 257, 2)])
@pytest.mark.parametrize("kernel", ["gaussian", "flat"])
def test_seeds_that_share_a_workgroup(n, m, d, kernel):
    X = _gpu(blobs(n + d, n, d, k=40, box=300.0))
    S = X[torch.randperm(n, device=DEV, generator=torch.Generator(device=DEV).manual_seed(m))[:m]].contiguous()
    h = 1.5 if kernel == "gaussian" else 2.5
    a = api.step(X, S, h, kernel=kernel, n_iter=2, tol=1e-30)
    b = api.step(X, S, h, kernel=kernel, n_iter=2, tol=1e-30, plain=True)
    assert torch.equal(a[1], b[1]) and torch.equal(a[2], b[2])
    # a window's edge is decided after one rounding on either side: a few points
    # of 10^3 to 10^4 in a window may differ after the first update
    tol = 1e-4 if kernel == "gaussian" else 2e-3
    assert float((a[0] - b[0]).abs().max()) < tol * h


# points, dimension, seeds (12 positions, repeated): rows, runs that share a
# seed, a seed per wave
@pytest.mark.parametrize("n,d,m", [(262144, 1, 12), (200000, 3, 600), (1100000, 2, 1200), (50000, 8, 24),
                                   (50000, 16, 12), (50000, 16, 2400), (70881, 24, 12), (70881, 24, 2400)])
def test_repeated_points_keep_the_sums(n, d, m):
    """Points of seven values, all within reach: the additions of equal terms
    round the same way, so that the error of a sum grows with the number of
    additions in a row.  One update against FP64, within 1.5 times the error of
    the form that evaluates every pair in short chunks, and 1e-6 h."""
    rng = np.random.default_rng(n + d)
    X = (4.0 * rng.standard_normal((7, d)))[rng.integers(0, 7, n)].astype(np.float32)
    h = 5.0 * np.sqrt(d)
    P = X[rng.choice(n, 12, replace=False)] + (0.1 * h * rng.standard_normal((12, d))).astype(np.float32)
    val, cnt = np.unique(X, axis=0, return_counts=True)
    val, P64 = val.astype(np.float64), P.astype(np.float64)
    w = cnt * np.exp(-0.5 * ((P64[:, None] - val[None]) ** 2).sum(-1) / h ** 2)
    ref = (w @ val) / w.sum(1, keepdims=True)
    S0 = np.tile(P, (m // 12, 1))
    err = []
    for plain in (False, True):
        S, conv, it, sh = api.step(_gpu(X), _gpu(S0), h, n_iter=1, plain=plain)
        err.append(np.abs(S.cpu().numpy().reshape(m // 12, 12, d) - ref).max() / h)
    assert err[0] <= 1.5 * err[1] + 1e-6, err


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
@pytest.mark.parametrize("d,k", [(16, 15), (13, 12), (16, 8), (24, 17), (32, 31), (32, 2)])
@pytest.mark.parametrize("kernel", ["gaussian", "flat"])
def test_point_not_finite_in_either_half(d, k, kernel, bad):
    """A point with a coordinate that is not finite fails every seed of its
    cloud, whichever half of a distance holds the coordinate, and no seed of
    another cloud.  Status, updates and coordinates as by all pairs."""
    X = blobs(d, 20000, d, box=30.0)
    S0 = X[np.random.default_rng(1).choice(20000, 300, replace=False)]
    clean = X.copy()
    X[777, k] = bad
    h = 1.5 * np.sqrt(d / 4.0)
    S, conv, it, sh = api.step(_gpu(X), _gpu(S0), h, kernel=kernel, n_iter=2)
    P, pconv, pit, psh = api.step(_gpu(X), _gpu(S0), h, kernel=kernel, n_iter=2, plain=True)
    assert (pconv == 2).all()
    assert torch.equal(conv, pconv) and torch.equal(it, pit)
    assert torch.equal(torch.isfinite(S), torch.isfinite(P))
    both = api.step_batched(_gpu(np.concatenate([X, clean])), [0, 20000, 40000], _gpu(np.concatenate([S0, S0])),
                            [0, 300, 600], h, kernel=kernel, n_iter=2)
    assert (both[1][:300] == 2).all() and (both[1][300:] != 2).all()


@pytest.mark.parametrize("d,n", [(1, 2), (2, 100), (3, 5000), (5, 100), (16, 5000), (32, 20000)])
@pytest.mark.parametrize("at", [0, 1])
@pytest.mark.parametrize("last", [False, True])
def test_packed_coordinate_that_overflows(d, n, at, last):
    """A finite coordinate that overflows in packed units (3e38, h = 0.5) fails
    the seeds of its cloud as an infinite one does, also where the point is the
    cloud's first row, which the index takes distances from."""
    X = blobs(d, n, d, k=2, box=2.0)
    S0 = X[:2].copy()
    X[at, d - 1 if last else 0] = 3e38
    P, pconv, pit, psh = api.step(_gpu(X), _gpu(S0), 0.5, n_iter=1, plain=True)
    for S, conv, it, sh in (api.step(_gpu(X), _gpu(S0), 0.5, n_iter=1),
                            api.step_batched(_gpu(X), [0, n], _gpu(S0), [0, 2], 0.5, n_iter=1)):
        assert torch.equal(conv, pconv) and torch.equal(it, pit)
    assert (pconv == 2).all()


@pytest.mark.parametrize("d,n", [(5, 100), (16, 5000), (32, 20000)])
@pytest.mark.parametrize("value", [1e17, 1e19, -1e20])
def test_seed_and_point_far_beyond_the_others(d, n, value):
    """A seed and one point share a coordinate far beyond any pivot: the point
    alone moves the seed, however far the pivots are."""
    X = blobs(d, n, d, k=2, box=2.0)
    S0 = X[3:4].copy()
    X[7, d - 1] = value
    S0[0, d - 1] = value
    h = 3.0 * np.sqrt(d)
    P, pconv, pit, psh = api.step(_gpu(X), _gpu(S0), h, n_iter=1, plain=True)
    for S, conv, it, sh in (api.step(_gpu(X), _gpu(S0), h, n_iter=1),
                            api.step_batched(_gpu(X), [0, n], _gpu(S0), [0, 1], h, n_iter=1)):
        assert torch.equal(conv, pconv) and torch.equal(it, pit)
        assert (S - P)[:, :-1].abs().max().item() <= 1e-5 * h
    assert (pconv != 2).all()
