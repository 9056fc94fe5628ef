"""Labels by candidates from the matrix cores (d > 4, 64 or 128 modes or more) against
FP64 distances: padded and exact dimensions, tails of points and modes,
coincident modes (lowest index), points whose candidate list overflows, data
far from the origin, and values that are not finite."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2112_13891_amd import api  # noqa: E402

DEV = "cuda:0"


def _data(seed, n, k, d, offset=0.0):
    rng = np.random.default_rng(seed)
    C = 4.0 * rng.standard_normal((40, d))
    X = C[rng.integers(0, 40, n)] + 0.5 * rng.standard_normal((n, d)) + offset
    M = X[rng.integers(0, n, k)] + 0.05 * rng.standard_normal((k, d))
    return X.astype(np.float32), M.astype(np.float32)


def _check(X, M):
    lab, mg = api.assign(torch.from_numpy(X).to(DEV), torch.from_numpy(M).to(DEV), margin=True)
    lab2 = api.assign(torch.from_numpy(X).to(DEV), torch.from_numpy(M).to(DEV))
    torch.cuda.synchronize()
    lab, mg = lab.cpu().numpy(), mg.cpu().numpy()
    assert np.array_equal(lab, lab2.cpu().numpy())
    # FP32 direct differences round a squared distance by at most (d + 2) ulps
    tol = (X.shape[1] + 2) * 2.0 ** -23
    for a in range(0, len(X), 2048):
        q = ((X[a:a + 2048, None, :].astype(np.float64) - M[None].astype(np.float64)) ** 2).sum(2)
        near = np.partition(q, 1, axis=1)[:, :2]
        got = q[np.arange(len(q)), lab[a:a + 2048]]
        assert (got <= near[:, 0] * (1 + tol)).all()
        ref = np.sqrt(near[:, 1]) - np.sqrt(near[:, 0])
        assert (np.abs(mg[a:a + 2048] - ref) <= 2 * tol * np.sqrt(near[:, 1]) + 1e-30).all()


@pytest.mark.parametrize("d", [5, 8, 13, 16, 31, 32, 33, 64])
@pytest.mark.parametrize("n,k", [(1, 64), (257, 65), (257, 129), (3000, 100), (5001, 927)])
def test_labels_and_margins(d, n, k):
    X, M = _data(n + k + d, n, k, d)
    _check(X, M)


def test_far_from_the_origin():
    X, M = _data(1, 3000, 200, 32, offset=3000.0)
    _check(X, M)


def test_coincident_modes_take_the_lowest_index():
    X, M = _data(2, 2000, 80, 16)
    M = np.concatenate([M, M, M[:7]])                     # every mode twice or three times
    lab = api.assign(torch.from_numpy(X).to(DEV), torch.from_numpy(M).to(DEV)).cpu().numpy()
    assert lab.max() < 80
    _check(X, M)
    M = np.repeat(M[:1], 200, axis=0)                     # all alike: every list overflows
    lab = api.assign(torch.from_numpy(X).to(DEV), torch.from_numpy(M).to(DEV)).cpu().numpy()
    assert (lab == 0).all()


def test_values_that_are_not_finite():
    X, M = _data(3, 1000, 100, 32)
    want = api.assign(torch.from_numpy(X).to(DEV), torch.from_numpy(M).to(DEV)).cpu().numpy()
    Y, N = X.copy(), M.copy()
    Y[5, 3] = np.nan
    Y[9, 0] = np.inf
    dead = int(np.bincount(want).argmax())
    N[dead, 7] = np.nan                                   # never the nearest
    if dead == 0:
        pytest.skip("the reference mode itself")
    lab = api.assign(torch.from_numpy(Y).to(DEV), torch.from_numpy(N).to(DEV)).cpu().numpy()
    assert lab[5] == 0 and lab[9] == 0                    # no distance is a finite number
    keep = (want != dead) & (np.arange(1000) != 5) & (np.arange(1000) != 9)
    assert np.array_equal(lab[keep], want[keep]) and not (lab == dead).any()


@pytest.mark.parametrize("d", [8, 16, 32, 64])
@pytest.mark.parametrize("side", [0, 1])
def test_one_half_of_the_candidates_overflows(d, side):
    """The lanes l and l + 32 of a wave share a point and list the candidates of
    different rows of a mode tile (rows j % 8 below 4, and the others).  More
    alike modes than a list holds on one side only: both halves scan."""
    X, M = _data(4 + d, 700, 256, d)
    at = [j for j in range(256) if (j % 8 < 4) == (side == 0)]
    near = X[:1] + 1e-3 * np.random.default_rng(side).standard_normal((len(at), d)).astype(np.float32)
    M += 100.0                                            # the others are far
    M[at[3:40]] = near[3:40]
    _check(X, M)
    # alike to the last bit: the lowest index, of either parity
    for first in (at[3], at[4]):
        N = M.copy()
        N[at[3:40]] = M[0]
        N[[j for j in at[3:40] if j >= first]] = X[0]
        lab = api.assign(torch.from_numpy(X).to(DEV), torch.from_numpy(N).to(DEV)).cpu().numpy()
        q = ((X[:, None, :].astype(np.float64) - N[None].astype(np.float64)) ** 2).sum(2)
        assert (lab == q.argmin(1)).all()
