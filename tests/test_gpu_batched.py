"""GPU parity of ms_step_batched -- many independent clouds of uneven size in
one launch per kernel -- against the FP64 oracle run on each cloud alone."""
import sys

import numpy as np
import pytest

from parity import ragged_check, step_parity

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2112_13891_amd import api, workloads  # noqa: E402

DEV = "cuda:0"


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def _batch(seed, sizes, d, max_seeds=150):
    """Clouds of the batched recipe (2..40 clusters, sigma 0.4 around centres
    N(0, 9 I)) with the given sizes; seeds drawn from each cloud's points."""
    rng = np.random.default_rng(seed)
    Xs, Ss = [], []
    for n in sizes:
        if n == 0:
            Xs.append(np.zeros((0, d), np.float32))
            Ss.append(np.zeros((0, d), np.float32))
            continue
        X, _, _ = workloads.cloud16(rng, n, d)
        m = int(min(n, rng.integers(0, max_seeds + 1)))
        Xs.append(X)
        Ss.append(X[rng.choice(n, m, replace=False)] if m else np.zeros((0, d), np.float32))
    xo = np.concatenate([[0], np.cumsum([len(x) for x in Xs])]).astype(np.int64)
    so = np.concatenate([[0], np.cumsum([len(s) for s in Ss])]).astype(np.int64)
    return Xs, Ss, xo, so


def _run(Xs, Ss, xo, so, h, kernel, n_iter, converged=None):
    Xa = torch.from_numpy(np.concatenate(Xs)).to(DEV)
    Sa = torch.from_numpy(np.concatenate(Ss)).to(DEV)
    return api.step_batched(Xa, xo, Sa, so, h, kernel=kernel, n_iter=n_iter, converged=converged)


SIZES = [1, 2, 300, 0, 1500, 64, 2047, 4100, 17, 1025]


@pytest.mark.parametrize("d", [2, 3, 16])
@pytest.mark.parametrize("kernel", ["gaussian", "flat"])
def test_batched_fixed_iterations(orc, d, kernel):
    Xs, Ss, xo, so = _batch(d * 10 + (kernel == "flat"), SIZES, d)
    h = 1.0
    for n_iter in (1, 3):
        S, conv, it, sh = _run(Xs, Ss, xo, so, h, kernel, n_iter)
        torch.cuda.synchronize()
        S, it, conv = S.cpu().numpy(), it.cpu().numpy(), conv.cpu().numpy()
        for c in range(len(Xs)):
            a, b = so[c], so[c + 1]
            if a == b:
                continue
            ref, ost, oit, osh = orc.step(Xs[c], Ss[c].astype(np.float64), h, kernel, tol=1e-3,
                                          n_iter=n_iter)
            ties = ragged_check(orc, Xs[c], Ss[c], h, kernel, n_iter, S[a:b], it[a:b], conv[a:b], ref, oit, ost)
            if ties:
                say("cloud", c, "flat boundary ties", ties)


@pytest.mark.parametrize("kernel", ["gaussian", "flat"])
def test_batched_to_convergence(orc, kernel):
    Xs, Ss, xo, so = _batch(77, SIZES, 3)
    h = 1.0
    S, conv, it, sh = _run(Xs, Ss, xo, so, h, kernel, 100)
    torch.cuda.synchronize()
    S, conv, it = S.cpu().numpy(), conv.cpu().numpy(), it.cpu().numpy()
    for c in range(len(Xs)):
        a, b = so[c], so[c + 1]
        if a == b:
            continue
        rep = step_parity(orc, Xs[c], Ss[c], h, kernel, 1e-3, S[a:b], it[a:b], conv[a:b])
        say("cloud", c, rep)


def test_batched_keeps_converged_seeds_and_matches_single_cloud_calls():
    Xs, Ss, xo, so = _batch(5, [500, 3000, 40], 16)
    M = int(so[-1])
    rng = np.random.default_rng(1)
    conv0 = (rng.random(M) < 0.3).astype(np.uint8)
    S, conv, it, sh = _run(Xs, Ss, xo, so, 1.0, "gaussian", 2,
                           converged=torch.from_numpy(conv0).to(DEV))
    torch.cuda.synchronize()
    S, conv, it = S.cpu().numpy(), conv.cpu().numpy(), it.cpu().numpy()
    S0 = np.concatenate(Ss)
    kept = conv0 == 1
    assert np.array_equal(S[kept], S0[kept]) and (it[kept] == 0).all() and (conv[kept] == 1).all()
    # the same seeds through ms_step, one cloud at a time
    for c in range(len(Xs)):
        a, b = so[c], so[c + 1]
        Sc, cc, ic, _ = api.step(torch.from_numpy(Xs[c]).to(DEV), torch.from_numpy(Ss[c]).to(DEV), 1.0,
                                 n_iter=2, converged=torch.from_numpy(conv0[a:b]).to(DEV))
        torch.cuda.synchronize()
        assert np.array_equal(ic.cpu().numpy(), it[a:b])
        assert np.abs(Sc.cpu().numpy() - S[a:b]).max() < 1e-5


def test_batched_uneven_clouds_workload_shape():
    """A slice of the batched recipe (clouds of 1,000..65,536 points, D = 16):
    every seed moves toward its own cloud's mass and never leaves its cloud's
    bounding box (a seed fed another cloud's points would)."""
    clouds = workloads.clouds16(seed=3, n_clouds=24)
    Xs = [c[0] for c in clouds]
    rng = np.random.default_rng(0)
    Ss = [X[rng.choice(len(X), min(len(X), 64), replace=False)] for X in Xs]
    xo = np.concatenate([[0], np.cumsum([len(x) for x in Xs])]).astype(np.int64)
    so = np.concatenate([[0], np.cumsum([len(s) for s in Ss])]).astype(np.int64)
    S, conv, it, sh = _run(Xs, Ss, xo, so, 1.0, "gaussian", 50)
    torch.cuda.synchronize()
    S = S.cpu().numpy()
    for c in range(len(Xs)):
        lo, hi = Xs[c].min(0), Xs[c].max(0)
        seg = S[so[c]:so[c + 1]]
        assert ((seg >= lo - 1e-4) & (seg <= hi + 1e-4)).all(), c
    assert conv.cpu().numpy().mean() > 0.9


def test_batched_graph_matches_eager_launches():
    """graph=1 captures the iterations as one HIP graph: every call, with
    eager work and synchronisations between the calls, gives bitwise the
    outputs of the kernel-by-kernel launches of the same call."""
    cases = [(_batch(31, SIZES, 3), "gaussian", 7), (_batch(32, SIZES[:6], 16), "flat", 3),
             (_batch(33, [4100, 1, 2047], 2), "gaussian", 25)]
    for rep in range(2):
        for (Xs, Ss, xo, so), kernel, n_iter in cases:
            say("graph case", len(Xs), "clouds", kernel, "n_iter", n_iter, "rep", rep)
            Xa = torch.from_numpy(np.concatenate(Xs)).to(DEV)
            Sa = torch.from_numpy(np.concatenate(Ss)).to(DEV)
            ref = api.step_batched(Xa, xo, Sa, so, 1.0, kernel=kernel, n_iter=n_iter)
            torch.cuda.synchronize()
            ref = [t.cpu() for t in ref]
            # unrelated eager work on the same stream between the two calls
            api.step(Xa, Sa[:5].contiguous(), 1.0, n_iter=2)
            junk = torch.randn(4096, device=DEV).cumsum(0)
            torch.cuda.synchronize()
            got = api.step_batched(Xa, xo, Sa, so, 1.0, kernel=kernel, n_iter=n_iter, graph=True)
            torch.cuda.synchronize()
            for a, b in zip(ref, got):
                torch.testing.assert_close(b.cpu(), a, rtol=0, atol=0, equal_nan=True)
            del junk


def test_batched_graph_reused_across_calls():
    """The executable graph is kept per thread and updated in place by a later
    call of the same topology (other clouds, other buffers), so it is
    instantiated once per shape; every launch gives bitwise the outputs of the
    kernel-by-kernel launches of the same call."""
    api.release_workspace()   # no kept graph on this thread
    i0, u0 = api.graph_stats()

    def run(seed, n_iter):
        Xs, Ss, xo, so = _batch(seed, SIZES[:8], 3)
        Xa = torch.from_numpy(np.concatenate(Xs)).to(DEV)
        Sa = torch.from_numpy(np.concatenate(Ss)).to(DEV)
        ref = [t.cpu() for t in api.step_batched(Xa, xo, Sa, so, 1.0, n_iter=n_iter, tile_R=1)]
        got = api.step_batched(Xa, xo, Sa, so, 1.0, n_iter=n_iter, tile_R=1, graph=True)
        torch.cuda.synchronize()
        for a, b in zip(ref, got):
            torch.testing.assert_close(b.cpu(), a, rtol=0, atol=0, equal_nan=True)
        return api.graph_stats()

    assert run(61, 5) == (i0 + 1, u0)       # instantiated
    assert run(62, 5) == (i0 + 1, u0 + 1)   # same topology, other data: updated in place
    assert run(63, 5) == (i0 + 1, u0 + 2)
    assert run(64, 6) == (i0 + 2, u0 + 2)   # one more iteration: another graph
    say("graph instantiations and updates", api.graph_stats())


@pytest.mark.parametrize("d,Rs", [(2, (1, 2, 4)), (8, (1, 2)), (16, (1, 2)), (32, (1,))])
def test_batched_tile_shapes_give_identical_results(d, Rs):
    """The seeds per lane change how seeds share a workgroup, never the order
    in which a seed's sums are formed: every shape gives the same bits."""
    Xs, Ss, xo, so = _batch(40 + d, SIZES, d, max_seeds=300)
    Xa = torch.from_numpy(np.concatenate(Xs)).to(DEV)
    Sa = torch.from_numpy(np.concatenate(Ss)).to(DEV)
    outs = []
    for R in Rs:
        say("tile_R", R, "d", d)
        outs.append([t.cpu() for t in api.step_batched(Xa, xo, Sa, so, 1.0, n_iter=4, tile_R=R)])
        torch.cuda.synchronize()
    for o in outs[1:]:
        for a, b in zip(outs[0], o):
            torch.testing.assert_close(b, a, rtol=0, atol=0, equal_nan=True)
    if 4 not in Rs:
        with pytest.raises(api.MeanShiftError, match="tile_R"):
            api.step_batched(Xa, xo, Sa, so, 1.0, n_iter=1, tile_R=4)


def test_batched_tuner_picks_a_built_shape():
    """The tuner searches seeds per lane, points per chunk and the step grid;
    later calls on inputs of the same kind take its shape, the grid never
    changes a bit of the results, and the caller's seeds are not written."""
    Xs, Ss, xo, so = _batch(50, SIZES, 3, max_seeds=300)
    Xa = torch.from_numpy(np.concatenate(Xs)).to(DEV)
    Sa = torch.from_numpy(np.concatenate(Ss)).to(DEV)
    S_before = Sa.cpu().clone()
    best, ms, chunk, grid = api.tune_batched(Xa, xo, Sa, so, 1.0, trials=3)
    say("tuned R", best, ms, "chunk", chunk, "grid", grid)
    assert best in (1, 2, 4) and set(ms) == {1, 2, 4} and all(v > 0 for v in ms.values())
    assert chunk in (512, 1024, 2048, 4096) and grid in (1024, 2048, 4096)
    assert torch.equal(Sa.cpu(), S_before)   # the caller's seeds are not written
    got = [t.cpu() for t in api.step_batched(Xa, xo, Sa, so, 1.0, n_iter=5)]
    explicit = [t.cpu() for t in api.step_batched(Xa, xo, Sa, so, 1.0, n_iter=5, tile_R=best,
                                                  tile_chunk=chunk, tile_grid=grid)]
    other_grid = [t.cpu() for t in api.step_batched(Xa, xo, Sa, so, 1.0, n_iter=5, tile_R=best,
                                                    tile_chunk=chunk, tile_grid=7 if grid != 7 else 9)]
    for a, b, c in zip(explicit, got, other_grid):
        torch.testing.assert_close(b, a, rtol=0, atol=0, equal_nan=True)
        torch.testing.assert_close(c, a, rtol=0, atol=0, equal_nan=True)


@pytest.mark.parametrize("chunk", [64, 512, 4096, 65536])
def test_batched_chunk_size_changes_rounding_only(chunk):
    """The points per chunk group each seed's sums differently: after a few
    iterations (no convergence decisions: tol 1e-30) the seeds agree with the
    default chunking to within the FP32 rounding of the sums."""
    Xs, Ss, xo, so = _batch(70, SIZES, 8, max_seeds=200)
    Xa = torch.from_numpy(np.concatenate(Xs)).to(DEV)
    Sa = torch.from_numpy(np.concatenate(Ss)).to(DEV)
    ref = api.step_batched(Xa, xo, Sa, so, 1.0, tol=1e-30, n_iter=3, tile_chunk=1024)[0].cpu().numpy()
    got = api.step_batched(Xa, xo, Sa, so, 1.0, tol=1e-30, n_iter=3, tile_chunk=chunk)[0].cpu().numpy()
    err = float(np.abs(got.astype(np.float64) - ref).max())
    say("chunk", chunk, "largest difference to 1024-point chunks", err)
    assert err <= 1e-4 * 1.0


def test_batched_full_size_sampled(orc):
    """The batched workload at full size (512 clouds of 1,000..65,536 points,
    D = 16, min(n, 256) seeds per cloud), in the launch shape the bench
    times: after 3 iterations, the seeds of sampled clouds (the smallest,
    the largest and two others) against the oracle run on each cloud alone."""
    clouds = workloads.clouds16(seed=0)
    Xs = [c[0] for c in clouds]
    rng = np.random.default_rng(0)
    Ss = [X[rng.choice(len(X), min(len(X), 256), replace=False)] for X in Xs]
    xo = np.concatenate([[0], np.cumsum([len(x) for x in Xs])]).astype(np.int64)
    so = np.concatenate([[0], np.cumsum([len(s) for s in Ss])]).astype(np.int64)
    say("full-size batched", len(Xs), "clouds", int(xo[-1]), "points")
    S, conv, it, sh = _run(Xs, Ss, xo, so, 1.0, "gaussian", 3)
    torch.cuda.synchronize()
    S, it, conv = S.cpu().numpy(), it.cpu().numpy(), conv.cpu().numpy()
    sizes = np.array([len(x) for x in Xs])
    for c in sorted({int(sizes.argmin()), int(sizes.argmax()), 100, 400}):
        a, b = so[c], so[c + 1]
        ref, ost, oit, osh = orc.step(Xs[c], Ss[c].astype(np.float64), 1.0, "gaussian", tol=1e-3, n_iter=3)
        say("cloud", c, "n", len(Xs[c]))
        ragged_check(orc, Xs[c], Ss[c], 1.0, "gaussian", 3, S[a:b], it[a:b], conv[a:b], ref, oit, ost)


@pytest.mark.parametrize("sizes,d", [(SIZES[:8], 4), ([20000], 16), (SIZES[2:7], 32)])
def test_batched_graph_of_the_seed_form(sizes, d):
    """Without a launch shape the updates are one launch of all clouds' seeds
    (two for one cloud of d >= 16): with graph=1 that is captured, kept,
    updated in place by later calls of any clouds and iteration count, and done
    when the call returns; the bits are those of the plain launch."""
    api.release_workspace()
    i0, u0 = api.graph_stats()
    for rep, n_iter in enumerate((5, 5, 2, 7)):
        Xs, Ss, xo, so = _batch(80 + rep, sizes, d, max_seeds=1500)
        Xa = torch.from_numpy(np.concatenate(Xs)).to(DEV)
        Sa = torch.from_numpy(np.concatenate(Ss)).to(DEV)
        ref = [t.cpu() for t in api.step_batched(Xa, xo, Sa, so, 1.0, n_iter=n_iter)]
        got = api.step_batched(Xa, xo, Sa, so, 1.0, n_iter=n_iter, graph=True)
        torch.cuda.synchronize()
        for a, b in zip(ref, got):
            torch.testing.assert_close(b.cpu(), a, rtol=0, atol=0, equal_nan=True)
        i, u = api.graph_stats()
        assert (i + u) - (i0 + u0) == rep + 1   # every call ran its updates as a graph
    assert api.graph_stats()[0] > i0
