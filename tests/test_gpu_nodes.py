"""GPU: the full-band sums over interpolation nodes against the sums over every
bin and the FP64 oracle, at the edges of what the node tables cover."""
import math

import numpy as np
import pytest

import gwsynth
from oracle import likelihood as L
from tests.gpu_common import oracle_many, with_injection

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def gw():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    import paper_2607_28265_amd as gw
    return gw


def _rows(prob, n):
    """Prior draws with, at fixed places, rows at and beyond the tables' edges:
    chirp mass, delays on both sides, heavy binaries, extreme tides and spins,
    and a row that is not physical."""
    th = gwsynth.prior_draws(11, max(n, 1))
    for j, (col, val) in enumerate(((0, 1.05), (0, 0.9), (0, 3.0), (0, 30.0), (12, 0.1), (12, -0.1), (12, 0.16),
                                    (12, -0.3), (4, 2e4), (2, 0.9), (1, 0.05), (1, 1.0))):
        th[5 * j + 3:: 67, col] = val
    th[1::90, 1] = 2.0
    return th


def _tol(prob, th, ref):
    """Interpolation error 1e-13 of sum |u||A P| <= sqrt(N_f <d|d> <h|h>) in the
    overlap, which log L follows with slope at most 1, and rounding of the sums
    (a few hundred units in the last place of log L)."""
    ok = np.isfinite(ref)
    hh = max(L.overlap(t, prob)[1] for t in th[ok][:64])
    return (1e-13 * math.sqrt(prob.n_freq * L.data_inner(prob) * hh)
            + 512 * np.finfo(float).eps * np.max(np.abs(ref[ok])))


@pytest.mark.parametrize("n_det,grid,n", [(1, (4.0, 20.0, 256.0), 1), (2, (8.0, 20.0, 512.0), 65),
                                          (3, (16.0, 10.0, 512.0), 250), (4, (8.0, 30.0, 1024.0), 64),
                                          (3, (1.0, 20.0, 40.0), 130), (2, (0.25, 20.0, 400.0), 63)])
def test_nodes_match_bins_and_oracle(gw, n_det, grid, n):
    prob = gwsynth.make_problem(*grid, psd_scale=1e-47, n_det=n_det)
    prob = with_injection(prob, gwsynth.prior_draws(gwsynth.SEEDS["injection"], 1)[0])
    th = _rows(prob, n)
    t = torch.from_numpy(th).cuda()
    with gw.Context(prob) as ctx:
        nodes, tau = gw.gw_full_nodes(ctx.handle)
        assert 1 <= nodes <= prob.n_freq and 0.1 <= tau <= 0.25
        for marg in (L.PLAIN, L.PHASE, L.PHASE_DIST):
            ref = oracle_many(th, prob, marg)
            tol = _tol(prob, th, ref)
            ok = np.isfinite(ref)
            got = {}
            for kind in (0, 1):
                ctx.set_full_kernel(kind)
                got[kind] = ctx.loglike(t, marg=marg).cpu().numpy()
                assert np.array_equal(np.isfinite(got[kind]), ok)
            assert np.max(np.abs(got[0][ok] - got[1][ok])) < 2 * tol
            assert np.max(np.abs(got[0][ok] - ref[ok])) < 1e-6 + tol
            # the mixed form: 1.2e-10 a phasor, so at most that of the same sum
            ctx.set_full_kernel(0)
            mix = ctx.loglike(t, marg=marg, prec=1).cpu().numpy()
            assert np.max(np.abs(mix[ok] - ref[ok])) < 1e-3


@pytest.mark.parametrize("tpb,chunks", [(0, 0), (0, 3), (64, 5), (128, 24), (256, 64)])
def test_node_sums_independent_of_launch_shape(gw, tpb, chunks):
    prob = with_injection(gwsynth.make_problem(8.0, 20.0, 512.0, psd_scale=1e-47),
                          gwsynth.prior_draws(gwsynth.SEEDS["injection"], 1)[0])
    th = _rows(prob, 333)
    t = torch.from_numpy(th).cuda()
    with gw.Context(prob) as ctx:
        want = ctx.loglike(t, marg=L.PHASE).cpu().numpy()
        ctx.set_full_shape(tpb, chunks)
        got = ctx.loglike(t, marg=L.PHASE).cpu().numpy()
    ok = np.isfinite(want)
    assert np.array_equal(np.isfinite(got), ok)
    assert np.max(np.abs(got[ok] - want[ok])) < 512 * np.finfo(float).eps * np.max(np.abs(want[ok]))


@pytest.mark.parametrize("n_slots,n", [(1, 1), (70, 65), (600, 700)])
def test_cache_mixes_node_and_moment_rows(gw, n_slots, n):
    # slots in and out of the tables' phase range, and extrinsic moves with
    # delays on either side of each table's and of the cache's own limit
    prob = with_injection(gwsynth.make_problem(8.0, 20.0, 512.0, psd_scale=1e-47),
                          gwsynth.prior_draws(gwsynth.SEEDS["injection"], 1)[0])
    rng = np.random.default_rng(3)
    base = gwsynth.prior_draws(21, n_slots)
    base[1::3, 0] = 0.9
    slots = rng.integers(0, n_slots, n)
    th = base[slots].copy()
    ext = gwsynth.prior_draws(22, n)
    th[:, 6:11], th[:, 12] = ext[:, 6:11], ext[:, 12]
    th[3::7, 12] = 0.19
    th[5::9, 12] = -0.2
    th[4::11, 12] = 0.31
    dt = np.array([[abs(t[12] + d) for d in (-np.array([math.cos(t[9]) * math.cos(t[8]), math.cos(t[9]) * math.sin(t[8]),
                                                        math.sin(t[9])]) @ prob.det_pos.T / 299792458.0)] for t in th])
    beyond = dt.max(axis=1) > 0.25
    with gw.Context(prob) as ctx:
        cache = gw.WaveformCache(ctx.handle, n_slots)
        cache.update(torch.from_numpy(base).cuda(), torch.arange(n_slots, dtype=torch.int32, device="cuda"))
        got = cache.loglike(torch.from_numpy(th).cuda(), torch.from_numpy(slots.astype(np.int32)).cuda(), 1).cpu().numpy()
        ctx.set_full_kernel(1)
        want = ctx.loglike(torch.from_numpy(th).cuda(), marg=L.PHASE_DIST).cpu().numpy()
        cache.close()
    assert np.array_equal(np.isnan(got), beyond)
    # FP32 moments carry 6e-8 of the overlap, which is at most sqrt(<d|d> <h|h>)
    # and enters the distance marginal with slope below sqrt(<d|d>)-sized SNR^2
    assert np.max(np.abs(got - want)[~beyond]) < 6e-8 * L.data_inner(prob)


@pytest.mark.parametrize("n_det,grid,n,window,over", [
    (3, (64.0, 20.0, 2048.0), 65, 0.0, 0), (2, (32.0, 10.0, 1024.0), 64, 0.05, 1), (4, (16.0, 20.0, 1024.0), 63, 0.0, 2),
    (1, (8.0, 20.0, 512.0), 130, 0.12, 4), (3, (4.0, 30.0, 256.0), 1, 0.0, 0), (3, (128.0, 20.0, 512.0), 513, 0.0, 0)])
def test_time_moments_over_nodes(gw, n_det, grid, n, window, over):
    """Time marginal: nodes against bins, rows in and beyond the tables mixed
    (one launch holds both).  A grid value carries the interpolation error of
    the block moments' nodes, which log L follows with slope at most 1."""
    prob = gwsynth.make_problem(*grid, psd_scale=1e-47, n_det=n_det)
    prob = with_injection(prob, gwsynth.prior_draws(gwsynth.SEEDS["injection"], 1)[0])
    th = _rows(prob, n)
    t = torch.from_numpy(th).cuda()
    with gw.Context(prob) as ctx:
        if window:
            gw.gw_set_time_window(ctx.handle, window)
        if over:
            gw.gw_set_time_oversample(ctx.handle, over)
        got = {}
        for prec in (0, 1):
            for kind in (0, 1):
                ctx.set_full_kernel(kind)
                got[prec, kind] = ctx.loglike(t, marg=L.PHASE_TIME, prec=prec).cpu().numpy()
        ref = got[0, 1]
        ok = np.isfinite(ref)
        assert all(np.array_equal(np.isfinite(v), ok) for v in got.values())
        tol = _tol(prob, th, ref)
        assert np.max(np.abs(got[0, 0] - ref)[ok]) < 2 * tol
        assert np.max(np.abs(got[1, 0] - ref)[ok]) < 1e-3
        assert np.max(np.abs(got[1, 1] - ref)[ok]) < 1e-3
