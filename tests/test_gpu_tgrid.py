"""GPU: the time marginal's frequency grid and transform at the edges of its
forms, against the oracle's direct sum over time shifts: every first radix and
count of nonzero inputs, grid points folded onto the transform, both workgroup
shapes, rows over nodes and over bins, one and several passes of norm moments."""
import math

import numpy as np
import pytest

import gwsynth
from oracle import heterodyne as H
from oracle import likelihood as L
from tests.gpu_common import oracle_het_many, oracle_many, with_injection

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def gw():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    import paper_2607_28265_amd as gw
    return gw


def _tol(prob, th, ref):
    """The window's images (6e-13) and the nodes' interpolation (1e-13) of
    sum |y| <= sqrt(N_f <d|d> <h|h>), which log L follows with slope at most 1,
    rounding of the sums, and the repository's 1e-6 against the oracle."""
    ok = np.isfinite(ref)
    hh = max(L.overlap(t, prob)[1] for t in th[ok][:16])
    return (7e-13 * math.sqrt(prob.n_freq * L.data_inner(prob) * hh)
            + 512 * np.finfo(float).eps * np.max(np.abs(ref[ok])) + 1e-6)


def _problem(grid, n_det=3):
    prob = gwsynth.make_problem(*grid, psd_scale=1e-47, n_det=n_det)
    th = gwsynth.prior_draws(gwsynth.SEEDS["injection"], 1)[0]
    return with_injection(prob, th), th


@pytest.mark.parametrize("grid,n_det,window,over,fft", [
    ((8.0, 20.0, 512.0), 3, 0.0, 1, 16),      # one point, L = 16
    ((8.0, 20.0, 512.0), 2, 0.01, 2, 64),     # second radix 4
    ((8.0, 20.0, 512.0), 1, 0.03, 4, 256),    # second radix 16
    ((8.0, 20.0, 512.0), 3, 0.1, 1, 256),     # points beyond L: folded
    ((8.0, 20.0, 512.0), 3, 0.03, 8, 512),    # first radix 2
    ((8.0, 20.0, 512.0), 4, 0.1, 4, 1024),    # first radix 4
    ((8.0, 20.0, 512.0), 3, 0.1, 8, 2048),    # first radix 8
    ((8.0, 20.0, 512.0), 2, 0.1, 16, 4096),   # first radix 16, 2 inputs
    ((8.0, 20.0, 512.0), 3, 0.4, 4, 4096),    # 4 inputs
    ((8.0, 20.0, 512.0), 1, 0.9, 2, 4096),    # 8 inputs
    ((8.0, 2.0, 512.0), 2, 0.9, 2, 4096),     # 16 inputs, cells of two bins
    ((0.25, 20.0, 400.0), 3, 0.1, 4, 1024),   # cells of half a bin
])
def test_time_grid_against_oracle(gw, monkeypatch, grid, n_det, window, over, fft):
    prob, inj = _problem(grid, n_det)
    th = np.concatenate([gwsynth.prior_draws(3, 8), gwsynth.near_posterior(5, inj, 8)])
    th[3, 0], th[11, 0] = 30.0, 0.9  # beyond the node tables
    monkeypatch.setattr(L, "TIME_WINDOW", window)
    monkeypatch.setattr(L, "TIME_OVERSAMPLE", over)
    ref = oracle_many(th, prob, L.PHASE_TIME)
    t = torch.from_numpy(th).cuda()
    with gw.Context(prob) as ctx:
        gw.gw_set_time_oversample(ctx.handle, over)
        gw.gw_set_time_window(ctx.handle, window)
        _, n_t, p, _ = gw.gw_time_grid_info(ctx.handle)
        assert n_t == L.time_grid(prob).size and p * over == fft
        tol = _tol(prob, th, ref)
        for kind in (0, 1):
            ctx.set_full_kernel(kind)
            got = ctx.loglike(t, marg=L.PHASE_TIME).cpu().numpy()
            assert np.max(np.abs(got - ref)) < tol
            mix = ctx.loglike(t, marg=L.PHASE_TIME, prec=1).cpu().numpy()
            assert np.max(np.abs(mix - ref)) < 1e-3
        # a row's value does not depend on the launch: 256 lanes a row or 512
        ctx.set_full_kernel(0)
        one = ctx.loglike(t, marg=L.PHASE_TIME).cpu().numpy()
        many = ctx.loglike(t.repeat(20, 1), marg=L.PHASE_TIME).cpu().numpy()
        assert np.array_equal(many, np.tile(one, 20))


@pytest.mark.parametrize("n_bins,window,over,n", [
    (20, 0.1, 4, 16), (60, 0.1, 2, 257), (400, 0.1, 4, 65), (400, 0.0, 1, 1)])
def test_het_time_grid_against_oracle(gw, monkeypatch, n_bins, window, over, n):
    # few bins: wide ones, so several passes of norm moments
    prob, inj = _problem((8.0, 20.0, 512.0))
    th = np.concatenate([gwsynth.near_posterior(5, inj, 12), gwsynth.prior_draws(3, 4)])
    th = np.tile(th, (17, 1))[:n]
    monkeypatch.setattr(L, "TIME_WINDOW", window)
    monkeypatch.setattr(L, "TIME_OVERSAMPLE", over)
    t = torch.from_numpy(th).cuda()
    with gw.Context(prob) as ctx:
        gw.gw_set_time_oversample(ctx.handle, over)
        gw.gw_set_time_window(ctx.handle, window)
        ctx.heterodyne_setup(inj, n_bins)
        try:
            got = ctx.loglike(t, gw.GW_HET, L.PHASE_TIME).cpu().numpy()
        except gw.GwError:
            assert n_bins == 20  # bins too wide for the norm series
            return
        ref = oracle_het_many(th[:16], prob, H.setup(prob, inj, n_bins), L.PHASE_TIME)
        tol = _tol(prob, th[:16], ref)
        assert np.max(np.abs(got[:16] - ref)) < tol
        for s in (1, 8, 256):  # any number of edge chunks
            gw.gw_set_het_tm_split(ctx.handle, s)
            again = ctx.loglike(t, gw.GW_HET, L.PHASE_TIME).cpu().numpy()
            assert np.max(np.abs(again - got)) < tol
