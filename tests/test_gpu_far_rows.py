"""GPU: valid rows far from what the prior holds, which the likelihoods take
like any other: phases of millions of cycles, and overlaps that are not
numbers."""
import numpy as np
import pytest

import gwsynth
from oracle import heterodyne as H
from oracle import likelihood as L
from oracle import waveform
from tests.gpu_common import oracle_het_many, with_injection

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

EPS = np.finfo(float).eps


@pytest.fixture(scope="module")
def gw():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    import paper_2607_28265_amd as gw
    return gw


def _problem(grid, n_det=3):
    prob = gwsynth.make_problem(*grid, psd_scale=1e-47, n_det=n_det, n_dist=300)
    th = gwsynth.prior_draws(gwsynth.SEEDS["injection"], 1)[0]
    return with_injection(prob, th), th


def _far(col, values):
    th = np.tile(gwsynth.prior_draws(77, 1), (len(values), 1))
    th[:, col] = values
    return th


# 8.4e6 cycles (2^23) lie at t_c = 8.2e3 s for 1024 Hz and at a chirp mass of
# 0.011 Msun for 20 Hz.
@pytest.mark.parametrize("col,values", [
    (12, [999.93, 8001.01, 8300.07, -8300.07, 20000.03, -100000.01]), (0, [0.02, 0.011, 0.009, 0.005, 0.001])])
def test_het_phases_of_many_cycles(gw, col, values):
    prob, inj = _problem((8.0, 20.0, 1024.0))
    th = _far(col, values)
    het = H.setup(prob, inj, 300)
    cycles = np.array([np.max(np.abs(waveform.phase(t, prob.freqs))) / (2.0 * np.pi) + abs(t[12]) * prob.freqs[-1]
                       for t in th])
    assert cycles.max() > 2.0 ** 24
    # the phase is a sum of terms of about that many cycles, rounded at some ten
    # places in the library and in the oracle; a phase error d changes the overlap
    # by at most d sum_e |W_e| <= d sqrt(n_bins <d|d> <h|h>) and the binned <h|h>
    # by 2 d <h|h>
    dd = L.data_inner(prob)
    hh = np.abs([np.sum(H.overlaps(t, prob, het)[1].real) for t in th])
    room = 2.0 * np.pi * cycles * 16.0 * EPS * (np.sqrt(300.0 * dd * hh) + 2.0 * hh)
    assert np.all(room < 0.05 * np.sqrt(hh))  # far below what another phasor changes
    with gw.Context(prob) as ctx:
        ctx.heterodyne_setup(inj, 300)
        for marg in (L.PLAIN, L.PHASE):
            ref = oracle_het_many(th, prob, het, marg)
            got = ctx.loglike(torch.from_numpy(th).cuda(), gw.GW_HET, marg, 0).cpu().numpy()
            assert np.all(np.abs(got - ref) < 1e-6 + room)


@pytest.mark.parametrize("like", ["full", "het"])
@pytest.mark.parametrize("window,n", [(0.0, 6), (0.1, 6), (0.1, 300)])  # one grid point; both workgroup shapes
def test_time_marginal_of_overlaps_that_are_not_numbers(gw, like, window, n):
    # a distance so small that the overlap or the norm overflows: log L is not a
    # number, as with the phase marginal, and the rows beside it are as ever
    prob, inj = _problem((8.0, 20.0, 512.0))
    th = np.tile(_far(6, [100.0, 1e-320, 200.0, 1e-200, 50.0, 1e-310]), (n // 6, 1))
    bad = np.tile([False, True, False, True, False, True], n // 6)
    with gw.Context(prob) as ctx:
        gw.gw_set_time_window(ctx.handle, window)
        ctx.heterodyne_setup(inj, 300)
        which = gw.GW_FULL if like == "full" else gw.GW_HET
        t = torch.from_numpy(th).cuda()
        good = torch.from_numpy(th[~bad]).cuda()
        for prec in (0, 1):
            assert np.array_equal(np.isnan(ctx.loglike(t, which, L.PHASE, prec).cpu().numpy()), bad)
            got = ctx.loglike(t, which, L.PHASE_TIME, prec).cpu().numpy()
            assert np.array_equal(np.isnan(got), bad)
            want = ctx.loglike(good, which, L.PHASE_TIME, prec).cpu().numpy()
            assert np.max(np.abs(got[~bad] - want)) < 512 * EPS * np.max(np.abs(want))
