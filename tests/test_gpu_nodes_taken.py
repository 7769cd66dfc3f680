"""GPU: which rows are summed over the interpolation nodes, and which norm series
the heterodyned time marginal takes or refuses."""
import numpy as np
import pytest

import gwsynth
from oracle import heterodyne as H
from oracle import likelihood as L
from tests.gpu_common import oracle_het_many, with_injection
from tests.test_gpu_nodes import _rows
from tests.test_gpu_tgrid import _tol

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def gw():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    import paper_2607_28265_amd as gw
    return gw


def _problem():
    prob = gwsynth.make_problem(8.0, 20.0, 512.0, psd_scale=1e-47)
    th = gwsynth.prior_draws(gwsynth.SEEDS["injection"], 1)[0]
    return with_injection(prob, th), th


def test_covered_rows_take_the_nodes(gw):
    # mixed, in eight chunks either way: a row within the tables is a sum of other
    # samples than the bins', so most have other last digits; a row beyond them
    # takes the same sums over the bins, bit for bit
    prob, _ = _problem()
    th = gwsynth.prior_draws(11, 200)
    inside = np.arange(200) % 3 != 0
    th[0::6, 0], th[3::6, 12] = 0.9, 0.2
    t = torch.from_numpy(th).cuda()
    with gw.Context(prob) as ctx:
        nodes, _ = gw.gw_full_nodes(ctx.handle)
        assert nodes < prob.n_freq // 2
        ctx.set_full_shape(0, 8)
        got = {}
        for kind in (0, 1):
            ctx.set_full_kernel(kind)
            got[kind] = ctx.loglike(t, marg=L.PHASE, prec=1).cpu().numpy()
    same = got[0] == got[1]
    assert np.all(same[~inside]) and np.mean(same[inside]) < 0.2


def test_rows_of_the_nodes_test_are_mixed(gw):
    # the rows that the other node tests use are of both kinds
    prob, _ = _problem()
    t = torch.from_numpy(_rows(prob, 250)).cuda()
    with gw.Context(prob) as ctx:
        ctx.set_full_shape(0, 8)
        a = ctx.loglike(t, marg=L.PHASE, prec=1)
        ctx.set_full_kernel(1)
        same = (a == ctx.loglike(t, marg=L.PHASE, prec=1)).cpu().numpy()
    assert 3 <= np.sum(same) <= 60


def test_bins_too_wide_for_the_norm_series_are_refused(gw):
    prob, inj = _problem()
    t = torch.from_numpy(gwsynth.near_posterior(5, inj, 16)).cuda()
    with gw.Context(prob) as ctx:
        ctx.heterodyne_setup(inj, 20)
        with pytest.raises(gw.GwError, match="norm terms"):
            ctx.loglike(t, gw.GW_HET, L.PHASE_TIME)
        assert np.all(np.isfinite(ctx.loglike(t, gw.GW_HET, L.PHASE).cpu().numpy()))


@pytest.mark.parametrize("n_bins", [30, 80])  # 48 and 27 norm terms: four passes, two
def test_norm_series_of_several_passes(gw, n_bins):
    prob, inj = _problem()
    th = np.concatenate([gwsynth.near_posterior(5, inj, 12), gwsynth.prior_draws(3, 4)])
    with gw.Context(prob) as ctx:
        ctx.heterodyne_setup(inj, n_bins)
        got = ctx.loglike(torch.from_numpy(th).cuda(), gw.GW_HET, L.PHASE_TIME).cpu().numpy()
    ref = oracle_het_many(th, prob, H.setup(prob, inj, n_bins), L.PHASE_TIME)
    assert np.max(np.abs(got - ref)) < _tol(prob, th, ref)
