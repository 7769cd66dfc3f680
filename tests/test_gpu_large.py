"""GPU: large heterodyned and full-band batches (their own reduction, distance
marginal and FP64 phasor forms) against small batches of the same rows."""
import numpy as np
import pytest

import gwsynth
from tests.gpu_common import with_injection

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _rows(th, n):
    rows = np.concatenate([gwsynth.prior_draws(3, 60), gwsynth.near_posterior(5, th, 37)])
    rows[5, 1] = 2.0   # not physical
    return rows, np.tile(rows, (n // 97 + 1, 1))[:n]


# The large batch sums in other chunks than the small one: of an overlap sum of
# size s = 1e4 over 1e3 terms, 1e3 eps s = 1e-9 at most.  Mixed, distance
# marginal: 1000 FP32 terms in another order, 1000 eps_32 / 2 = 6e-5.
@pytest.mark.parametrize("n_det,n,n_bins", [(1, 8192, 300), (2, 8193, 40), (3, 12001, 500), (4, 8200, 64)])
def test_large_het_batches(n_det, n, n_bins):
    import paper_2607_28265_amd as gw
    prob = gwsynth.make_problem(8.0, 20.0, 512.0, psd_scale=1e-47, n_det=n_det, n_dist=1000)
    th = gwsynth.prior_draws(gwsynth.SEEDS["injection"], 1)[0]
    prob = with_injection(prob, th)
    few, many = _rows(th, n)
    with gw.Context(prob) as ctx:
        ctx.heterodyne_setup(th, n_bins)
        a, b = torch.from_numpy(few).cuda(), torch.from_numpy(many).cuda()
        off = gwsynth.uneven_split(1, n, 500, 900)
        subs = torch.from_numpy(np.stack([off[:-1], np.diff(off)], axis=1)).cuda()
        for marg in (0, 1, 2):
            for prec, tol in ((0, 1e-9), (1, 1e-4 if marg == 2 else 1e-9)):
                small = ctx.loglike(a, gw.GW_HET, marg, prec).cpu().numpy()
                ref = np.tile(small, n // 97 + 1)[:n]
                ok = np.isfinite(ref)
                for got in (ctx.loglike(b, gw.GW_HET, marg, prec), ctx.loglike_uneven(b, subs, marg, prec)):
                    got = got.cpu().numpy()
                    assert np.array_equal(np.isfinite(got), ok)
                    assert np.max(np.abs(got - ref)[ok]) < tol
        # one edge chunk, and more than the combine's unrolled eight
        for ech in (1, 9):
            ctx.set_het_shape(4, 0, ech)
            got = ctx.loglike(b, gw.GW_HET, 1, 0).cpu().numpy()
            ref = np.tile(ctx.loglike(a, gw.GW_HET, 1, 0).cpu().numpy(), n // 97 + 1)[:n]
            assert np.max(np.abs(got - ref)[ok]) < 1e-9


@pytest.mark.parametrize("prec,tol", [(0, 1e-9), (1, 1e-4)])
def test_large_full_batches_distance(prec, tol):
    import paper_2607_28265_amd as gw
    prob = gwsynth.make_problem(8.0, 20.0, 512.0, psd_scale=1e-47, n_dist=1000)
    th = gwsynth.prior_draws(gwsynth.SEEDS["injection"], 1)[0]
    prob = with_injection(prob, th)
    few, many = _rows(th, 8200)
    with gw.Context(prob) as ctx:
        ref = ctx.loglike(torch.from_numpy(few).cuda(), marg=2, prec=prec).cpu().numpy()
        got = ctx.loglike(torch.from_numpy(many).cuda(), marg=2, prec=prec).cpu().numpy()
        ref = np.tile(ref, 85)[:8200]
        ok = np.isfinite(ref)
        assert np.array_equal(np.isfinite(got), ok)
        assert np.max(np.abs(got - ref)[ok]) < tol


@pytest.mark.parametrize("n", [1, 3, 4, 5, 63, 66])
def test_small_full_batches_distance(n):
    """Four rows a workgroup: ragged ends, rows over nodes and over bins."""
    import paper_2607_28265_amd as gw
    prob = gwsynth.make_problem(8.0, 20.0, 512.0, psd_scale=1e-47, n_det=2, n_dist=300)
    th = gwsynth.prior_draws(gwsynth.SEEDS["injection"], 1)[0]
    prob = with_injection(prob, th)
    few, _ = _rows(th, 97)
    few[1::7, 0] = 0.9  # outside the node tables
    with gw.Context(prob) as ctx:
        t = torch.from_numpy(few).cuda()
        for prec, tol in ((0, 1e-9), (1, 1e-4)):
            ref = ctx.loglike(t, marg=2, prec=prec).cpu().numpy()
            got = ctx.loglike(t[:n].contiguous(), marg=2, prec=prec).cpu().numpy()
            ok = np.isfinite(ref[:n])
            assert np.array_equal(np.isfinite(got), ok)
            assert np.max(np.abs(got - ref[:n])[ok]) < tol


@pytest.mark.parametrize("psd_scale", [1e-43, 1e-45, 1e-46, 1e-47, 1e-48, 1e-49])
def test_fp64_distance_series_lengths(psd_scale):
    """From x = |Z1| / d far below 1 to hundreds: every length of the two I0
    series, against the oracle (the FP64 form's 1e-6)."""
    import paper_2607_28265_amd as gw
    from oracle import likelihood as L
    from tests.gpu_common import oracle_many
    prob = gwsynth.make_problem(4.0, 20.0, 256.0, psd_scale=psd_scale, n_dist=200)
    th = gwsynth.prior_draws(gwsynth.SEEDS["injection"], 1)[0]
    prob = with_injection(prob, th)
    few, _ = _rows(th, 97)
    ref = oracle_many(few, prob, L.PHASE_DIST)
    ok = np.isfinite(ref)
    with gw.Context(prob) as ctx:
        got = ctx.loglike(torch.from_numpy(few).cuda(), marg=2, prec=0).cpu().numpy()
        assert np.array_equal(np.isfinite(got), ok)
        assert np.max(np.abs(got - ref)[ok]) < 1e-6
