"""GPU: device tables whose filling fails (forced from the host with
GW_FAULT=tables, after their allocation) are not taken for built ones later."""
import numpy as np
import pytest

import gwsynth
from oracle import likelihood as L
from tests.gpu_common import with_injection

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture()
def setup():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    import paper_2607_28265_amd as gw
    inj = gwsynth.prior_draws(gwsynth.SEEDS["injection"], 1)[0]
    prob = with_injection(gwsynth.make_problem(8.0, 20.0, 512.0, psd_scale=1e-47, n_dist=100), inj)
    with gw.Context(prob) as ctx:
        yield gw, ctx, prob, inj


def test_cache_after_a_failed_table(setup, monkeypatch):
    gw, ctx, prob, _ = setup
    monkeypatch.setenv("GW_FAULT", "tables")
    with pytest.raises(gw.GwError, match="injected"):
        gw.WaveformCache(ctx.handle, 4)
    monkeypatch.delenv("GW_FAULT")
    cache = gw.WaveformCache(ctx.handle, 4)
    th = gwsynth.prior_draws(5, 4)
    slots = torch.arange(4, dtype=torch.int32, device="cuda")
    cache.update(torch.from_numpy(th).cuda(), slots)
    th[:, 12] = [0.19, -0.19, 0.2, 0.01]  # beyond the context's own table, within the wide one
    t = torch.from_numpy(th).cuda()
    got = cache.loglike(t, slots, 1).cpu().numpy()
    want = ctx.loglike(t, marg=L.PHASE_DIST).cpu().numpy()
    cache.close()
    assert np.max(np.abs(got - want)) < 6e-8 * L.data_inner(prob)


@pytest.mark.parametrize("like", ["full", "het"])
def test_time_marginal_after_a_failed_table(setup, monkeypatch, like):
    # tables of one grid, a failed change to another (other edge chunks, or another
    # window), and back
    gw, ctx, prob, inj = setup
    ctx.heterodyne_setup(inj, 200)
    which = gw.GW_FULL if like == "full" else gw.GW_HET
    t = torch.from_numpy(gwsynth.near_posterior(5, inj, 20)).cuda()

    def change(on):
        if like == "full":
            gw.gw_set_time_window(ctx.handle, 0.05 if on else 0.1)
        else:
            gw.gw_set_het_tm_split(ctx.handle, 8 if on else 0)

    want = ctx.loglike(t, which, L.PHASE_TIME).cpu().numpy()
    change(True)
    monkeypatch.setenv("GW_FAULT", "tables")
    with pytest.raises(gw.GwError, match="injected"):
        ctx.loglike(t, which, L.PHASE_TIME)
    monkeypatch.delenv("GW_FAULT")
    change(False)
    assert np.array_equal(ctx.loglike(t, which, L.PHASE_TIME).cpu().numpy(), want)
    change(True)
    assert np.all(np.isfinite(ctx.loglike(t, which, L.PHASE_TIME).cpu().numpy()))
