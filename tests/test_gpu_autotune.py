"""GPU: the autotuner's candidates hold the automatic launch shape."""
import pytest

import gwsynth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_automatic_shape_is_a_candidate():
    # a band too narrow for any explicit number of chunks leaves it alone
    import paper_2607_28265_amd as gw
    prob = gwsynth.make_problem(1.0, 20.0, 100.0, psd_scale=1e-47, n_dist=16)
    t = torch.from_numpy(gwsynth.prior_draws(3, 70)).cuda()
    with gw.Context(prob) as ctx:
        assert prob.n_freq < 8 * 16
        want = ctx.loglike(t, marg=1)
        shape, ms = gw._lib.gw_autotune(ctx.handle, t, gw.GW_FULL, 1, 0, 1)
        assert shape == (0, 0, 0) and 0.0 < ms < 1e3
        assert torch.equal(ctx.loglike(t, marg=1), want)

