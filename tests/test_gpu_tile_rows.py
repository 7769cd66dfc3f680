"""GPU: batches of rows on both sides of the node tables.  Rows are dealt to tiles
by kind, which changes no row's value: a batch in another order gives the same
values in that order, bit for bit."""
import numpy as np
import pytest

import gwsynth
from oracle import likelihood as L
from tests.gpu_common import with_injection

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    import paper_2607_28265_amd as gw
    prob = with_injection(gwsynth.make_problem(8.0, 20.0, 512.0, psd_scale=1e-47, n_dist=100),
                          gwsynth.prior_draws(gwsynth.SEEDS["injection"], 1)[0])
    with gw.Context(prob) as c:
        yield c


def _rows(n, where):
    th = gwsynth.prior_draws(17, n)
    off = {"first": np.arange(n) < 1, "last": np.arange(n) == n - 1, "few": np.arange(n) % 50 == 7,
           "half": np.arange(n) % 2 == 0, "most": np.arange(n) % 40 != 3, "all": np.ones(n, bool),
           "block": (np.arange(n) // 64) % 3 == 1}[where]
    th[off, 0] = 0.9
    th[::77, 1] = 2.0  # not physical
    return th


@pytest.mark.parametrize("where", ["first", "last", "few", "half", "most", "all", "block"])
@pytest.mark.parametrize("n", [1, 63, 64, 65, 130, 1023, 1024, 1025, 2500])
def test_order_of_a_mixed_batch(ctx, n, where):
    th = _rows(n, where)
    perm = np.random.default_rng(n).permutation(n)
    a, b = torch.from_numpy(th).cuda(), torch.from_numpy(th[perm]).cuda()
    at = torch.from_numpy(perm).cuda()
    for marg, prec in ((L.PLAIN, 0), (L.PHASE, 1), (L.PHASE_DIST, 1), (L.PHASE_TIME, 0), (L.PHASE_TIME, 1)):
        want = ctx.loglike(a, marg=marg, prec=prec)
        got = ctx.loglike(b, marg=marg, prec=prec)
        assert not bool(torch.isnan(want).any())
        assert torch.equal(got, want[at])


@pytest.mark.parametrize("prec", [0, 1])
def test_time_marginal_in_several_passes(prec):
    # more rows than one pass of the workspace takes (1 GiB), against a batch small
    # enough for a block's cells to be summed by two waves: the same bits
    import paper_2607_28265_amd as gw
    prob = with_injection(gwsynth.make_problem(32.0, 20.0, 1024.0, psd_scale=1e-47, n_det=2),
                          gwsynth.prior_draws(gwsynth.SEEDS["injection"], 1)[0])
    few = _rows(97, "few")
    few[11, 12], few[13::9, 0] = 0.05, 30.0
    with gw.Context(prob) as c:
        want = c.loglike(torch.from_numpy(few).cuda(), marg=L.PHASE_TIME, prec=prec)
        many = torch.from_numpy(np.tile(few, (207, 1))[:20011]).cuda()
        got = c.loglike(many, marg=L.PHASE_TIME, prec=prec)
    assert torch.equal(got, want.repeat(207)[:20011])
