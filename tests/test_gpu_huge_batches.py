"""GPU: batches whose launches come near the 2^32 threads that one launch takes,
against small batches of the same rows."""
import numpy as np
import pytest

import gwsynth
from tests.gpu_common import with_injection

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# 64 threads a row in the FP64 distance marginal (2^26 rows), 32 in the sums over
# the band in eight chunks (2^27 rows).
@pytest.mark.parametrize("n,marg,prec", [((1 << 26) + 70, 2, 0), ((1 << 27) + 70, 1, 1)])
def test_huge_full_batches(n, marg, prec):
    import paper_2607_28265_amd as gw
    prob = gwsynth.make_problem(1.0, 20.0, 40.0, psd_scale=1e-47, n_det=1, n_dist=16)
    prob = with_injection(prob, gwsynth.prior_draws(gwsynth.SEEDS["injection"], 1)[0])
    few = gwsynth.prior_draws(3, 97)
    few[5, 1] = 2.0        # not physical
    few[1::7, 0] = 0.9     # outside the node tables
    need = n * 8 * (13 + 32 + 16 + 2 + 2)  # theta, coefficients, partial sums, marginal, log L
    if torch.cuda.mem_get_info()[0] < need + (8 << 30):
        pytest.skip("needs %d GiB of device memory" % (need >> 30))
    a = torch.from_numpy(few).cuda()
    b = torch.empty((n, 13), dtype=torch.float64, device="cuda")
    whole = n // 97 * 97
    b[:whole].view(n // 97, 97, 13)[:] = a
    b[whole:] = a[:n - whole]
    with gw.Context(prob) as ctx:
        ref = ctx.loglike(a, marg=marg, prec=prec)
        got = ctx.loglike(b, marg=marg, prec=prec)
        torch.cuda.synchronize()
    want = torch.empty_like(got)
    want[:whole].view(n // 97, 97)[:] = ref
    want[whole:] = ref[:n - whole]
    ok = torch.isfinite(want)
    assert torch.equal(torch.isfinite(got), ok)
    # other chunks of the sums: as for the large batches' test
    assert float((got - want)[ok].abs().max()) < 1e-9
    del a, b, got, want, ok
    torch.cuda.empty_cache()


def test_launch_beyond_the_limit_is_refused():
    import paper_2607_28265_amd as gw
    prob = gwsynth.make_problem(1.0, 20.0, 40.0, psd_scale=1e-47, n_det=1, n_dist=16)
    th = torch.from_numpy(gwsynth.prior_draws(3, 1)).cuda()
    with gw.Context(prob) as ctx:
        ctx.set_full_shape(64, 1 << 26)  # 2^32 threads for one row
        with pytest.raises(gw.GwError, match="too large"):
            ctx.loglike(th, marg=1)
        ctx.set_full_shape(0, 0)
        assert np.isfinite(ctx.loglike(th, marg=1).cpu().numpy()[0])
