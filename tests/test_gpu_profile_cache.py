"""GPU: the kernel timer of the waveform cache's fast rows covers their sums."""
import numpy as np
import pytest

import gwsynth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("mc", [1.2, 0.9])  # slots of nodes, slots of moments
def test_fast_rows_timer(mc):
    import paper_2607_28265_amd as gw
    n = 8192
    prob = gwsynth.make_problem(32.0, 20.0, 1024.0, psd_scale=1e-47, n_dist=100)
    th = gwsynth.prior_draws(5, n)
    th[:, 0] = mc
    t = torch.from_numpy(th).cuda()
    with gw.Context(prob) as ctx:
        cache = gw.WaveformCache(ctx.handle, 64)
        cache.update(t[:64].contiguous(), torch.arange(64, dtype=torch.int32, device="cuda"), prec=1)
        slots = torch.from_numpy((np.arange(n) % 64).astype(np.int32)).cuda()

        def kernel(f):
            for _ in range(3):
                f()
            torch.cuda.synchronize()
            gw.gw_profile_read(ctx.handle)
            gw.gw_profile_enable(ctx.handle, 1)
            for _ in range(10):
                f()
            ms, launches = gw.gw_profile_read(ctx.handle)
            gw.gw_profile_enable(ctx.handle, 0)
            assert launches == 10
            return ms / launches

        def whole(f):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            a.record()
            for _ in range(10):
                f()
            b.record()
            torch.cuda.synchronize()
            return a.elapsed_time(b) / 10

        fast = lambda: cache.loglike(t, slots, 1, marg=1, prec=1)
        cached = lambda: cache.loglike(t, slots, 2, marg=1, prec=1)
        # kind 2 is kind 1 without the sums: what is left of kind 1 is the timer's
        sums = whole(fast) - whole(cached)
        assert kernel(fast) > 0.4 * sums
        cache.close()
