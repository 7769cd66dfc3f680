"""GPU: the look-ahead rounds of the slice sampler make the moves of the
one-candidate walk, whatever number of candidates a chain proposes at once."""
import numpy as np
import pytest

from oracle import sampler as S
from tests.gpu_common import problem
from tests.test_gpu_slice_prescreen import to_unit

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def gw():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    import paper_2607_28265_amd as gw
    return gw


def sweep(gw, ctx, x, logl, lstar, blocks, chols, like, max_out, max_shrink, use_graph=True, record=False):
    k = len(x)
    xt, lt = torch.from_numpy(x.copy()).cuda(), torch.from_numpy(logl.copy()).cuda()
    ne = torch.zeros(k, dtype=torch.int32, device="cuda")
    st = torch.zeros(k, dtype=torch.int32, device="cuda")
    rec = None
    if record:  # recorded calls run the one-candidate rounds
        rec = (torch.empty((1 << 16, 11), dtype=torch.float64, device="cuda"),
               torch.empty(1 << 16, dtype=torch.float64, device="cuda"),
               torch.zeros(1, dtype=torch.int64, device="cuda"))
    gw.slice_sweep(ctx.handle, xt, lt, lstar, blocks, chols, seed=8, counter=5, max_out=max_out, max_shrink=max_shrink,
                   like=like, prec=gw.GW_PREC_FP64, n_evals=ne, status=st, use_graph=use_graph, record=rec)
    return [t.cpu().numpy() for t in (xt, lt, ne, st)], int(rec[2].item()) if record else None


# 600, 200, 100 and 40 chains propose 2, 4, 8 and 16 candidates each; budgets of
# no and few steps out, and shrink caps below and above the candidates of a
# round; points near the cube's walls, so that draws fall outside it
@pytest.mark.parametrize("like", ["full", "het"])
@pytest.mark.parametrize("max_out,max_shrink", [(0, 1), (1, 3), (10, 100), (3, 17)])
@pytest.mark.parametrize("blocks", [tuple(S.BLOCKS), (tuple(range(11)), (9,))])
def test_moves_do_not_depend_on_the_candidates_per_round(gw, like, max_out, max_shrink, blocks):
    prob = problem("cfg1", loud=True)
    rng = np.random.default_rng(2)
    x = np.clip(to_unit(prob.theta_inj) + 0.02 * rng.standard_normal((600, 11)), 1e-6, 1.0 - 1e-6)
    x[::4, 2] = rng.uniform(0.0, 0.02, 150)
    x[1::4, 10] = rng.uniform(0.98, 1.0, 150)
    kind = gw.GW_FULL if like == "full" else gw.GW_HET
    with gw.Context(prob) as ctx:
        if like == "het":
            ctx.heterodyne_setup(prob.theta_inj, 200)
        logl = ctx.loglike(gw.gw_prior_transform(ctx.handle, torch.from_numpy(x).cuda()), kind,
                           gw.GW_MARG_PHASE_DIST).cpu().numpy()
        lstar = float(np.quantile(logl, 0.3))
        chols = [3.0 * S.block_cholesky(x, b) for b in blocks]
        args = (lstar, blocks, chols, kind, max_out, max_shrink)
        want, _ = sweep(gw, ctx, x, logl, *args)
        walk, n_rec = sweep(gw, ctx, x, logl, *args, record=True)
        assert n_rec == int(walk[2].sum())
        # the log L of one row may differ in its last places between launch
        # shapes (summation order); every decision and point must not
        tol = 64 * np.finfo(float).eps * np.max(np.abs(logl))
        for got, k in [(walk, 600)] + [(sweep(gw, ctx, x[:k], logl[:k], *args, use_graph=g)[0], k)
                                       for k, g in ((200, True), (100, False), (40, True))]:
            assert np.array_equal(got[0], want[0][:k])
            assert np.max(np.abs(got[1] - want[1][:k])) <= tol
            assert np.array_equal(got[2], want[2][:k]) and np.array_equal(got[3], want[3][:k])
    assert want[2].min() >= 0 and np.any(want[0] != x)
