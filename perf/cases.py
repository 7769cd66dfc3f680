"""Performance cases of the batched likelihood library.

Each case is one call (or the few calls that belong together) that a program
using the library makes: batches of log-likelihoods on the full band and on
heterodyned bins, with each marginalisation and precision, one Gibbs sweep of
the slice sampler, the waveform cache's slow and fast calls, and the
prescreen network's prediction and gradient.  Sizes are the benchmark's and
the tests' (8 s up to 512 Hz; 128 s up to 2048 Hz; 500 and 5000 bins; 125
chains, whose rounds evaluate up to 250 rows; batches up to 65,536).  The
signal sits at network SNR 24, and a batch is half prior draws and half
proposals near the posterior, as a nested-sampling run meets them.
"""
import dataclasses
import math

import numpy as np
import torch

import gwsynth
import paper_2607_28265_amd as gw
from gwsynth.workload import PRIOR as P

DEV = "cuda:0"
MARG = {"none": gw.GW_MARG_NONE, "phase": gw.GW_MARG_PHASE, "dist": gw.GW_MARG_PHASE_DIST,
        "time": gw.GW_MARG_PHASE_TIME}
PREC = {"fp64": gw.GW_PREC_FP64, "mixed": gw.GW_PREC_MIXED}
BLOCKS = ((0, 1, 4, 5), (2,), (3,), (6,), (7, 8), (9,), (10,))
WINDOW = 0.1     # s, half-width of the coalescence-time prior
OVERSAMPLE = 4   # time-grid points per sampling interval
N_DIST = 1000
SNR = 24.0


# -- the cases ----------------------------------------------------------------

def _batch(name, like, marg, prec, rows, duration=128.0, f_max=2048.0, n_bins=0, uneven=False, n_det=3):
    return {"name": name, "kind": "batch", "like": like, "marg": marg, "prec": prec, "rows": rows,
            "duration": duration, "f_max": f_max, "n_bins": n_bins, "uneven": uneven, "n_det": n_det}


def listed():
    return [
        # one round of the heterodyned sampler: two bracket ends of 125 chains
        _batch("het_round_250", "het", "dist", "mixed", 250, n_bins=500),
        # the same round on the full band
        _batch("full_round_250", "full", "dist", "mixed", 250),
        # the throughput batch of the benchmark: a live set's worth of proposals, exact likelihood
        _batch("full_batch_4096", "full", "dist", "mixed", 4096),
        # a short segment in plain FP64, nothing marginalised: parity runs, re-weighting of stored samples
        _batch("full_plain_8s_1024", "full", "none", "fp64", 1024, duration=8.0, f_max=512.0),
        # the reference precision on the long segment, an odd batch: confirming the posterior samples of a run
        _batch("full_phase_fp64_1531", "full", "phase", "fp64", 1531),
        # a large heterodyned batch in uneven sub-batches, one replayed launch sequence
        _batch("het_uneven_65536", "het", "dist", "mixed", 65536, n_bins=500, uneven=True),
        # the same call at the paper's bin count in FP64, a ragged total
        _batch("het_fp64_5000_20011", "het", "dist", "fp64", 20011, n_bins=5000, uneven=True),
        # coalescence time marginalised on the full band: a live set of the event analysis
        _batch("time_full_1000", "full", "time", "mixed", 1000),
        # one round of the heterodyned event analysis (64 chains) with the time marginal
        _batch("time_het_round_128", "het", "time", "mixed", 128, n_bins=5000),
        # one Gibbs sweep of 125 chains: the call a nested-sampling iteration consists of
        {"name": "sweep_het_125", "kind": "sweep", "like": "het", "prec": "mixed", "chains": 125, "live": 1000,
         "n_bins": 500, "duration": 128.0, "f_max": 2048.0},
        # fast/slow likelihood pair: cache the waveforms of a live set, then extrinsic proposals on them
        {"name": "cache_512_2048", "kind": "cache", "prec": "mixed", "slots": 512, "rows": 2048, "duration": 128.0,
         "f_max": 2048.0},
        # learned prescreen: predict a batch of candidates, gradient of one training batch
        {"name": "network_16384", "kind": "network", "rows": 16384, "batch": 1024},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["full", "full", "full", "het", "het", "het", "time_full", "time_het", "sweep", "cache",
                       "network"])
    duration, f_max = rng.choice([(8.0, 512.0), (32.0, 1024.0), (64.0, 2048.0), (128.0, 2048.0), (128.0, 2048.0)])
    prec = rng.choice(["fp64", "mixed", "mixed"])
    n_det = rng.choice([2, 3, 3])
    if kind == "full":
        c = _batch("", "full", rng.choice(["none", "phase", "dist", "dist"]), prec,
                   _log_int(rng, 30, 2000 if prec == "fp64" else 4096), duration, f_max, n_det=n_det)
    elif kind == "het":
        n_bins = _log_int(rng, 200, 5000)
        c = _batch("", "het", rng.choice(["phase", "dist", "dist"]), prec,
                   _log_int(rng, 100, 65536 if n_bins <= 600 else 16000), 128.0, 2048.0, n_bins,
                   rng.random() < 0.5, n_det)
    elif kind == "time_full":
        c = _batch("", "full", "time", prec, _log_int(rng, 50, 1000), duration, f_max, n_det=n_det)
    elif kind == "time_het":
        c = _batch("", "het", "time", prec, _log_int(rng, 50, 4000), 128.0, 2048.0, _log_int(rng, 300, 5000),
                   n_det=n_det)
    elif kind == "sweep":
        c = {"kind": "sweep", "like": rng.choice(["het", "het", "full"]), "prec": "mixed",
             "chains": _log_int(rng, 25, 250), "live": 1000, "n_bins": _log_int(rng, 300, 5000), "duration": 128.0,
             "f_max": 2048.0}
    elif kind == "cache":
        c = {"kind": "cache", "prec": prec, "slots": _log_int(rng, 30, 600), "rows": _log_int(rng, 100, 4096),
             "duration": duration, "f_max": f_max}
    else:
        c = {"kind": "network", "rows": _log_int(rng, 250, 65536), "batch": _log_int(rng, 256, 2048)}
    c.pop("name", None)
    return c


# -- inputs -------------------------------------------------------------------

def _problem(case, seed):
    """Strain data with a signal at network SNR 24 in Gaussian noise, and the
    signal's parameters."""
    rng = np.random.default_rng([seed, 1])
    prob = gwsynth.make_problem(case["duration"], 20.0, case["f_max"], psd_scale=1e-49, noise_seed=None,
                                n_det=case.get("n_det", 3), n_dist=N_DIST)
    theta = gwsynth.prior_draws(seed, 1)[0]
    theta[12] *= 0.5
    h = _strain(torch.from_numpy(theta[None]).to(DEV), prob)[0].cpu().numpy()
    rho = math.sqrt(float(np.sum(4.0 * prob.df * np.abs(h) ** 2 / prob.psd)))
    theta[6] *= rho / SNR
    sig = np.sqrt(prob.psd / (4.0 * prob.df))
    noise = sig * rng.standard_normal(prob.psd.shape) + 1j * sig * rng.standard_normal(prob.psd.shape)
    return dataclasses.replace(prob, data=h * (SNR / rho) + noise), theta


def _rows(theta, seed, n):
    near = gwsynth.near_posterior(seed + 2, theta, n - n // 2)
    return np.concatenate([gwsynth.prior_draws(seed + 1, n // 2), near])[np.random.default_rng([seed, 3]).permutation(n)]


def _to_cube(theta):
    """Parameter vectors [n, 13] to the sampler's unit cube [n, 11]."""
    lin = lambda v, r: (v - r[0]) / (r[1] - r[0])  # noqa: E731
    u = np.stack([lin(theta[:, 0], P["mc"]), lin(theta[:, 1], P["q"]), lin(theta[:, 2], P["chi"]),
                  lin(theta[:, 3], P["chi"]), lin(theta[:, 4], P["lam"]), lin(theta[:, 5], P["lam"]),
                  0.5 * (1.0 - np.cos(theta[:, 7])), theta[:, 8] / (2.0 * np.pi), 0.5 * (1.0 + np.sin(theta[:, 9])),
                  theta[:, 10] / np.pi, lin(theta[:, 12], P["tc"])], axis=1)
    return np.clip(u, 1e-9, 1.0 - 1e-9)


def _network(seed):
    rng = np.random.default_rng([seed, 5])
    sizes = (11, 256, 256, 256, 1)
    return [(rng.normal(0.0, math.sqrt(2.0 / a), (a, b)).astype(np.float32), rng.normal(0.0, 0.1, b).astype(np.float32))
            for a, b in zip(sizes[:-1], sizes[1:])]


def _network_io(case, seed):
    rng = np.random.default_rng([seed, 6])
    x = rng.uniform(size=(case["rows"], 11))
    xb = rng.uniform(size=(case["batch"], 11))
    lb = -1e4 - 400.0 * np.sum((xb - 0.5) ** 2, axis=1) + rng.normal(0.0, 5.0, case["batch"])
    return x, xb, lb, (np.full(11, 0.5), np.full(11, 0.29), -1.035e4, 100.0)


def _uneven(seed, n):
    off = gwsynth.uneven_split(seed, n)
    return np.stack([off[:-1], np.diff(off)], axis=1)


def _cache_rows(case, theta, seed):
    """The cached points and, per proposal row, its slot and extrinsic move."""
    rng = np.random.default_rng([seed, 4])
    base = _rows(theta, seed, case["slots"])
    slots = rng.integers(0, case["slots"], case["rows"]).astype(np.int32)
    fast = base[slots].copy()
    ext = gwsynth.prior_draws(seed + 9, case["rows"])
    fast[:, 6:11] = ext[:, 6:11]
    fast[:, 12] = ext[:, 12]
    return base, slots, fast


def prepare(case, seed):
    kind = case["kind"]
    if kind == "network":
        x, xb, lb, scale = _network_io(case, seed)
        prob = gwsynth.make_problem(4.0, 20.0, 256.0)
        ctx = gw.Context(prob)
        net = gw.Mlp(ctx)
        net.set_params(np.concatenate([np.concatenate([w.ravel(), b]) for w, b in _network(seed)]))
        net.set_scaling(*scale)
        t = lambda a: torch.from_numpy(a).to(DEV)  # noqa: E731
        return {"kind": kind, "ctx": ctx, "net": net, "x": t(x), "xb": t(xb), "lb": t(lb)}
    prob, theta = _problem(case, seed)
    ctx = gw.Context(prob)
    state = {"kind": kind, "ctx": ctx}
    if kind == "batch":
        if case["like"] == "het":
            ctx.heterodyne_setup(theta, case["n_bins"])
        state.update(theta=torch.from_numpy(_rows(theta, seed, case["rows"])).to(DEV), marg=MARG[case["marg"]],
                     prec=PREC[case["prec"]], like=gw.GW_HET if case["like"] == "het" else gw.GW_FULL)
        if case["uneven"]:
            state["subs"] = torch.from_numpy(_uneven(seed, case["rows"])).to(DEV)
    elif kind == "cache":
        base, slots, fast = _cache_rows(case, theta, seed)
        n = case["slots"]
        # the cache goes first in the state: it has to be released before its context
        state = {"cache": gw.WaveformCache(ctx.handle, n), **state}
        state.update(prec=PREC[case["prec"]], base=torch.from_numpy(base).to(DEV),
                     base_slots=torch.arange(n, dtype=torch.int32, device=DEV),
                     fast=torch.from_numpy(fast).to(DEV), slots=torch.from_numpy(slots).to(DEV))
    else:  # sweep: a live set around the signal, the lowest points deleted, chains start from survivors
        if case["like"] == "het":
            ctx.heterodyne_setup(theta, case["n_bins"])
        like = gw.GW_HET if case["like"] == "het" else gw.GW_FULL
        x = _to_cube(gwsynth.near_posterior(seed + 2, theta, case["live"], 1.5))
        xt = torch.from_numpy(x).to(DEV)
        logl = ctx.loglike(gw.gw_prior_transform(ctx.handle, xt), like, gw.GW_MARG_PHASE_DIST, PREC[case["prec"]])
        order = torch.argsort(logl).cpu().numpy()
        rng = np.random.default_rng([seed, 7])
        start = torch.from_numpy(rng.choice(order[case["chains"]:], case["chains"])).to(DEV)
        chols = [np.linalg.cholesky(np.atleast_2d(np.cov(x[:, b], rowvar=False))) for b in BLOCKS]
        state.update(live=xt, logl=logl, start=start, star=float(logl[order[case["chains"] - 1]]), chols=chols,
                     like=like, prec=PREC[case["prec"]], seed=seed)
    return state


# -- one pass -----------------------------------------------------------------

def run(state):
    ctx, kind = state["ctx"], state["kind"]
    if kind == "batch":
        if "subs" in state:
            return ctx.loglike_uneven(state["theta"], state["subs"], state["marg"], state["prec"])
        return ctx.loglike(state["theta"], state["like"], state["marg"], state["prec"])
    if kind == "cache":
        slow = state["cache"].update(state["base"], state["base_slots"], prec=state["prec"])
        return slow, state["cache"].loglike(state["fast"], state["slots"], 1, prec=state["prec"])
    if kind == "network":
        pred = state["net"].forward(state["x"])
        grads, loss = state["net"].grad(state["xb"], state["lb"])
        return pred, grads, loss
    x, logl = state["live"][state["start"]], state["logl"][state["start"]]
    n_evals = torch.zeros(x.shape[0], dtype=torch.int32, device=x.device)
    status = torch.zeros_like(n_evals)
    gw.slice_sweep(ctx.handle, x, logl, state["star"], BLOCKS, state["chols"], seed=state["seed"], like=state["like"],
                   prec=state["prec"], n_evals=n_evals, status=status)
    return x, logl, n_evals, status


# -- the least a pass has to do -----------------------------------------------

def _grid(case):
    return gwsynth.freq_grid(case["duration"], 20.0, case["f_max"])


def _samples(g):
    """Fewest samples of the template over the band: two per cycle of its
    phase (chirp mass 1.25, shifted by the time prior), at most one per bin."""
    f = g.freqs
    t = 5.0 / 256.0 * math.pi ** (-8.0 / 3.0) * (1.25 * 4.925490947641267e-6) ** (-5.0 / 3.0) * f ** (-8.0 / 3.0)
    return float(np.sum(np.minimum(1.0, 2.0 * (t + WINDOW) * g.df)))


def _time_points(g):
    n = 1
    while n < 2 * (g.k0 + g.n_freq - 1):
        n *= 2
    return n, 2 * OVERSAMPLE * int(math.floor(WINDOW * n * g.df + 1e-9)) + 1


def work(case):
    kind = case["kind"]
    if kind == "network":
        mac = 11 * 256 + 2 * 256 * 256 + 256
        return {"bytes": case["rows"] * 96 + case["batch"] * 96 + 134913 * 8,
                "flops": 2 * mac * (case["rows"] + 3 * case["batch"])}
    g, nd = _grid(case), case.get("n_det", 3)
    data = 24 * nd * g.n_freq                      # complex strain and PSD
    per_sample = 25 + 30 + 8 * nd                  # phase, sine and cosine, one complex product per detector
    dist = 4 * N_DIST                              # one exponent per distance
    full = _samples(g) * per_sample
    het = (case.get("n_bins", 0) + 1) * (25 + 46 * nd)
    if kind == "cache":
        return {"bytes": data + 116 * (case["slots"] + case["rows"]),
                "flops": (case["slots"] + case["rows"]) * (full + dist)}
    if kind == "sweep":                            # about six evaluations per chain and block
        rows = 6 * len(BLOCKS) * case["chains"]
        each = full if case["like"] == "full" else het
        table = data if case["like"] == "full" else 8 * (case["n_bins"] + 1) * (6 + 7 * nd)
        return {"bytes": table + 192 * case["chains"],
                "flops": rows * (each + dist)}
    rows = case["rows"]
    each = full if case["like"] == "full" else het
    if case["marg"] == "dist":
        each += dist
    if case["marg"] == "time":
        n, nt = _time_points(g)
        each += 5.0 * nt * math.log2(nt) + 20.0 * nt  # transform and ln I0 of every grid point
    return {"bytes": (data if case["like"] == "full" else 8 * (case["n_bins"] + 1) * (6 + 7 * nd)) + 112 * rows,
            "flops": rows * each}


# -- the same results from plain torch and numpy in 64 bits --------------------

MSUN_S, C_SI, MPC_SI = 4.925490947641267e-6, 299792458.0, 3.085677581491367e22


def _phase(th, f):
    """TaylorF2 phase (rad) of rows th [n, 13] at frequencies f [m] -> [n, m]."""
    mc, q, s1, s2, l1, l2 = (th[:, j, None] for j in range(6))
    x1 = 1.0 / (1.0 + q)
    x2 = q * x1
    eta, d = x1 * x2, x1 - x2
    v = (math.pi * mc * eta ** -0.6 * MSUN_S * f[None, :]) ** (1.0 / 3.0)
    pi, e2, e3 = math.pi, eta ** 2, eta ** 3
    sl = x1 * x1 * s1 + x2 * x2 * s2
    ds = d * (x2 * s2 - x1 * s1)
    p2 = 3715.0 / 756.0 + 55.0 / 9.0 * eta
    p3 = -16.0 * pi + (s1 * (113.0 * x1 * x1 + 75.0 * eta) + s2 * (113.0 * x2 * x2 + 75.0 * eta)) / 3.0
    p4 = (15293365.0 / 508032.0 + 27145.0 / 504.0 * eta + 3085.0 / 72.0 * e2
          - 10.0 * (79.0 / 8.0 * eta * s1 * s2 + 81.0 / 16.0 * ((x1 * s1) ** 2 + (x2 * s2) ** 2)))
    p5 = (pi * (38645.0 / 756.0 - 65.0 / 9.0 * eta) - (554345.0 / 1134.0 + 110.0 / 9.0 * eta) * sl
          - (13915.0 / 84.0 - 10.0 / 3.0 * eta) * ds)
    p6 = (11583231236531.0 / 4694215680.0 - 640.0 / 3.0 * pi ** 2 - 6848.0 / 21.0 * (0.5772156649015329 + math.log(4.0))
          + (-15737765635.0 / 3048192.0 + 2255.0 / 12.0 * pi ** 2) * eta + 76055.0 / 1728.0 * e2 - 127825.0 / 1296.0 * e3
          + pi * (3760.0 * sl + 1490.0 * ds) / 3.0)
    p7 = (pi * (77096675.0 / 254016.0 + 378515.0 / 1512.0 * eta - 74045.0 / 756.0 * e2)
          + (-8980424995.0 / 762048.0 + 6586595.0 / 756.0 * eta - 305.0 / 36.0 * e2) * sl
          - (170978035.0 / 48384.0 - 2876425.0 / 672.0 * eta - 4735.0 / 144.0 * e2) * ds)
    lp, lm = l1 + l2, l1 - l2
    lt = 8.0 / 13.0 * ((1.0 + 7.0 * eta - 31.0 * e2) * lp + d * (1.0 + 9.0 * eta - 11.0 * e2) * lm)
    dlt = 0.5 * (d * (1.0 - 13272.0 / 1319.0 * eta + 8944.0 / 1319.0 * e2) * lp
                 + (1.0 - 15910.0 / 1319.0 * eta + 32850.0 / 1319.0 * e2 + 3380.0 / 1319.0 * e3) * lm)
    lv = torch.log(v)
    t10 = -19.5 * lt
    t12 = -3115.0 / 64.0 * lt + 6595.0 / 364.0 * d * dlt
    s = 1.0 + v * v * (p2 + v * (p3 + v * (p4 + v * (p5 * (1.0 + 3.0 * lv) + v * (p6 - 6848.0 / 21.0 * lv + v * (
        p7 + v * v * v * (t10 + v * v * t12)))))))
    return 2.0 * pi * f * th[:, 12, None] - th[:, 11, None] - 0.25 * pi + 3.0 / (128.0 * eta * v ** 5) * s


def _project(th, prob):
    """Per detector: complex amplitude of f^(-7/6) exp(-i Psi) [n] and delay [n] (s)."""
    ph, dec, psi, ci = th[:, 8] - prob.gmst, th[:, 9], th[:, 10], torch.cos(th[:, 7])
    z = torch.zeros_like(ph)
    s = torch.stack([torch.cos(dec) * torch.cos(ph), torch.cos(dec) * torch.sin(ph), torch.sin(dec)])
    m = torch.stack([-torch.sin(ph), torch.cos(ph), z])
    n = torch.stack([-torch.sin(dec) * torch.cos(ph), -torch.sin(dec) * torch.sin(ph), torch.cos(dec)])
    X = -torch.cos(psi) * m + torch.sin(psi) * n
    Y = torch.sin(psi) * m + torch.cos(psi) * n
    amp = (math.sqrt(5.0 / 24.0) * math.pi ** (-2.0 / 3.0) * C_SI / (th[:, 6] * MPC_SI)
           * (th[:, 0] * MSUN_S) ** (5.0 / 6.0))
    out = []
    for i in range(prob.data.shape[0]):
        D = torch.from_numpy(prob.det_tensor[i]).to(th.device)
        r = torch.from_numpy(prob.det_pos[i]).to(th.device)
        fp = (X * (D @ X)).sum(0) - (Y * (D @ Y)).sum(0)
        fx = (X * (D @ Y)).sum(0) + (Y * (D @ X)).sum(0)
        out.append((torch.complex(amp * fp * 0.5 * (1.0 + ci * ci), -amp * fx * ci), -(r @ s) / C_SI))
    return out


def _strain(th, prob, f=None):
    """Projected templates [n, n_det, m]."""
    f = torch.from_numpy(prob.freqs).to(th.device) if f is None else f
    g = f ** (-7.0 / 6.0) * torch.exp(-1j * _phase(th, f))
    return torch.stack([a[:, None] * g * torch.exp(-2j * math.pi * f[None, :] * dt[:, None])
                        for a, dt in _project(th, prob)], dim=1)


def _log_i0(x):
    return x + torch.log(torch.special.i0e(x))


def _marginal(th, z, hh, dd, marg, prob):
    """log L from the overlap z [n] and norm hh [n] (taken at d_L = 1 Mpc for the distance marginal)."""
    if marg == "none":
        return -0.5 * dd + z.real - 0.5 * hh
    if marg == "phase":
        return -0.5 * dd - 0.5 * hh + _log_i0(z.abs())
    d = torch.from_numpy(prob.dist_grid).to(z.device)[None, :]
    w = torch.from_numpy(prob.dist_logw).to(z.device)[None, :]
    return -0.5 * dd + torch.logsumexp(w - 0.5 * hh[:, None] / (d * d) + _log_i0(z.abs()[:, None] / d), dim=1)


def _as_marg(th, marg):
    th = th.clone()
    if marg != "none":
        th[:, 11] = 0.0
    if marg == "dist":
        th[:, 6] = 1.0
    if marg == "time":
        th[:, 12] = 0.0
    return th


def _exact_full(prob, theta, marg):
    psd = torch.from_numpy(prob.psd).to(DEV)
    u = 4.0 * prob.df * torch.from_numpy(prob.data.conj()).to(DEV) / psd
    dd = float(np.sum(4.0 * prob.df * np.abs(prob.data) ** 2 / prob.psd))
    th = _as_marg(torch.from_numpy(theta).to(DEV), marg)
    out = torch.empty(len(theta), dtype=torch.float64, device=DEV)
    step = max(1, (1 << 22) // prob.n_freq)
    for a in range(0, len(theta), step):
        t = th[a:a + step]
        h = _strain(t, prob)
        hh = (4.0 * prob.df * (h.real ** 2 + h.imag ** 2) / psd).sum((1, 2))
        y = (u * h).sum(1)
        if marg != "time":
            out[a:a + step] = _marginal(t, y.sum(1), hh, dd, marg, prob)
            continue
        n, nt = _time_points(prob)
        pad = torch.zeros((len(t), n * OVERSAMPLE), dtype=torch.complex128, device=DEV)
        pad[:, prob.k0:prob.k0 + prob.n_freq] = y
        z = torch.fft.fft(pad, dim=1).abs()
        j = nt // 2
        li = _log_i0(torch.cat([z[:, :j + 1], z[:, -j:]], dim=1))
        out[a:a + step] = -0.5 * dd - 0.5 * hh + torch.logsumexp(li, dim=1) - math.log(nt)
    return out.cpu().numpy()


def _edges(prob, n_bins):
    """Bin edges of equal steps of the phase bound, as indices into the fine grid."""
    f = prob.freqs
    phi = sum(math.copysign(1.0, g) * (f / (f[-1] if g > 0 else f[0])) ** g
              for g in (-5.0 / 3.0, -2.0 / 3.0, 1.0, 5.0 / 3.0, 7.0 / 3.0))
    fe = np.interp(phi[0] + np.arange(n_bins + 1) * (phi[-1] - phi[0]) / n_bins, phi, f)
    e = np.clip(np.rint((fe - f[0]) / (f[1] - f[0])).astype(np.int64), 0, len(f) - 1)
    e[0], e[-1] = 0, len(f) - 1
    return np.unique(e)


def _exact_het(prob, theta0, theta, marg, n_bins):
    e = _edges(prob, n_bins)
    f, fe = prob.freqs, prob.freqs[e]
    h0 = _strain(torch.from_numpy(theta0[None]).to(DEV), prob)[0].cpu().numpy()
    w = 4.0 * prob.df / prob.psd
    dh, hh0 = np.conj(prob.data) * h0 * w, np.abs(h0) ** 2 * w
    b = np.minimum(np.searchsorted(e, np.arange(len(f)), side="right") - 1, len(e) - 2)
    dfc = f - 0.5 * (fe[b] + fe[b + 1])
    red = lambda v: torch.from_numpy(np.add.reduceat(v, e[:-1], axis=1)).to(DEV)  # noqa: E731
    A0, A1, B0, B1 = red(dh), red(dh * dfc), red(hh0), red(hh0 * dfc)
    dd = float(np.sum(w * np.abs(prob.data) ** 2))
    th = _as_marg(torch.from_numpy(theta).to(DEV), marg)
    fet = torch.from_numpy(fe).to(DEV)
    wid = torch.diff(fet)
    r0e = torch.from_numpy(h0[:, e]).to(DEV)
    out = torch.empty(len(theta), dtype=torch.float64, device=DEV)

    def sums(r):  # ratios [n, n_det, edges] -> overlap and norm [n]
        r0, r1 = 0.5 * (r[..., 1:] + r[..., :-1]), (r[..., 1:] - r[..., :-1]) / wid
        z = (A0 * r0 + A1 * r1).sum((-2, -1))
        return z, (B0 * (r0.real ** 2 + r0.imag ** 2) + 2.0 * B1 * (r0 * r1.conj()).real).sum((-2, -1))

    if marg != "time":
        step = max(1, (1 << 22) // len(e))
        for a in range(0, len(theta), step):
            t = th[a:a + step]
            z, hh = sums(_strain(t, prob, fet) / r0e)
            out[a:a + step] = _marginal(t, z, hh, dd, marg, prob)
        return out.cpu().numpy()
    n, nt = _time_points(prob)
    t = torch.arange(-(nt // 2), nt // 2 + 1, dtype=torch.float64, device=DEV) / (n * prob.df * OVERSAMPLE)
    # both sums are linear in what the shift multiplies: edge phasors in the overlap,
    # products of neighbouring edges in the norm
    shift = torch.exp(-2j * math.pi * fet[:, None] * t[None, :])
    wshift = torch.exp(-2j * math.pi * wid[:, None] * t[None, :])
    for a in range(0, len(theta), 64):
        r = _strain(th[a:a + 64], prob, fet) / r0e
        lo, hi = r[..., :-1], r[..., 1:]
        we = torch.zeros_like(r)
        we[..., 1:] += (0.5 * A0 + A1 / wid) * hi
        we[..., :-1] += (0.5 * A0 - A1 / wid) * lo
        z = we.sum(1) @ shift
        # |r0|^2 = (|lo|^2 + |hi|^2 + 2 Re(hi lo*)) / 4 and Re(r0 r1*) = (|hi|^2 - |lo|^2) / (2 w)
        al, ah = lo.abs() ** 2, hi.abs() ** 2
        const = (B0 * 0.25 * (al + ah) + B1 * (ah - al) / wid).sum((1, 2))
        cross = (0.5 * B0 * hi * lo.conj()).sum(1) @ wshift
        hh = const[:, None] + cross.real
        out[a:a + 64] = -0.5 * dd + torch.logsumexp(_log_i0(z.abs()) - 0.5 * hh, dim=1) - math.log(nt)
    return out.cpu().numpy()


def exact(case, seed):
    kind = case["kind"]
    if kind == "sweep":
        return None
    if kind == "network":
        x, xb, lb, (xm, xs, ym, ys) = _network_io(case, seed)
        params = [(torch.from_numpy(w).to(DEV).double().requires_grad_(),
                   torch.from_numpy(b).to(DEV).double().requires_grad_()) for w, b in _network(seed)]

        def net(v):
            a = (torch.from_numpy(v).to(DEV) - 0.5) / xs[0]
            for i, (w, b) in enumerate(params):
                a = a @ w + b
                if i < 3:
                    a = 0.5 * a * (1.0 + torch.erf(a / math.sqrt(2.0)))
            return a[:, 0]

        with torch.no_grad():
            pred = ym + ys * net(x)
        loss = ((net(xb) - (torch.from_numpy(lb).to(DEV) - ym) / ys) ** 2).mean()
        loss.backward()
        grads = torch.cat([torch.cat([w.grad.ravel(), b.grad]) for w, b in params])
        return pred.cpu().numpy(), grads.cpu().numpy(), float(loss)
    prob, theta0 = _problem(case, seed)
    if kind == "cache":
        base, _, fast = _cache_rows(case, theta0, seed)
        return _exact_full(prob, base, "dist"), _exact_full(prob, fast, "dist")
    rows = _rows(theta0, seed, case["rows"])
    if case["like"] == "full":
        return _exact_full(prob, rows, case["marg"])
    if case["marg"] != "time" and case["rows"] * case["n_bins"] > 1.2e8:
        return None
    return _exact_het(prob, theta0, rows, case["marg"], case["n_bins"])
