"""The work a user of this library has it do, as timed cases.

Every case goes through the public entry points of `paper_1505_00965_amd.mlmc`
with the models, payoffs and sizes of `workloads.py`, `bench.py` and the tests
(GBM and Heston at S0 = 100, strikes 100, M = 2 or 4): whole adaptive
estimates (device-planned and per-level), single level sums, the four-payoff
batch of all levels, the standard Monte Carlo comparator, the randomised
estimator and training of the control-variate network.  The random numbers
come from a counter generator keyed by the case's seed, so a seed fixes the
inputs; `exact` draws the same numbers and steps every path in fp64 torch.
"""
import math

import numpy as np
import torch

from paper_1505_00965_amd import mlmc as A
from paper_1505_00965_amd import workloads as W

DEV = "cuda:0"
GBM, HESTON = 0, 1
PAYOFFS = {"call": W.CALL, "asian": W.ASIAN, "lookback": W.LOOKBACK, "digital": W.DIGITAL}
# Philox streams of the estimation, training and comparator samples (the
# bridge uniforms of each follow at +1), network weights, level draws
S_EST, S_TRAIN, S_STD, S_DRAW = 0, 2, 4, 7


# ------------------------------------------------------------------- cases
def listed():
    return [
        # one estimate at the accuracy users ask for (0.1% of spot): two short
        # iterations, all latency
        dict(name="run_planned_rmse_1e-3", kind="run", model="gbm", payoff="call", M=4, eps=0.1,
             pilot=10000, persistent=True, precision=32, cv="none"),
        # the benchmark's estimate: 2e8 samples at level 0
        dict(name="run_planned_rmse_2e-5", kind="run", model="gbm", payoff="call", M=4, eps=2e-3,
             pilot=10000, persistent=True, precision=32, cv="none"),
        # the default form of mlmc_run on the stochastic-volatility model
        dict(name="run_levels_heston_1e-4", kind="run", model="heston", payoff="call", M=4, eps=1e-2,
             pilot=10000, persistent=False, precision=32, cv="none"),
        # an estimate with the learned control variate, tabulated
        dict(name="run_planned_cv_table", kind="run", model="heston", payoff="call", M=4, eps=5e-2,
             pilot=10000, persistent=True, precision=32, cv="table"),
        # one level's sums for a pilot: the smallest call
        dict(name="level_pilot_1000", kind="level", model="gbm", payoff="call", M=4, l=2, N=1000,
             offset=0, precision=32, scheme=0, anti=0, cv="none"),
        # few very long paths from a serving loop that may not allocate
        dict(name="noalloc_deep_asian", kind="noalloc", model="gbm", payoff="asian", M=4, l=8, N=331,
             offset=0, precision=32, scheme=1, anti=0, cv="none"),
        # an odd range of a level with the dearest plain payoff, M = 2
        dict(name="level_lookback_ragged", kind="level", model="gbm", payoff="lookback", M=2, l=6,
             N=1000003, offset=12345, precision=32, scheme=0, anti=0, cv="none"),
        # the fp64 path option, as the parity checks and error studies use it
        dict(name="level_fp64", kind="level", model="gbm", payoff="call", M=4, l=3, N=1048576,
             offset=0, precision=64, scheme=0, anti=0, cv="none"),
        # four payoffs on one model, levels 0..8 in one call: the largest
        dict(name="batch_four_payoffs", kind="batch", model="gbm", payoff="all", M=4, L=8, n0=2 ** 26,
             scheme=0),
        # the comparator of the complexity experiment (uncoupled paths, M = 2)
        dict(name="stdmc_digital", kind="stdmc", model="gbm", payoff="digital", M=2, l=6, N=4000037,
             precision=32, scheme=0),
        # the randomised single-term estimator with the scheme it needs
        dict(name="randomised_milstein", kind="rg", model="gbm", payoff="call", M=4, L=6, N=4194304,
             precision=32, scheme=1),
        # Adam steps of the control-variate network (forward and backward)
        dict(name="train_asian", kind="train", model="gbm", payoff="asian", M=4, lmax=3, steps=8,
             batch=16384),
    ]


def _log(rng, lo, hi):
    """An odd size, uniform over the logarithm of [lo, hi]."""
    return max(int(lo), min(int(hi), int(math.exp(rng.uniform(math.log(lo), math.log(hi)))) | 1))


def draw(rng):
    kind = rng.choice(["level"] * 6 + ["run"] * 4 + ["noalloc", "batch", "stdmc", "rg", "train", "train"])
    model = rng.choice(["gbm", "gbm", "heston"])
    payoff = rng.choice(["call", "asian", "lookback", "digital"])
    M = rng.choice([2, 4, 4])
    scheme = 0 if model == "heston" else rng.choice([0, 0, 1])
    if kind == "run":
        cv = rng.choice(["none", "none", "none", "table"])
        eps = math.exp(rng.uniform(math.log(8e-3), math.log(0.3)))
        if payoff == "digital":
            eps = max(eps / 50.0, 1e-3)     # the digital pays 1, not ~10
        precision = 64 if cv == "none" and rng.random() < 0.2 else 32
        return dict(kind="run", model=model, payoff=payoff, M=M, eps=round(eps, 7),
                    pilot=_log(rng, 1000, 20000), persistent=precision == 32 and rng.random() < 0.6,
                    precision=precision, cv=cv)
    if kind in ("level", "noalloc", "stdmc"):
        cv = "none"
        precision = rng.choice([32, 32, 32, 64])
        anti = int(kind != "stdmc" and rng.random() < 0.15)
        if kind == "level" and rng.random() < 0.3:
            cv, precision, anti, scheme = rng.choice(["net", "table"]), 32, 0, 0
        l = rng.randint(0, 6) if M == 4 else rng.randint(0, 12)
        nf = M ** l
        steps = 2 ** 28 if payoff != "lookback" and model == "gbm" else 2 ** 27
        if precision == 64:
            steps //= 4
        if cv == "net":
            steps //= 32
        N = _log(rng, 100, max(200, min(2 ** 26, steps // nf)))
        c = dict(kind=kind, model=model, payoff=payoff, M=M, l=l, N=N, precision=precision,
                 scheme=scheme)
        if kind != "stdmc":
            c.update(offset=rng.choice([0, rng.randrange(1, 100000)]), anti=anti, cv=cv)
        return c
    if kind == "batch":
        return dict(kind="batch", model=model, payoff=rng.choice(["all", payoff]), M=M,
                    L=rng.randint(2, 8), n0=_log(rng, 10000, 2 ** 23), scheme=scheme)
    if kind == "rg":
        return dict(kind="rg", model="gbm", payoff=payoff, M=M, L=rng.randint(2, 6),
                    N=_log(rng, 10000, 2 ** 22), precision=32, scheme=1)
    return dict(kind="train", model=model, payoff=payoff, M=M, lmax=rng.randint(1, 3),
                steps=rng.randint(2, 6), batch=_log(rng, 1024, 16384))


# ------------------------------------------------------- inputs and the call
def _model_dict(case):
    m = dict(W.HESTON_MODEL if case["model"] == "heston" else W.GBM_MODEL)
    m.update(scheme=case.get("scheme", 0), antithetic=case.get("anti", 0))
    return m


def _payoffs(case):
    names = list(PAYOFFS) if case["payoff"] == "all" else [case["payoff"]]
    return [PAYOFFS[n] for n in names]


def _levels_n(case):
    return [max(1, case["n0"] // case["M"] ** l) for l in range(case["L"] + 1)]


def _q(case):
    return case["M"] ** -1.5


def _net_weights(seed, d):
    """A network as training leaves it: weights of unit scale and an output
    near the hedge ratio (0.57 of sref S0 at the money)."""
    r = np.random.RandomState(seed % (2 ** 31))
    w1 = r.uniform(-1, 1, (64, d)) * math.sqrt(6.0 / (64 + d))
    w2 = r.uniform(-1, 1, (64, 64)) * math.sqrt(6.0 / 128)
    w3 = 0.2 * r.uniform(-1, 1, 64) * math.sqrt(6.0 / 65)
    return np.concatenate([w1.ravel(), 0.1 * r.randn(64), w2.ravel(), 0.1 * r.randn(64), w3,
                           [0.55]]).astype(np.float32)


def prepare(case, seed):
    m = _model_dict(case)
    s = {"case": case, "seed": seed, "m": A.model(**m), "p": [A.payoff(**p) for p in _payoffs(case)],
         "ctx": A.Context(0), "cv": None}
    if case["kind"] == "noalloc":
        s["out"] = torch.zeros(9, dtype=torch.float64, device=DEV)
    if case["kind"] == "batch":
        s["N"] = [_levels_n(case)] * len(s["p"])
    if case["kind"] == "train" or case.get("cv", "none") != "none":
        d = 3 if case["model"] == "heston" else 2
        s["cv"] = A.ControlVariate(s["ctx"], in_dim=d, init_seed=seed)
        s["cv"].set_params(_net_weights(seed, d))
        if case.get("cv") == "table":
            s["cv"].set_tabulated(True)
    return s


def run(s):
    c, ctx, m, p, seed = s["case"], s["ctx"], s["m"], s["p"][0], s["seed"]
    kind = c["kind"]
    if kind == "run":
        r = ctx.mlmc_run(m, p, c["eps"], M=c["M"], L_min=2, L_max=8 if c["M"] == 4 else 12,
                         n_pilot=c["pilot"], seed=seed, precision=c["precision"],
                         persistent=c["persistent"], cv=s["cv"], allow_notconv=True)
        return _run_out(r)
    if kind == "level":
        return ctx.mlmc_level(m, p, c["l"], c["M"], c["N"], seed, path_offset=c["offset"],
                              precision=c["precision"], cv=s["cv"])
    if kind == "noalloc":
        A.mlmc_level_noalloc(m, p, c["l"], c["M"], c["N"], seed, s["out"], path_offset=c["offset"],
                             precision=c["precision"], stream=torch.cuda.current_stream())
        return s["out"]
    if kind == "stdmc":
        return ctx.mlmc_stdmc(m, p, c["l"], c["M"], c["N"], seed, precision=c["precision"])
    if kind == "batch":
        return _batch_out(ctx.mlmc_levels_batch(m, s["p"], c["M"], c["L"], s["N"], seed))
    if kind == "rg":
        r = ctx.mlmc_rhee_glynn(m, p, c["M"], c["L"], _q(c), c["N"], seed, precision=c["precision"])
        r.pop("wall_s")
        return r
    hist = s["cv"].train(m, p, M=c["M"], lmax=c["lmax"], steps=c["steps"], batch=c["batch"], lr=1e-3,
                         seed=seed)
    return {"loss": hist, "params": s["cv"].get_params()}


def _run_out(r):
    """An estimate without its wall-clock time, per-level values as arrays of
    the most levels there can be."""
    r = {k: v for k, v in r.items() if k != "wall_s"}
    for k in ("N", "E", "V", "C", "sum_y", "sum_y2"):
        a = np.zeros(A.MAX_LEVELS, dtype=np.int64 if k == "N" else np.float64)
        a[:len(r[k])] = r[k]
        r[k] = a
    return r


FIELDS = ("sum_y", "sum_y2", "sum_pf", "sum_pf2", "sum_pc", "sum_pc2", "cost")


def _batch_out(res):
    out = {f: np.array([[r[f] for r in row] for row in res]) for f in FIELDS}
    out["n"] = np.array([[r["n"] for r in row] for row in res], dtype=np.int64)
    return out


# ------------------------------------------------------------ work of a pass
def _step_ops(model, payoff, M, scheme=0, anti=0, coupled=True):
    """Operations per fine step: a generator block's share (80 per four words),
    Box-Muller, the steps of both paths, payoff accumulators."""
    ops = 40.0 + 13.0 + 12.0 if model == "heston" else 20.0 + 13.0 / 2 + 4.0
    ops = ops / 2 + 6.0
    if coupled:
        ops += (6.0 if model == "heston" else 2.0) / M + 1.0
    ops += 2.0 * scheme + (2.0 if anti else 0.0)
    if payoff == "asian":
        ops += 4.0 + (4.0 / M if coupled else 0.0)
    if payoff == "lookback":
        ops += 10.0 + 5.0 + 10.0 + (12.0 if coupled else 0.0)
    return ops


PHI_OPS = 2.0 * 64 * 64 + 12.0 * 64      # one network evaluation (multiply-adds count 2)


def _level_ops(case, l, N, payoff=None, coupled=True):
    nf = case["M"] ** l
    c = coupled and l > 0
    ops = N * (nf * _step_ops(case["model"], payoff or case["payoff"], case["M"], case.get("scheme", 0),
                              case.get("anti", 0), c) + 11.0)
    pts = N * (nf + (nf / case["M"] if l else 0)) if l else 0
    if case.get("cv") == "net":
        ops += pts * PHI_OPS
    if case.get("cv") == "table":
        ops += pts * (40.0 if case["model"] == "heston" else 16.0)
    return ops


def work(case):
    kind = case["kind"]
    if kind in ("level", "noalloc", "stdmc"):
        return {"bytes": 72, "flops": _level_ops(case, case["l"], case["N"], coupled=kind != "stdmc")}
    if kind == "batch":
        names = list(PAYOFFS) if case["payoff"] == "all" else [case["payoff"]]
        f = sum(_level_ops(case, l, n, payoff=p) for p in names for l, n in enumerate(_levels_n(case)))
        return {"bytes": 72 * len(names) * (case["L"] + 1), "flops": f}
    if kind == "rg":
        q = _q(case)
        pl = [(1 - q) * q ** l / (1 - q ** (case["L"] + 1)) for l in range(case["L"] + 1)]
        return {"bytes": 600, "flops": sum(_level_ops(case, l, case["N"] * p) for l, p in enumerate(pl)) +
                20.0 * case["N"]}
    if kind == "train":
        B, M = case["batch"], case["M"]
        pts = sum(B * (M ** l + (M ** (l - 1) if l else 0)) for l in range(case["lmax"] + 1))
        np_ = 4481 if case["model"] == "heston" else 4417
        return {"bytes": case["steps"] * np_ * 24, "flops": case["steps"] * pts * PHI_OPS * 3}
    # an estimate: the sample counts its accuracy needs, from rough level
    # variances of the payoff (the driver measures them)
    v0 = {"call": 200.0, "asian": 60.0, "lookback": 160.0, "digital": 0.25}[case["payoff"]]
    M = case["M"]
    V = [v0] + [(v0 / 4) * M ** -(0.5 * l if case["payoff"] == "digital" else 1.0 * l) for l in range(1, 5)]
    C = [1.0] + [M ** l + M ** (l - 1) for l in range(1, 5)]
    tot = sum(math.sqrt(v * c) for v, c in zip(V, C))
    n = [max(case["pilot"] if l < 3 else 0, 2 / case["eps"] ** 2 * math.sqrt(v / c) * tot)
         for l, (v, c) in enumerate(zip(V, C))]
    return {"bytes": 600, "flops": sum(_level_ops(case, l, x) for l, x in enumerate(n))}


# ------------------------------------------------------------ fp64 reference
def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 words of counters given as int64 tensors (broadcast)."""
    mask = 0xFFFFFFFF
    k0, k1 = seed & mask, (seed >> 32) & mask
    c = [x if torch.is_tensor(x) else torch.tensor(x, dtype=torch.int64, device=DEV) for x in (c0, c1, c2, c3)]
    for _ in range(10):
        pa, pb = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = [((pb >> 32) & mask) ^ c[1] ^ k0, pb & mask, ((pa >> 32) & mask) ^ c[3] ^ k1, pa & mask]
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    return torch.stack(torch.broadcast_tensors(*c), dim=-1)


def _u01(words):
    return ((words >> 8).double() + 0.5) * 2.0 ** -24


def _words(seed, l, s, stream, per_sample):
    """[n, per_sample] generator words of samples s: their own blocks, or for
    fewer than four words a block shared by neighbours."""
    if per_sample >= 4:
        j = torch.arange(per_sample // 4, device=DEV)[None, :]
        w = _philox(j, (s & 0xFFFFFFFF)[:, None], (l + 256 * (s >> 32))[:, None], stream, seed)
        return w.reshape(len(s), per_sample)
    q = 4 // per_sample
    b = s // q
    w = _philox(0, b & 0xFFFFFFFF, l + 256 * (b >> 32), stream, seed)
    at = (s % q)[:, None] * per_sample + torch.arange(per_sample, device=DEV)[None, :]
    return torch.gather(w, 1, at)


def _normals(seed, l, s, stream, per_sample):
    if per_sample == 1:                      # the other word of the sample's pair
        b, r = s // 4, s % 4
        w = _philox(0, b & 0xFFFFFFFF, l + 256 * (b >> 32), stream, seed)
        u = _u01(torch.gather(w, 1, torch.stack([r - r % 2, r - r % 2 + 1], 1)))
        rho = torch.sqrt(-2.0 * torch.log(u[:, 0]))
        ang = 2.0 * math.pi * u[:, 1]
        return (rho * torch.where(r % 2 == 0, torch.cos(ang), torch.sin(ang)))[:, None]
    u = _u01(_words(seed, l, s, stream, per_sample)).reshape(len(s), -1, 2)
    rho, ang = torch.sqrt(-2.0 * torch.log(u[..., 0])), 2.0 * math.pi * u[..., 1]
    return torch.stack([rho * torch.cos(ang), rho * torch.sin(ang)], -1).reshape(len(s), per_sample)


def _scan(x, op, start):
    """Running products or sums along axis 1, with the start value before them."""
    if x.shape[1] > 1024:
        return torch.cat([torch.full_like(x[:, :1], start),
                          (torch.cumprod if op is torch.mul else torch.cumsum)(x, 1)], 1)
    out = [torch.full_like(x[:, 0], start)]
    for k in range(x.shape[1]):
        out.append(op(out[-1], x[:, k]))
    return torch.stack(out, 1)


def _paths(m, dw, dwp, h):
    """States S (and v) at the grid points 0..n of Euler (or GBM Milstein)
    paths with increments dw [N, n] (dwp: Heston's independent factor)."""
    if m["kind"] == GBM:
        f = 1.0 + m["r"] * h + m["sigma"] * dw
        if m["scheme"]:
            f = f + 0.5 * m["sigma"] ** 2 * (dw * dw - h)
        return m["S0"] * _scan(f, torch.mul, 1.0), None
    rc = math.sqrt(1.0 - m["rho"] ** 2)
    S, v = torch.full_like(dw[:, 0], m["S0"]), torch.full_like(dw[:, 0], m["v0"])
    Ss, vs = [S], [v]
    for k in range(dw.shape[1]):
        vp = v.clamp(min=0)
        vol = vp.sqrt()
        S, v = (S + S * (m["r"] * h + vol * dw[:, k]),
                v + m["kappa"] * h * (m["theta"] - vp) + m["xi"] * vol * (m["rho"] * dw[:, k] + rc * dwp[:, k]))
        Ss.append(S)
        vs.append(v)
    return torch.stack(Ss, 1), torch.stack(vs, 1)


def _vol(m, v, like):
    return torch.full_like(like, m["sigma"]) if m["kind"] == GBM else v[:, : like.shape[1]].clamp(min=0).sqrt()


def _bridge(x0, x1, b, e):
    return (0.5 * (x0 + x1 - torch.sqrt((x1 - x0) ** 2 + b * b * e))).amin(1)


def _value(m, p, S, mn, h):
    disc = math.exp(-m["r"] * m["T"])
    x = S[:, -1]
    if p["kind"] == 0:
        u = (x - p["K"]).clamp(min=0)
    elif p["kind"] == 1:
        u = ((S[:, 1:].sum(1) + 0.5 * (m["S0"] - x)) * h / m["T"] - p["K"]).clamp(min=0)
    elif p["kind"] == 2:
        u = x - mn
    else:
        u = p["payout"] * ((x > p["K"]).double() + 0.5 * (x == p["K"]).double())
    return disc * u


def _pair(m, p, M, l, dw, dwp, e, phi=None, coupled=True):
    """Fine and coarse payoffs of samples with increments dw [N, n]; with a
    network phi each minus its sum phi(t, X) dW on its own grid."""
    n = dw.shape[1]
    h = m["T"] / n
    S, v = _paths(m, dw, dwp, h)
    mn = _bridge(S[:, :-1], S[:, 1:], _vol(m, v, dw) * S[:, :-1], e) if p["kind"] == 2 else None
    pf = _value(m, p, S, mn, h)
    if phi is not None:
        pf = pf - (phi(torch.arange(n, device=DEV), n, S[:, :-1], None if v is None else v[:, :-1]) * dw).sum(1)
    if l == 0 or not coupled:
        return pf, torch.zeros_like(pf)
    nc, H = n // M, M * h
    part = dw.reshape(len(dw), nc, M)
    dwc = part.sum(2)
    dwpc = None if dwp is None else dwp.reshape(len(dw), nc, M).sum(2)
    Sc, vc = _paths(m, dwc, dwpc, H)
    mc = None
    if p["kind"] == 2:
        # the coarse step refined at the fine times with frozen coefficients
        vol, X = _vol(m, vc, dwc)[..., None], Sc[:, :-1, None]
        w = _scan(part.reshape(-1, M), torch.add, 0.0)[:, 1:].reshape(part.shape)
        tau = h * torch.arange(1, M + 1, device=DEV, dtype=torch.float64)
        rel = m["r"] * tau + vol * w
        if m["scheme"]:
            rel = rel + 0.5 * m["sigma"] ** 2 * (w * w - tau)
        x1 = X + X * rel
        x0 = torch.cat([X, x1[..., :-1]], 2)
        mc = _bridge(x0.reshape(len(dw), n), x1.reshape(len(dw), n),
                     (vol * X).expand(-1, -1, M).reshape(len(dw), n), e)
    pc = _value(m, p, Sc, mc, H)
    if phi is not None:
        pc = pc - (phi(M * torch.arange(nc, device=DEV), n, Sc[:, :-1],
                       None if vc is None else vc[:, :-1]) * dwc).sum(1)
    return pf, pc


def _samples(m, p, M, l, first, N, seed, stream, phi=None, coupled=True, most=2 ** 24):
    """Yields (pf, pc) of samples first .. first + N - 1 in chunks."""
    n, d = M ** l, 2 if m["kind"] == HESTON else 1
    rows = max(1, (most // 64 if phi is not None else most) // (n * d))
    for a in range(first, first + N, rows):
        s = torch.arange(a, min(a + rows, first + N), device=DEV)
        z = _normals(seed, l, s, stream, n * d) * math.sqrt(m["T"] / n)
        dw, dwp = (z[:, 0::2], z[:, 1::2]) if d == 2 else (z, None)
        e = None
        if p["kind"] == 2:
            e = -2.0 * (m["T"] / n) * torch.log(_u01(_words(seed, l, s, stream + 1, n)))
        pf, pc = _pair(m, p, M, l, dw, dwp, e, phi, coupled)
        if m["antithetic"] and l:
            def back(x):
                return None if x is None else x.reshape(len(s), n // M, M).flip(2).reshape(len(s), n)
            qf, qc = _pair(m, p, M, l, back(dw), back(dwp), back(e))
            pf, pc = 0.5 * (pf + qf), 0.5 * (pc + qc) if p["kind"] == 2 else pc
        yield pf, pc


def _sums(*args, **kw):
    t = torch.zeros(6, dtype=torch.float64, device=DEV)
    for pf, pc in _samples(*args, **kw):
        y = pf - pc
        t += torch.stack([y.sum(), (y * y).sum(), pf.sum(), (pf * pf).sum(), pc.sum(), (pc * pc).sum()])
    return t.tolist()


def _cost(M, l, anti=0):
    return 1.0 if l == 0 else (2.0 if anti else 1.0) * M ** l + M ** (l - 1)


def _net(m, par):
    """phi(step numbers, steps of the fine grid, S, v) of the parameters."""
    d = 3 if m["kind"] == HESTON else 2
    o = np.cumsum([0, 64 * d, 64, 4096, 64, 64, 1])
    w1, b1, w2, b2, w3, b3 = (par[o[i]:o[i + 1]] for i in range(6))
    w1, w2 = w1.reshape(64, d), w2.reshape(64, 64)
    sref = m["sigma"] if m["kind"] == GBM else math.sqrt(m["theta"])

    def phi(t, S, v):
        x = [t.expand_as(S), torch.log(S.clamp(min=m["S0"] * 2.0 ** -40) / m["S0"]) / (sref * math.sqrt(m["T"]))]
        if d == 3:
            x.append((v - m["theta"]) / m["theta"])
        a = torch.tanh(torch.stack(x, -1).reshape(-1, d) @ w1.T + b1)
        a = torch.tanh(a @ w2.T + b2)
        return (sref * m["S0"] * (a @ w3 + b3)).reshape(S.shape)

    return phi


def _phi_of(m, par, form):
    """The network as the sampler takes it: evaluated, or from its table
    (linear in S, bilinear with v, in the last time row at or before t)."""
    net = _net(m, par)
    if form == "net":
        return lambda k, n, S, v: net(k.double() / n, S, v)
    he = m["kind"] == HESTON
    rows, ns, nv = (16, 16, 32) if he else (256, 32, 1)
    w = 4.0 * (math.sqrt(m["theta"]) if he else m["sigma"]) * math.sqrt(m["T"])
    lo, hi = m["S0"] * math.exp(-w), m["S0"] * math.exp(w)
    vhi = 4.0 * max(m["theta"], m["v0"])
    f64 = dict(dtype=torch.float64, device=DEV)
    T, Vg, Sg = torch.meshgrid(torch.arange(rows, **f64) / rows,
                               torch.arange(nv, **f64) * (vhi / max(nv - 1, 1)),
                               lo + torch.arange(ns, **f64) * ((hi - lo) / (ns - 1)), indexing="ij")
    tab = net(T, Sg, Vg)

    def look(k, n, S, v):
        row = ((k * rows) // n).expand(S.shape)
        u = ((S - lo) * ((ns - 1) / (hi - lo))).clamp(0, ns - 1)
        i = u.long().clamp(max=ns - 2)
        f = u - i

        def at(j):
            return tab[row, j, i] * (1 - f) + tab[row, j, i + 1] * f

        if not he:
            return at(torch.zeros_like(i))
        g = (v * ((nv - 1) / vhi)).clamp(0, nv - 1)
        j = g.long().clamp(max=nv - 2)
        g = g - j
        return at(j) * (1 - g) + at(j + 1) * g

    return look


def _exact_run(case, m, p, seed, phi):
    """The adaptive loop with every sum in fp64."""
    M, eps, Lmax = case["M"], case["eps"], 8 if case["M"] == 4 else 12
    L, n = 2, [0.0] * 16
    s1, s2, E, V, C = ([0.0] * 16 for _ in range(5))
    dN = [float(case["pilot"])] * 3 + [0.0] * 13
    it = 0
    while True:
        for l in range(L + 1):
            if dN[l] > 0:
                t = _sums(m, p, M, l, int(n[l]), int(dN[l]), seed, S_EST, phi=phi)
                s1[l], s2[l], n[l] = s1[l] + t[0], s2[l] + t[1], n[l] + dN[l]
            C[l] = _cost(M, l)
            E[l], V[l] = abs(s1[l] / n[l]), max(s2[l] / n[l] - (s1[l] / n[l]) ** 2, 0.0)
            if l >= 2:
                E[l], V[l] = max(E[l], E[l - 1] / M), max(V[l], V[l - 1] / M)
        it += 1

        def need():
            tot = sum(math.sqrt(V[l] * C[l]) for l in range(L + 1))
            return [math.ceil(2 / (eps * eps) * math.sqrt(V[l] / C[l]) * tot) for l in range(L + 1)]

        d = [x - n[l] for l, x in enumerate(need())]
        dN = [x if x > 0.01 * n[l] else 0.0 for l, x in enumerate(d)] + [0.0] * (15 - L)
        if not any(dN):
            bias = max(E[L], E[L - 1] / M) / (M - 1.0)
            done = bias <= eps / math.sqrt(2.0)
            if done or L == Lmax:
                break
            L += 1
            V[L], E[L], C[L] = V[L - 1] / M, E[L - 1] / M, _cost(M, L)
            N = need()
            dN = [x - n[l] if x - n[l] > 0.01 * n[l] else 0.0 for l, x in enumerate(N)] + [0.0] * (15 - L)
            dN[L] = max(float(N[L]), 1.0)
    k = L + 1
    e = [s1[l] / n[l] for l in range(k)]
    v = [s2[l] / n[l] - e[l] ** 2 for l in range(k)]
    var = sum(max(v[l], 0) / n[l] for l in range(k))

    def rate(y):
        at = [(l, math.log(y[l]) / math.log(M)) for l in range(1, k) if y[l] > 0]
        return float(np.polyfit([a for a, _ in at], [b for _, b in at], 1)[0])

    return _run_out({"estimate": sum(e), "rmse_est": math.sqrt(var + bias ** 2), "L": L, "converged": bool(done),
                     "iterations": it, "alpha": -rate([abs(x) for x in e]), "beta": -rate(v),
                     "gamma": rate(C), "cost": sum(n[l] * C[l] for l in range(k)), "n_nonfinite": 0,
                     "N": [int(x) for x in n[:k]], "E": e, "V": v, "C": C[:k], "sum_y": s1[:k],
                     "sum_y2": s2[:k]})


def _exact_train(case, m, p, seed):
    """Adam on the training objective, gradients by autograd in fp64."""
    d = 3 if m["kind"] == HESTON else 2
    par = torch.tensor(_net_weights(seed, d), dtype=torch.float64, device=DEV)
    m1, m2 = torch.zeros_like(par), torch.zeros_like(par)
    B, M, hist = case["batch"], case["M"], []
    for k in range(case["steps"]):
        q = par.clone().requires_grad_(True)
        phi = _phi_of(m, q, "net")
        loss = 0.0
        for l in range(case["lmax"] + 1):
            got = list(_samples(m, p, M, l, k * B, B, seed, S_TRAIN, phi=phi, most=2 ** 40))
            y = torch.cat([f - c for f, c in got])
            loss = loss + torch.sqrt(_cost(M, l) * y.var())
        g, = torch.autograd.grad(loss, q)
        m1, m2 = 0.9 * m1 + 0.1 * g, 0.999 * m2 + 0.001 * g * g
        par = par - 1e-3 * (m1 / (1 - 0.9 ** (k + 1))) / (torch.sqrt(m2 / (1 - 0.999 ** (k + 1))) + 1e-8)
        hist.append(float(loss.detach()))
    return {"loss": np.array(hist), "params": par.detach().cpu().numpy()}


def exact(case, seed):
    kind, M = case["kind"], case["M"]
    m, ps = _model_dict(case), _payoffs(case)
    if kind == "train":
        return _exact_train(case, m, ps[0], seed)
    phi = None
    if case.get("cv", "none") != "none":
        par = torch.tensor(_net_weights(seed, 3 if case["model"] == "heston" else 2), dtype=torch.float64,
                           device=DEV)
        phi = _phi_of(m, par, case["cv"])
    if kind == "run":
        return _exact_run(case, m, ps[0], seed, phi)
    if kind in ("level", "noalloc", "stdmc"):
        std = kind == "stdmc"
        t = _sums(m, ps[0], M, case["l"], case.get("offset", 0), case["N"], seed, S_STD if std else S_EST,
                  phi=phi, coupled=not std)
        cost = case["N"] * (float(M ** case["l"]) if std else _cost(M, case["l"], case["anti"]))
        if kind == "noalloc":
            tail = torch.tensor([case["N"], 0], dtype=torch.int64).view(torch.float64)
            return torch.cat([torch.tensor(t + [cost], dtype=torch.float64), tail])
        return dict(zip(FIELDS, t + [cost]))
    if kind == "batch":
        rows = [[_sums(m, p, M, l, 0, n, seed, S_EST) + [n * _cost(M, l)]
                 for l, n in enumerate(_levels_n(case))] for p in ps]
        return {f: np.array([[c[i] for c in row] for row in rows]) for i, f in enumerate(FIELDS)}
    # the randomised estimator: levels drawn by inversion, then Y_L / p_L
    q, L, N = _q(case), case["L"], case["N"]
    pl = [(1 - q) * q ** l / (1 - q ** (L + 1)) for l in range(L + 1)]
    F = torch.tensor(np.cumsum(pl)[:-1], dtype=torch.float64, device=DEV)
    u = _u01(_words(seed, 0, torch.arange(N, device=DEV), S_DRAW, 1)[:, 0])
    cnt = torch.bincount(torch.searchsorted(F, u, right=True), minlength=L + 1).tolist()
    s = [_sums(m, ps[0], M, l, 0, n, seed, S_EST) if n else [0.0] * 6 for l, n in enumerate(cnt)]
    est = sum(t[0] / x for t, x in zip(s, pl)) / N
    var = sum(t[1] / (x * x) for t, x in zip(s, pl)) / N - est * est
    return {"estimate": est, "variance": var, "rmse_est": math.sqrt(max(var, 0.0) / N),
            "cost": float(sum(n * _cost(M, l) for l, n in enumerate(cnt))), "p": pl,
            # Milstein differences of deep levels are as small as fp32 steps round
            "sum_y": [t[0] if M ** l < 1024 else None for l, t in enumerate(s)],
            "sum_y2": [t[1] if M ** l < 1024 else None for l, t in enumerate(s)]}
