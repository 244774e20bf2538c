"""Timed cases of the framework's public entry points.

Each case is one piece of work that a user of the sampler has it do, called as a user's
program calls it:

  loglik   likelihood estimates of a set of parameter vectors (``pf_loglik``): profiling a
           likelihood, checking a fitted model, feeding an optimiser
  score    likelihood and score estimates (``pf_score``): gradient-based exploration
  sampler  one whole inference: a ``Sampler`` on new data, its K iterations, the records,
           the recycled estimate and the final population
  pmcmc    the comparison method (``PMCMC``), a set of chains advanced together

Sizes come from the presets of ``workloads``, scaled so that a pass takes at most about a
second, and from the odd sizes that the tests use.
"""
import math

import numpy as np
import torch

import paper_2311_12973_amd as G
from paper_2311_12973_amd import workloads as W

# algorithmic operations per particle-step, as the package's operation count gives them
# near the posterior (draws, attempts, Philox calls, transcendentals at 20 each); the score
# adds a division and a few products per flow, the linear-Gaussian step is one Box-Muller
# normal, one exponential and the weight
OPS = {"sir": 475.0, "seir": 650.0, "age": 1393.0, "lg": 190.0}
FAMILY = {"sir_fp64": "sir", "paper_sir": "sir", "seir": "seir", "seir_batched": "seir", "seir_learned": "seir",
          "age_seir": "age", "lingauss": "lg"}
PROPOSALS = {"rw": G.PROP_RW, "mlp": G.PROP_MLP, "langevin": G.PROP_LANGEVIN, "rw_pop": G.PROP_RW_POP}


def listed():
    return [
        # the smallest call: a handful of particles, where launches and the host count
        dict(name="loglik_sir_small", kind="loglik", preset="sir_fp64", n=64, nx=64, T=50),
        # a real-valued state-space model in FP64 at sizes that fill no wave or block evenly
        dict(name="loglik_lingauss_odd", kind="loglik", preset="lingauss", n=100, nx=257, T=100),
        # a likelihood surface over a thousand parameter vectors, odd particle count
        dict(name="loglik_seir_1000", kind="loglik", preset="seir_learned", n=1000, nx=1000, T=150),
        # a few expensive likelihoods of the age-structured model: fewer filters than CUs
        dict(name="loglik_age_few", kind="loglik", preset="age_seir", n=50, nx=1500, T=200),
        # likelihoods and scores together, multinomial resampling as in the paper's filter
        dict(name="score_seir_512", kind="score", preset="seir_learned", n=512, nx=500, T=100, multinomial=True),
        # a few chains, one small launch after another
        dict(name="pmcmc_paper", kind="pmcmc", preset="paper_sir", n=16, nx=500, T=30, K=64),
        # the paper's own experiment, FP64
        dict(name="sampler_paper_sir", kind="sampler", preset="paper_sir", n=1024, nx=500, T=30, K=10,
             proposal="rw", graph=False),
        # the SEIR shape, iterations replayed as a graph
        dict(name="sampler_seir", kind="sampler", preset="seir", n=1024, nx=512, T=100, K=5, proposal="rw",
             graph=True),
        # gradient-informed proposal: every filter carries its score
        dict(name="sampler_langevin", kind="sampler", preset="seir_learned", n=1024, nx=512, T=100, K=4,
             proposal="langevin", graph=False),
        # many uneven series in one context, population random walk
        dict(name="sampler_batched", kind="sampler", preset="seir_batched", n=256, nx=0, T=0, K=2, runs=48,
             proposal="rw_pop", graph=False),
        # the learned proposal at its preset's shape
        dict(name="sampler_learned", kind="sampler", preset="seir_learned", n=4096, nx=1024, T=150, K=3,
             proposal="mlp", graph=False),
        # the age-structured model, full length and particle count: the largest
        dict(name="sampler_age", kind="sampler", preset="age_seir", n=2048, nx=2048, T=365, K=2, proposal="mlp",
             graph=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any kind, model, proposal and resampling scheme, sizes over their whole
    range (evenly in the logarithm), within the largest listed case's work."""
    kind = rng.choice(["loglik", "loglik", "score", "sampler", "sampler", "pmcmc"])
    if kind == "loglik":
        preset = rng.choice(["sir_fp64", "paper_sir", "seir", "seir_learned", "age_seir", "lingauss"])
        c = dict(kind=kind, preset=preset, n=_log_int(rng, 1, 2000), nx=_log_int(rng, 33, 2048), T=_log_int(rng, 20, 365),
                 multinomial=rng.random() < 0.25)
    elif kind == "score":
        preset = rng.choice(["paper_sir", "seir_learned", "lingauss"])
        c = dict(kind=kind, preset=preset, n=_log_int(rng, 1, 1500), nx=_log_int(rng, 33, 1024), T=_log_int(rng, 20, 200),
                 multinomial=rng.random() < 0.25)
    elif kind == "pmcmc":
        preset = rng.choice(["sir_fp64", "paper_sir", "seir", "lingauss"])
        c = dict(kind=kind, preset=preset, n=_log_int(rng, 1, 200), nx=_log_int(rng, 64, 1024), T=_log_int(rng, 20, 100),
                 K=_log_int(rng, 20, 100))
    else:
        preset = rng.choice(["sir_fp64", "paper_sir", "seir", "seir_batched", "seir_learned", "age_seir"])
        runs = _log_int(rng, 2, 40) if preset == "seir_batched" else 1
        props = ["rw", "mlp", "rw_pop"] + ([] if preset == "age_seir" else ["langevin"])
        c = dict(kind=kind, preset=preset, n=_log_int(rng, 64, 256 if runs > 1 else 4096),
                 nx=0 if runs > 1 else _log_int(rng, 64, 2048 if preset == "age_seir" else 1024),
                 T=0 if runs > 1 else _log_int(rng, 20, 365 if preset == "age_seir" else 150),
                 K=_log_int(rng, 2, 10), runs=runs, proposal=rng.choice(props), graph=rng.random() < 0.5)
    if kind != "score":  # odd and even sizes alike, now and then a whole number of waves
        if c["nx"] > 64 and rng.random() < 0.3:
            c["nx"] = c["nx"] // 64 * 64
    largest = work(listed()[-1])["flops"]
    while work(c)["flops"] > 0.5 * largest:
        if c.get("K", 1) > 2:
            c["K"] = max(2, c["K"] // 2)
        else:
            c["n"] = max(1, c["n"] * 2 // 3)
    return c


def _workload(case):
    w = W.preset(case["preset"])
    if case.get("multinomial"):
        w["pf_resampling"] = G.PF_RS_MULTINOMIAL
    if case.get("proposal"):
        w["proposal"] = PROPOSALS[case["proposal"]]
    return w


def _series(w, T, seed):
    return W.simulate(w["model"], w["obs"], w["n_pop"], w["truth"], T, seed, w.get("fixed", ()))


def _run_shapes(case):
    """(T, n_x) of every run: the case's, or for the batched shape T in [30, 200] and n_x in
    {128, 256, 512, 1024}, the same for every seed."""
    if case.get("runs", 1) <= 1:
        return [(case["T"], case["nx"])]
    rng = np.random.default_rng(100000 + case["runs"])
    return [(int(rng.integers(30, 201)), int(rng.choice([128, 256, 512, 1024]))) for _ in range(case["runs"])]


def prepare(case, seed):
    w = _workload(case)
    base = 1000 * int(seed) + 17
    runs = [dict(T=T, nx=nx, seed=base + r, y=_series(w, T, base + 50000 + 64 * r))
            for r, (T, nx) in enumerate(_run_shapes(case))]
    state = dict(case=case, w=w, runs=runs)
    if case["kind"] in ("loglik", "score"):
        # parameter vectors about a fitted value, 10% apart (a likelihood surface)
        rng = np.random.default_rng(base)
        state["theta"] = np.array(w["truth"]) * np.exp(0.1 * rng.standard_normal((case["n"], w["D"])))
        if w["model"] == W.LINGAUSS:
            state["theta"][:, 0] = np.minimum(state["theta"][:, 0], 0.99)
    return state


def run(state):
    case, w, runs = state["case"], state["w"], state["runs"]
    r = runs[0]
    if case["kind"] == "loglik":
        return G.pf_loglik(w, state["theta"], r["y"], r["nx"], r["seed"], 1)
    if case["kind"] == "score":
        return G.pf_score(w, state["theta"], r["y"], r["nx"], r["seed"], 1)
    if case["kind"] == "pmcmc":
        s = G.PMCMC(w, r, case["n"], case["K"])
        s.step(case["K"])
        mean, cov, rate = s.estimate(case["K"] // 2)
        out = dict(mean=mean, cov=cov, rate=rate, phi=s.dump("phi"), ll=s.dump("ll"), accepted=s.dump("accepted"))
        s.close()
        return out
    s = G.Sampler(w, runs, N=case["n"], K=case["K"], use_graph=int(case["graph"]))
    for _ in range(case["K"]):
        s.step()
    each = []
    for i in range(len(runs)):
        mean, cov = s.estimate(run=i)
        each.append(dict(records=s.records(i), mean=mean, cov=cov, phi=s.dump("phi", i), ll=s.dump("ll", i)))
    s.close()
    return {k: np.stack([e[k] for e in each]) for k in each[0]}


def work(case):
    """One pass: each filter's operations (n_x x T particle-steps at the model's count), and
    the parameters, series and estimates that go in and out once. The particles themselves
    need no memory traffic."""
    w = W.preset(case["preset"])
    D, n = w["D"], case["n"]
    iters = {"sampler": case.get("K", 1), "pmcmc": case.get("K", 1) + 1}.get(case["kind"], 1)
    steps = obs = 0
    for T, nx in _run_shapes(case):
        steps += T * nx * n
        obs += T * W.n_obs(w["model"]) * (8 if w["model"] == W.LINGAUSS else 4)
    runs = case.get("runs", 1)
    per_sample = 8 * D + 8 + (8 * D if case["kind"] == "score" else 0) + (16 * D if case["kind"] == "sampler" else 0)
    return {"bytes": float(obs + iters * runs * n * per_sample), "flops": float(iters * steps * OPS[FAMILY[case["preset"]]])}


# ------------------------------------------------------------------ 64-bit values
# The FP64 filters (linear-Gaussian, SIR) in numpy, every filter and particle at once: the
# same counter-based streams, so the estimates themselves are comparable.
_M0, _M1 = np.uint64(0xD2511F53), np.uint64(0xCD9E8D57)
_LOW = np.uint64(0xFFFFFFFF)
_S32 = np.uint64(32)


def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 on broadcast counters; four uint64 arrays holding 32-bit words."""
    c = [np.asarray(x, dtype=np.uint64) for x in np.broadcast_arrays(c0, c1, c2, c3)]
    k0, k1 = seed & 0xFFFFFFFF, (seed >> 32) & 0xFFFFFFFF
    for _ in range(10):
        p0, p1 = _M0 * c[0], _M1 * c[2]
        c = [(p1 >> _S32) ^ c[1] ^ np.uint64(k0), p1 & _LOW, (p0 >> _S32) ^ c[3] ^ np.uint64(k1), p0 & _LOW]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return c


def _u24(x):
    return (2.0 * (x >> np.uint64(9)).astype(np.float64) + 1.0) * 2.0 ** -24


def _u53(lo, hi):
    return (2.0 * (((hi << _S32) | lo) >> np.uint64(12)).astype(np.float64) + 1.0) * 2.0 ** -53


def _normal(c0, c1, c2, c3, seed):
    w = _philox(c0, c1, c2, c3, seed)
    return np.sqrt(-2.0 * np.log(_u53(w[0], w[1]))) * np.cos(2.0 * math.pi * _u53(w[2], w[3]))


def _lgamma(x):
    return torch.lgamma(torch.from_numpy(np.asarray(x, dtype=np.float64))).numpy()


def _inversion(n, p, u):
    """Sequential search of the binomial distribution function, all elements in step."""
    f = np.exp(n * np.log1p(-p))
    total, k, r = f.copy(), np.zeros(n.shape), p / (1.0 - p)
    live = (u > total) & (k < np.minimum(n, 127))
    while live.any():
        f = np.where(live, f * ((n - k) * r / (k + 1.0)), f)
        k = np.where(live, k + 1.0, k)
        live &= total + f != total
        total = np.where(live, total + f, total)
        live &= (u > total) & (k < np.minimum(n, 127))
    return k


def _btrs(n, p, words):
    """Hoermann's transformed rejection, all elements in step; words(e) gives attempt e's pair."""
    spq = np.sqrt(n * p * (1.0 - p))
    b = 1.15 + 2.53 * spq
    a = -0.0873 + 0.0248 * b + 0.01 * p
    alpha, vr, centre, m = (2.83 + 5.1 / b) * spq, 0.92 - 4.2 / b, n * p + 0.5, np.floor((n + 1.0) * p)
    lpq, h = np.log(p / (1.0 - p)), _lgamma(m + 1.0) + _lgamma(n - m + 1.0)
    out, todo = m.copy(), np.arange(n.size)
    for e in range(256):
        if not todo.size:
            break
        wu, wv = words(e, todo)
        u, v = _u24(wu) - 0.5, _u24(wv)
        us = 0.5 - np.abs(u)
        at = lambda x: x[todo]  # noqa: E731
        k = np.floor((2.0 * at(a) / us + at(b)) * u + at(centre))
        inside = (k >= 0) & (k <= at(n))
        kk = np.where(inside, k, 0.0)
        lhs = np.log(v * at(alpha) / (at(a) / (us * us) + at(b)))
        rhs = at(h) - _lgamma(kk + 1.0) - _lgamma(at(n) - kk + 1.0) + (kk - at(m)) * at(lpq)
        ok = inside & (((us >= 0.07) & (v <= at(vr))) | (lhs <= rhs))
        out[todo[ok]] = k[ok]
        todo = todo[~ok]
    return out


def _binomial(n, p, j, i, kt, b, seed):
    """Binomial(n, p) for arrays n (float) and p in [0, 1] at the draws' coordinates."""
    n, p, j, i = (np.ascontiguousarray(x).reshape(-1) for x in np.broadcast_arrays(n, p, j, i))
    flip = p > 0.5
    pp = np.where(flip, 1.0 - p, p)
    some = (n > 0) & (p > 0) & (p < 1)
    k = np.zeros(n.shape)
    small = some & (n * pp < 10.0)
    large = some & ~small
    head = (1 << 24) | (b << 16)
    if small.any():
        k[small] = _inversion(n[small], pp[small], _u24(_philox(j[small], i[small], kt, head, seed)[0]))
    if large.any():
        jl, il = j[large], i[large]

        def words(e, at):
            w = _philox(jl[at], il[at], kt, head | (e >> 1), seed)
            return (w[2], w[3]) if e & 1 else (w[0], w[1])

        k[large] = _btrs(n[large], pp[large], words)
    return np.where(some & flip, n - k, np.where((n > 0) & (p >= 1), n, k))


def _resample(q, i, kt, seed, multinomial):
    """Ancestors of one filter's quantised weights q (uint64), exact integers."""
    n, C = q.size, np.cumsum(q)
    Q = int(C[-1])
    if multinomial:
        m = np.arange(n)
        w = _philox(m >> 1, i, kt, (2 << 24) | (1 << 16), seed)
        odd = (m & 1) == 1
        lo, hi = np.where(odd, w[2], w[0]), np.where(odd, w[3], w[1])
        U = np.array([((int(h) << 32 | int(x)) * Q) >> 64 for x, h in zip(lo, hi)], dtype=np.uint64)
        return np.searchsorted(C, U, side="right")
    w = _philox(0, i, kt, 2 << 24, seed)
    U = ((int(w[0]) | (int(w[1]) << 32)) * Q) >> 64
    return np.searchsorted(C * np.uint64(n), np.arange(n, dtype=np.uint64) * np.uint64(Q) + np.uint64(U), side="right")


def _filter_fp64(state):
    w, r, th = state["w"], state["runs"][0], state["theta"]
    n, nx, T, seed, kit = th.shape[0], r["nx"], r["T"], r["seed"], 1
    y = np.asarray(r["y"], dtype=np.float64).reshape(T, -1)[:, 0]
    i, j = np.arange(n)[:, None], np.arange(nx)[None, :]
    lg = w["model"] == W.LINGAUSS
    if lg:
        a, sq, sr = (th[:, d:d + 1] for d in range(3))
        x = [w["fixed"][0] + w["fixed"][1] * _normal(j, i, kit << 16, 8 << 24, seed)]
    else:
        x = [np.full((n, nx), float(w["n_pop"] - w["fixed"][0])), np.full((n, nx), float(w["fixed"][0]))]
        p_ir = -np.expm1(-th[:, 1:2])
    lw, ll, log_prev = np.zeros((n, nx)), np.zeros(n), np.full(n, math.log(nx))
    for t in range(1, T + 1):
        kt = (kit << 16) | t
        if lg:
            x = [a * x[0] + sq * _normal(j, i, kt, 8 << 24, seed)]
            z = (y[t - 1] - x[0]) / sr
            part, const = -0.5 * z * z, -np.log(sr[:, 0]) - 0.5 * math.log(2.0 * math.pi)
        else:
            new = _binomial(x[0], -np.expm1(-(th[:, :1] / w["n_pop"]) * x[1]), j, i, kt, 0, seed).reshape(n, nx)
            out = _binomial(x[1], np.broadcast_to(p_ir, x[1].shape), j, i, kt, 1, seed).reshape(n, nx)
            x = [x[0] - new, x[1] + new - out]
            mu = x[1] if w["obs"] == W.OBS_POIS_PREV else new
            with np.errstate(divide="ignore", invalid="ignore"):
                part = np.where(mu > 0, y[t - 1] * np.log(mu) - mu, 0.0 if y[t - 1] == 0 else -np.inf)
            const = -math.lgamma(y[t - 1] + 1.0)
        lw = lw + part
        m = lw.max(axis=1, keepdims=True)
        dead = ~np.isfinite(m[:, 0])
        lw = lw - np.where(dead[:, None], 0.0, m)
        wt = np.exp(lw)
        with np.errstate(divide="ignore"):
            ls = np.log(wt.sum(axis=1))
        ll = np.where(dead, -np.inf, ll + (m[:, 0] + ls - log_prev + const))
        log_prev = np.where(dead, log_prev, ls)
        if t == T:
            break
        q = np.floor(wt * 2.0 ** 32).astype(np.uint64)
        for f in np.flatnonzero(~dead & np.isfinite(ll)):
            h = q[f] >> np.uint64(8)
            s1, s2 = int(h.sum()), int((h * h).sum())
            if 2 * s1 * s1 < nx * s2:
                anc = _resample(q[f], int(f), kt, seed, state["case"].get("multinomial"))
                for c in x:
                    c[f] = c[f][anc]
                lw[f], log_prev[f] = 0.0, math.log(nx)
    return ll


def exact(case, seed):
    """The likelihood estimates in 64 bits. Only the FP64 filters have such a value: in FP32
    the rounding of a weight or a probability decides which trajectories the filter takes.
    The samplers and chains iterate on those decisions, and have none either."""
    if case["kind"] != "loglik" or W.preset(case["preset"])["prec"] != W.PREC_FP64:
        return None
    steps = case["n"] * case["nx"] * case["T"]
    if steps > (8e6 if FAMILY[case["preset"]] == "lg" else 1.5e6):  # about 20 seconds of numpy
        return None
    return _filter_fp64(prepare(case, seed))
