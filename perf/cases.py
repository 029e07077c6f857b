"""The work this package is timed on: whole sampler runs, likelihood calls and
weight updates, each through the public entry points.

listed() holds the cases, draw() makes more of the same ranges, prepare() builds
what a program holds before the call (data, sampler, captured buffers), run()
makes one pass and returns its results, work() counts the bytes and operations
a pass cannot do without, exact() gives the results in 64 bits where they have
such a value.

Kinds:
  smc      SMCSampler: prior draws, then `steps` tempering steps as hipGraph replays
  pt       PTSampler: prior draws, then `steps` population-MCMC iterations
  batch    BatchSampler: R independent runs of uneven sizes advanced together
  fsv      FSVFilter: particle filter of the factor stochastic-volatility model
  loglik   one smc_loglik call
  weights  smc_reweight then smc_resample under the ESS test, as a program that
           composes a tempering step from the single calls does
"""

import math
import random
import types

import numpy as np
import torch

import paper_0905_2441_amd as smc
from paper_0905_2441_amd import samplers

MEANS_1D = (-3.0, 0.0, 3.0, 6.0)
TERM_FLOPS = 3                      # one exponential, its sum and its share of the log

# The factor model of the paper's particle filter.
FSV = types.SimpleNamespace(
    B=((1.0, 0.0, 0.0), (0.5, 1.0, 0.0), (0.5, 0.5, 1.0), (0.2, 0.6, 0.3), (0.8, 0.7, 0.5)),
    psi=(0.5,) * 5, phi=(0.9,) * 3,
    U=((0.5, 0.2, 0.1), (0.2, 0.5, 0.2), (0.1, 0.2, 0.5)))


def listed():
    return [
        # the plain FP64 sampler on the paper's data size: every launch is tiny
        dict(name="smc_small_fp64", kind="smc", k=4, d=1, n=100, N=1024, prec="fp64", T=50,
             steps=50, group=10, moves=1, prior="gauss", sd=0.5, scheme="systematic"),
        # the headline workload, the whole run of 100 tempering steps
        dict(name="smc_run_fp32", kind="smc", k=4, d=1, n=1000, N=131072, prec="fp32", T=100,
             steps=100, group=10, moves=1, prior="gauss", sd=0.5, scheme="systematic"),
        # the same workload in FP64, its first 20 steps
        dict(name="smc_run_fp64", kind="smc", k=4, d=1, n=1000, N=131072, prec="fp64", T=100,
             steps=20, group=20, moves=1, prior="gauss", sd=0.5, scheme="systematic"),
        # the paper's own sampler settings: box prior, ten unit moves per step
        dict(name="smc_paper_fp32", kind="smc", k=4, d=1, n=100, N=8192, prec="fp32", T=200,
             steps=40, group=20, moves=10, prior="box", sd=1.0, scheme="systematic"),
        # eight components in eight dimensions on the matrix cores
        dict(name="smc_d8_bf16x3", kind="smc", k=8, d=8, n=65536, N=16384, prec="bf16x3", T=100,
             steps=5, group=5, moves=1, prior="gauss", sd=0.5, scheme="systematic"),
        # the same model's FP64 likelihood of a population that has found the modes
        dict(name="loglik_d8_fp64", kind="loglik", k=8, d=8, n=65536, N=16384, prec="fp64",
             start="near"),
        # the likelihood of a million prior draws
        dict(name="loglik_prior_fp32", kind="loglik", k=4, d=1, n=4096, N=1048576, prec="fp32",
             start="prior"),
        # population MCMC with many chains and long data
        dict(name="pt_large_fp32", kind="pt", k=4, n=10000, M=8192, prec="fp32", steps=20,
             group=20, prior="gauss", sd=0.5, parity=0, wrap=False),
        # the paper's population MCMC with few chains
        dict(name="pt_small_fp32", kind="pt", k=4, n=100, M=32, prec="fp32", steps=256,
             group=64, prior="box", sd=1.0, parity=1, wrap=True),
        # a batch of 64 runs of very uneven sizes
        dict(name="batch_fp32", kind="batch", k=4, R=64, n_lo=100, n_hi=100000, N_lo=1024,
             N_hi=65536, plan=5000, prec="fp32", steps=3, moves=1),
        # a reweight and a resampling of a million particles
        dict(name="weights_systematic", kind="weights", N=1048576, kd=4, scheme="systematic",
             spread=1.2),
        # a quarter of the paper's particle filter run
        dict(name="fsv_filter", kind="fsv", N=8192, steps=50, group=50, scheme="systematic"),
    ]


def _log_int(rng, lo, hi):
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return min(hi, max(lo, v))


def draw(rng):
    kind = rng.choice(("smc", "smc", "smc", "smc", "loglik", "loglik", "loglik", "pt", "pt",
                       "batch", "weights", "weights", "fsv"))
    if kind in ("smc", "loglik") and rng.random() < 0.3:
        # eight dimensions: the matrix form and FP64
        k = rng.choice((2, 4, 8))
        prec = rng.choice(("bf16x3", "fp64"))
        N = _log_int(rng, 500, 16384)
        n = _log_int(rng, 1000, min(65536, (1 << 33) // (N * k)))
        if kind == "loglik":
            return dict(kind=kind, k=k, d=8, n=n, N=N, prec=prec, start=rng.choice(("near", "prior")))
        return dict(kind=kind, k=k, d=8, n=min(n, 16384), N=N, prec=prec, T=100,
                    steps=rng.randint(2, 5), group=5, moves=1, prior="gauss", sd=0.5,
                    scheme="systematic")
    if kind == "smc":
        prec = rng.choice(("fp32", "fp64"))
        N = _log_int(rng, 200, 262144)
        n = _log_int(rng, 50, min(10000, (1 << 27) // N))
        paper = rng.random() < 0.25
        steps = rng.randint(10, 50)
        while steps > 10 and N * n * steps * (10 if paper else 1) > (1 << 32):
            steps -= 1
        return dict(kind=kind, k=rng.choice((2, 3, 4, 4, 4, 8)), d=1, n=n, N=N, prec=prec, T=100,
                    steps=steps, group=10, moves=10 if paper else 1,
                    prior="box" if paper else "gauss", sd=1.0 if paper else 0.5,
                    scheme=rng.choice(("systematic", "systematic", "stratified", "multinomial")))
    if kind == "loglik":
        prec = rng.choice(("fp32", "fp64"))
        N = _log_int(rng, 100, 1048576)
        n = _log_int(rng, 50, min(65536, (1 << 31) // N))
        return dict(kind=kind, k=rng.choice((1, 2, 4, 4, 4, 8)), d=1, n=n, N=N, prec=prec,
                    start=rng.choice(("near", "prior")))
    if kind == "pt":
        M = _log_int(rng, 8, 16384)
        n = _log_int(rng, 100, 10000)
        return dict(kind=kind, k=4, n=n, M=M, prec=rng.choice(("fp32", "fp32", "fp64")),
                    steps=rng.randint(20, 64), group=rng.choice((10, 20, 64)),
                    prior=rng.choice(("gauss", "box")), sd=0.5, parity=rng.randint(0, 1),
                    wrap=rng.random() < 0.5)
    if kind == "batch":
        n_hi = _log_int(rng, 1000, 50000)
        return dict(kind=kind, k=4, R=rng.randint(4, 64), n_lo=100, n_hi=n_hi, N_lo=1024,
                    N_hi=rng.choice((4096, 16384, 65536)), plan=rng.randint(0, 1 << 20),
                    prec=rng.choice(("fp32", "fp32", "fp64")), steps=rng.randint(2, 4),
                    moves=rng.choice((1, 1, 2)))
    if kind == "weights":
        return dict(kind=kind, N=_log_int(rng, 1000, 1 << 24), kd=rng.choice((2, 4, 8)),
                    scheme=rng.choice(("systematic", "systematic", "stratified", "multinomial")),
                    spread=rng.choice((0.5, 1.2, 3.0)))
    return dict(kind="fsv", N=_log_int(rng, 1000, 1 << 20), steps=rng.randint(20, 60), group=20,
                scheme=rng.choice(("systematic", "stratified", "multinomial")))


# ---------------------------------------------------------------- inputs

_STREAM = []


def _stream():
    # one side stream for every state, as a program with one sampler at a time has
    if not _STREAM:
        _STREAM.append(torch.cuda.Stream())
    return _STREAM[0]


def _rng(seed, salt=0):
    return np.random.Generator(np.random.PCG64([int(seed), int(salt)]))


def _means(k, d, seed):
    if d > 1:
        return 3.0 * _rng(seed, 7).standard_normal((k, d))
    if k == 4:
        return np.asarray(MEANS_1D).reshape(4, 1)
    return (-3.0 + 3.0 * np.arange(k, dtype=np.float64)).reshape(k, 1)


def _data(n, mu, sigma2, seed):
    g = _rng(seed, 1)
    z = g.integers(0, mu.shape[0], size=n)
    y = mu[z] + math.sqrt(sigma2) * g.standard_normal((n, mu.shape[1]))
    y = y.astype(np.float32)
    return y.reshape(n) if mu.shape[1] == 1 else y


def _sigma2(case):
    if case.get("d", 1) > 1:
        return 1.0
    return 0.55 ** 2 if case.get("prior") == "box" else 0.55


def _model(case):
    kw = dict(prior="box", prior_a=-10.0, prior_b=10.0) if case.get("prior") == "box" else {}
    return smc.Gmm.equal_weights(case["k"], case.get("d", 1), _sigma2(case), **kw)


def _quadratic(T):
    b = (np.arange(T + 1, dtype=np.float64) / T) ** 2
    b[-1] = 1.0
    return b


def _ladder(M):
    return (np.arange(1, M + 1, dtype=np.float64) / M) ** 4


def _theta(case, mu, seed):
    """[k*d, N] FP64 on the GPU: prior draws, or near a mode (a relabelling of the
    means plus N(0, 0.1^2))."""
    k, d, N = case["k"], case["d"], case["N"]
    g = torch.Generator(device="cuda").manual_seed(int(seed) + 17)
    if case["start"] == "prior":
        return 10.0 * torch.randn((k * d, N), generator=g, device="cuda", dtype=torch.float64)
    order = torch.rand((N, k), generator=g, device="cuda").argsort(dim=1)
    th = torch.as_tensor(mu, device="cuda", dtype=torch.float64)[order]      # [N, k, d]
    th = th.reshape(N, k * d).t().contiguous()
    return th + 0.1 * torch.randn(th.shape, generator=g, device="cuda", dtype=torch.float64)


def _batch_sizes(case):
    r = random.Random(case["plan"])
    Ns = [v for v in (1024, 4096, 16384, 65536) if case["N_lo"] <= v <= case["N_hi"]]
    return [(_log_int(r, case["n_lo"], case["n_hi"]), r.choice(Ns)) for _ in range(case["R"])]


def _fsv_data(steps, seed):
    g = _rng(seed, 3)
    B, L = np.asarray(FSV.B), np.linalg.cholesky(np.asarray(FSV.U))
    phi, psi = np.asarray(FSV.phi), np.asarray(FSV.psi)
    x, y = np.zeros(3), np.zeros((steps, 5))
    for t in range(steps):
        x = phi * x + L @ g.standard_normal(3)
        y[t] = B @ (np.exp(0.5 * x) * g.standard_normal(3)) + np.sqrt(psi) * g.standard_normal(5)
    return y


def _weights_inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(int(seed) + 29)

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda", dtype=torch.float64)

    N = case["N"]
    # log-likelihoods about -2000 and the tempering increment that gives their
    # reweight the wanted spread
    return dict(logw=0.3 * normal(N), l=-2000.0 + 10.0 * case["spread"] * normal(N),
                theta=3.0 * normal(case["kd"], N), dbeta=0.1)


def prepare(case, seed):
    kind, seed = case["kind"], int(seed)
    ctx = smc.Context(0)
    st = types.SimpleNamespace(case=case, ctx=ctx)
    if kind in ("smc", "pt"):
        d = case.get("d", 1)
        mu = _means(case["k"], d, seed)
        y = _data(case["n"], mu, _sigma2(case), seed)
        if kind == "smc":
            st.s = samplers.SMCSampler(ctx, _model(case), y, case["N"], _quadratic(case["T"]),
                                       case["sd"], case["moves"], seed + 101, prec=case["prec"],
                                       stream=_stream(), scheme=case["scheme"])
        else:
            st.s = samplers.PTSampler(ctx, _model(case), y, _ladder(case["M"]), case["sd"],
                                      seed + 103, parity_mode=case["parity"], wrap=case["wrap"],
                                      prec=case["prec"], stream=_stream())
    elif kind == "batch":
        sizes = _batch_sizes(case)
        datas = [_data(n, _rng(seed, 1000 + r).uniform(-6.0, 9.0, (case["k"], 1)), 0.55,
                       1000 * seed + r)
                 for r, (n, _) in enumerate(sizes)]
        st.s = samplers.BatchSampler(ctx, _model(case), datas, [N for _, N in sizes],
                                     [5000 + 1000 * seed + r for r in range(case["R"])],
                                     _quadratic(100), 0.5, case["moves"], prec=case["prec"],
                                     stream=_stream())
    elif kind == "fsv":
        st.s = samplers.FSVFilter(ctx, FSV, _fsv_data(case["steps"], seed), case["N"], seed + 7,
                                  stream=_stream(), scheme=case["scheme"])
    elif kind == "loglik":
        mu = _means(case["k"], case["d"], seed)
        st.model = _model(case)
        st.y = torch.as_tensor(_data(case["n"], mu, _sigma2(case), seed)).cuda()
        if case["d"] == 1:
            smc.smc_sort_data(st.y)
        st.theta = _theta(case, mu, seed)
        st.out = torch.empty(case["N"], device="cuda", dtype=torch.float64)
        ctx.reserve(case["N"], st.model.kd, case["n"] if case["prec"] == "bf16x3" else 0)
    else:
        N = case["N"]
        x = _weights_inputs(case, seed)
        st.logw, st.l, st.theta, st.dbeta = x["logw"], x["l"], x["theta"], x["dbeta"]
        st.W = torch.empty_like(st.logw)
        st.logZ = torch.zeros(1, device="cuda", dtype=torch.float64)
        st.ess = torch.zeros(1, device="cuda", dtype=torch.float64)
        st.idx = torch.empty(N, device="cuda", dtype=torch.int32)
        st.theta_out, st.l_out = torch.empty_like(st.theta), torch.empty_like(st.l)
        st.seed = seed + 11
        ctx.reserve(N, case["kd"])
    torch.cuda.synchronize()
    return st


def run(st):
    case = st.case
    kind = case["kind"]
    if kind == "smc":
        s = st.s
        s.init()
        s.advance(case["steps"], graph=True, steps_per_graph=case["group"])
        return dict(theta=s.theta, l=s.loglik, logw=s.logw, W=s.W, stats=s.stats,
                    n_accept=s.n_accept, t=s.t)
    if kind == "pt":
        s = st.s
        s.init()
        s.advance(case["steps"], graph=True, iters_per_graph=case["group"])
        return dict(theta=s.theta, l=s.loglik, n_accept=s.n_accept, n_swap=s.n_swap, it=s.it)
    if kind == "batch":
        s = st.s
        s.init()
        for _ in range(case["steps"]):
            s.capture().launch()
        return dict(theta=s.theta, l=s.loglik, logw=s.logw, W=s.W, stats=s.stats,
                    n_accept=s.n_accept, t=s.t)
    if kind == "fsv":
        s = st.s
        s.init()
        s.advance(case["steps"], graph=True, steps_per_graph=case["group"])
        return dict(x=s.x, logw=s.logw, stats=s.stats, moments=s.moments, t=s.t)
    if kind == "loglik":
        return smc.smc_loglik(st.ctx, st.model, st.y, st.theta, case["prec"], out=st.out)
    smc.smc_reweight(st.ctx, st.logw, st.l, st.dbeta, W=st.W, logZ=st.logZ, ess=st.ess)
    smc.smc_resample(st.ctx, st.W, case["scheme"], st.seed, 3, ess=st.ess,
                     ess_threshold=0.5 * case["N"], idx=st.idx, theta_in=st.theta,
                     theta_out=st.theta_out, l_in=st.l, l_out=st.l_out, logw=st.logw)
    return dict(W=st.W, logZ=st.logZ, ess=st.ess, idx=st.idx, theta=st.theta_out, l=st.l_out,
                logw=st.logw)


# ---------------------------------------------------------------- what a pass needs

def _likelihood_flops(n, N, k, d):
    # per datum, particle and component: d multiply-adds and one exponential's share
    return float(n) * N * k * (2 * d + TERM_FLOPS)


def _population_bytes(N, kd):
    # theta, l and logw of every particle, read and written
    return 2.0 * 8 * N * (kd + 2)


def work(case):
    kind = case["kind"]
    if kind == "loglik":
        kd = case["k"] * case["d"]
        return dict(bytes=8.0 * case["N"] * (kd + 1) + 4.0 * case["n"] * case["d"],
                    flops=_likelihood_flops(case["n"], case["N"], case["k"], case["d"]))
    if kind == "smc":
        kd, evals = case["k"] * case["d"], 1 + case["steps"] * case["moves"]
        return dict(bytes=(1 + case["steps"]) * _population_bytes(case["N"], kd),
                    flops=evals * _likelihood_flops(case["n"], case["N"], case["k"], case["d"]))
    if kind == "pt":
        return dict(bytes=(1 + case["steps"]) * _population_bytes(case["M"], case["k"]),
                    flops=(1 + case["steps"]) * _likelihood_flops(case["n"], case["M"], case["k"], 1))
    if kind == "batch":
        sizes = _batch_sizes(case)
        return dict(bytes=(1 + case["steps"]) * sum(_population_bytes(N, case["k"]) for _, N in sizes),
                    flops=(1 + case["steps"] * case["moves"]) *
                    sum(_likelihood_flops(n, N, case["k"], 1) for n, N in sizes))
    if kind == "fsv":
        # read x and logw, write x and logw; about 300 operations of the 5 x 5
        # Cholesky, its solve and the propagation
        return dict(bytes=64.0 * case["N"] * case["steps"], flops=300.0 * case["N"] * case["steps"])
    # reweight: read l and logw, write logw and W; resampling: read W, write idx,
    # gather theta and l, reset logw
    return dict(bytes=case["N"] * (40.0 + 36.0 + 16.0 * case["kd"]), flops=20.0 * case["N"])


# ---------------------------------------------------------------- 64-bit values

def exact(case, seed):
    if case["kind"] == "weights":
        x = _weights_inputs(case, int(seed))
        N = case["N"]
        lw = x["logw"] + x["dbeta"] * x["l"]
        e = torch.exp(lw - lw.max())
        W = e / e.sum()
        logZ = torch.logsumexp(lw, 0) - torch.logsumexp(x["logw"], 0)
        ess = 1.0 / (W * W).sum()
        fires = bool(ess < 0.5 * N)
        return dict(W=W, logZ=logZ.reshape(1), ess=ess.reshape(1), idx=None, theta=None, l=None,
                    logw=torch.zeros_like(lw) if fires else lw)
    if case["kind"] != "loglik":
        return None              # a random walk: its decisions have no 64-bit value
    k, d, N = case["k"], case["d"], case["N"]
    mu = _means(k, d, int(seed))
    y = torch.as_tensor(_data(case["n"], mu, _sigma2(case), int(seed))).cuda().double()
    y = y.reshape(case["n"], d)
    th = _theta(case, mu, int(seed)).reshape(k, d, N)
    s2 = _sigma2(case)
    out = torch.zeros(N, device="cuda", dtype=torch.float64)
    rows = max(1, (1 << 26) // (k * N))
    for j in range(0, case["n"], rows):
        yc = y[j:j + rows]
        q = torch.zeros((yc.shape[0], k, N), device="cuda", dtype=torch.float64)
        for c in range(d):
            q += (yc[:, c, None, None] - th[None, :, c, :]) ** 2
        out += torch.logsumexp(q.mul_(-0.5 / s2), dim=1).sum(0)
    return out + case["n"] * (math.log(1.0 / k) - 0.5 * d * math.log(2.0 * math.pi * s2))
