"""Timed cases of the library, through its Python binding.

Each case is one call sequence that a program using the library makes: batch evaluation of a
target and its gradient (BF16, FP16, FP32 and FP64 GEMMs, both point layouts, with and without
gradients, the plain spectrum model), the weight gradients of a fit through the emulator, the
production steps of every sampler, a burn-in window, an epoch of emulator training, the
effective sample size of a record and the convergence metrics.  The networks, dimensions and
chain counts are those of workloads/synth.py and of the sweep, comparison and benchmark
programs; inputs are made here from the seed.

  listed()            the cases
  draw(rng)           one more case of the same ranges
  prepare(case, seed) contexts, inputs and buffers on the GPU
  run(state)          one pass
  work(case)          bytes and operations that a pass cannot do without
  exact(case, seed)   the pass's outputs in FP64 with plain torch / numpy
"""
import math

import numpy as np
import torch

import paper_2606_04895_amd as B

# d, hidden width, hidden layers, twisted pair
NETS = {
    "c1": (6, 128, 2, False),
    "c2": (6, 512, 4, False),
    "c3": (12, 1024, 4, True),
    "c5": (27, 1024, 5, False),
}
N_BINS, N_TERMS = 2500, 8  # spectrum of the plain model
CREDIBLE_LEVEL, N_PROJ, PROJ_SEED = 0.68, 500, 0x5EED
# relative rate of one evaluation against BF16 (caps the size of drawn cases)
RATE = {"bf16": 2e14, "fp16": 2e14, "fp32": 8e13, "fp64": 1.5e13}


def net(name):
    d, width, nh, twist = NETS[name]
    return dict(d=d, width=width, n_hidden=nh, twist=twist)


def listed():
    return [
        # one small batch: an interactive log-likelihood call, latency only
        dict(name="eval_bf16_c2_64", kind="eval", prec="bf16", n=64, chains=64, grad=True,
             aos=False, penalty=False, **net("c2")),
        # a large point set in the [n][d] layout of torch programs, on the 27-parameter network
        dict(name="eval_bf16_c5_65537_aos", kind="eval", prec="bf16", n=65537, chains=64,
             grad=True, aos=True, penalty=False, **net("c5")),
        # training data of the learned emulator: plain-model log-likelihoods of a design
        dict(name="plain_c4_20000", kind="plain", prec="fp32", n=20000, chains=16, grad=False,
             **net("c2")),
        # value, input gradient and weight gradients of one batch (differentiating through the
        # emulator), ragged batch, FP16 GEMMs
        dict(name="vjp_fp16_c2_4099", kind="vjp", prec="fp16", n=4099, chains=4096, **net("c2")),
        # the benchmark's production run: HMC, ten leapfrog steps, every step recorded
        dict(name="hmc_bf16_c2_4096", kind="step", sampler="hmc", prec="bf16", chains=4096,
             steps=20, thin=1, eps=0.99, **net("c2")),
        # a burn-in window: dual averaging after every step, then the covariance update
        dict(name="burnin_mala_fp32_c2_4096", kind="burnin", sampler="mala", prec="fp32",
             chains=4096, steps=40, **net("c2")),
        # the sampler with the highest min-ESS/s on the 27-parameter network
        dict(name="nuts_bf16_c5_16384", kind="step", sampler="nuts", prec="bf16", chains=16384,
             steps=4, thin=1, eps=0.73, **net("c5")),
        # the stretch move (log-likelihood only, two launches per step)
        dict(name="aies_fp16_c3_16384", kind="step", sampler="aies", prec="fp16", chains=16384,
             steps=10, thin=2, eps=0.0, **net("c3")),
        # the small FP64 configuration: random-walk Metropolis with 64 chains
        dict(name="mh_fp64_c1_64", kind="step", sampler="mh", prec="fp64", chains=64, steps=200,
             thin=1, eps=0.0, **net("c1")),
        # an epoch of emulator training (ragged tail dropped), with the weights at its end
        dict(name="train_fp32_c4_1024", kind="train", prec="fp32", batch=1024, n=65573,
             **net("c2")),
        # effective sample size of the benchmark's production record
        dict(name="ess_c2_4000x4096", kind="ess", T=4000, chains=4096, d=6, rho=0.47, spread=0.0),
        # R - 1, credible limits and the sliced Wasserstein distance of a 27-parameter record
        dict(name="metrics_c5_256x4096", kind="metrics", T=256, chains=4096, d=27, rho=0.3,
             spread=0.05, tail=8),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_net(rng):
    if rng.random() < 0.5:
        return net(rng.choice(sorted(NETS)))
    d = rng.randint(1, 32)
    return dict(d=d, width=rng.choice([128, 128, 256, 512, 512, 1024]),
                n_hidden=rng.randint(1, 5), twist=d >= 4 and rng.random() < 0.25)


def _eval_flops(c, grad):
    d, w, nh = c["d"], c["width"], c["n_hidden"]
    return 2.0 * (d * w + (nh - 1) * w * w + w) * (2 if grad else 1)


def draw(rng):
    """A case of the listed kinds at other sizes, shapes, types and options."""
    kind = rng.choice(["eval", "eval", "eval", "step", "step", "step", "step", "burnin", "vjp",
                       "train", "ess", "metrics", "plain"])
    prec = rng.choice(["bf16", "bf16", "fp16", "fp32", "fp32", "fp64"])
    if kind in ("burnin", "vjp", "train") and prec == "fp64":
        prec = "fp32"
    c = dict(kind=kind, prec=prec, **_draw_net(rng))
    if prec == "fp64":
        c["width"] = min(c["width"], 512)  # the widest layers an FP64 tile holds
    budget = 0.004  # seconds of emulator work at the RATE of the precision
    per = _eval_flops(c, True) / RATE[prec]
    if kind == "eval":
        c.update(n=max(1, min(_log_int(rng, 1, 70000), int(budget / per))),
                 chains=rng.choice([16, 64, 1000, 4096]), grad=rng.random() < 0.75,
                 aos=rng.random() < 0.4, penalty=rng.random() < 0.2)
    elif kind == "vjp":
        c.update(n=max(1, min(_log_int(rng, 16, 20000), int(budget / (1.5 * per)))),
                 chains=rng.choice([16, 4096]))
    elif kind == "plain":
        c.update(net("c2"), n=_log_int(rng, 1, 20000), chains=16, grad=rng.random() < 0.4)
        if c["grad"]:
            c["n"] = max(1, c["n"] // 2)
    elif kind in ("step", "burnin"):
        s = rng.choice(["mala", "hmc", "nuts", "aies", "de", "mh"]) if kind == "step" else \
            rng.choice(["mala", "hmc"])
        if prec == "fp64" and s in ("mala", "hmc", "nuts"):
            s = "mh"
        chains = 2 * max(2, min(_log_int(rng, 8, 16384), int(budget / per) // 10))
        if s not in ("aies", "de") and rng.random() < 0.5:
            chains -= 1
        evals = {"hmc": 10, "nuts": 8}.get(s, 1)
        wide = max(chains, 2048)  # fewer chains leave the chip idle
        steps = max(1, min(60, int(budget / (per * evals * wide))))
        if kind == "burnin":
            steps = max(4, steps)
        eps = {"mala": 0.6, "hmc": 0.8, "nuts": 0.7}.get(s, 0.0) / c["d"] ** 0.125
        c.update(sampler=s, chains=chains, steps=steps, eps=eps)
        if kind == "step":
            c["thin"] = rng.choice([1, 1, 1, 2, 3])
    elif kind == "train":
        c["batch"] = 16 * max(1, min(_log_int(rng, 1, 128), int(budget / (24 * per))))
        c["n"] = c["batch"] * rng.randint(2, 24) + rng.randint(0, 15)
    elif kind == "ess":
        chains, T = _log_int(rng, 1, 16384), _log_int(rng, 4, 4000)
        # chain means that differ (spread) keep the autocorrelations above zero, so every lag
        # of the window enters, as in a record shorter than its autocorrelation
        c = dict(kind=kind, d=c["d"], chains=chains, T=T,
                 rho=rng.choice([-0.3, 0.0, 0.47, 0.8, 0.95]),
                 spread=rng.choice([0.0, 0.0, 0.0, 0.05]))
        c["T"] = max(4, min(T, 6 * 4096 * 4000 // (6 * c["d"] * chains),
                            600 if c["spread"] else 4000))
    else:
        chains = _log_int(rng, 16, 4096)
        c = dict(kind=kind, d=c["d"], chains=chains, rho=rng.choice([0.0, 0.3, 0.8]),
                 spread=rng.choice([0.0, 0.05]), tail=rng.randint(1, 8))
        c["T"] = max(c["tail"], 2, min(_log_int(rng, 8, 1000),
                                       27 * 4096 * 256 // (4 * c["d"] * chains)))
    return c


# ---- problems ----------------------------------------------------------------------------
def _nparams(c):
    d, w, nh = c["d"], c["width"], c["n_hidden"]
    return w * d + w + (nh - 1) * (w * w + w) + w + 1


def _xavier(rng, c):
    d, w, nh = c["d"], c["width"], c["n_hidden"]
    parts, fan = [], d
    for _ in range(nh):
        parts += [rng.standard_normal(w * fan) * math.sqrt(2.0 / (w + fan)),
                  rng.standard_normal(w) * 0.02]
        fan = w
    parts += [rng.standard_normal(w) * math.sqrt(2.0 / (w + 1)), rng.standard_normal(1) * 0.02]
    return np.concatenate(parts)


def _problem(c, rng, params=True):
    """Gaussian part of condition number 1e3 (the last pair twisted if asked for) plus half
    the emulator, in a box of +-10 marginal standard deviations."""
    d = c["d"]
    mu = rng.standard_normal(d)
    q, r = np.linalg.qr(rng.standard_normal((d, d)))
    q = q * np.sign(np.diag(r))
    lam = 1e3 ** (np.arange(d) / max(d - 1, 1))
    cov = (q * lam) @ q.T
    twist = None
    if c.get("twist"):
        u, v, su, sw = d - 2, d - 1, 0.8, 0.3
        beta = 10.0 * sw / su ** 2
        cov[[u, v], :] = 0.0
        cov[:, [u, v]] = 0.0
        cov[u, u], cov[v, v] = su ** 2, sw ** 2
        twist = dict(u=u, v=v, beta=beta, center=float(mu[u]), kappa=su ** 2)
    prec = np.linalg.inv(cov)
    prec = 0.5 * (prec + prec.T)
    var = np.diag(cov).copy()
    if twist:
        var[v] += 2.0 * beta ** 2 * su ** 4
    sd = np.sqrt(var)
    return dict(d=d, lower=mu - 10 * sd, upper=mu + 10 * sd, gauss_coef=1.0, gauss_mean=mu,
                gauss_prec=prec, gauss_cov=cov, sd=sd, twist=twist, width=c["width"],
                n_hidden=c["n_hidden"], mlp_params=_xavier(rng, c) if params else None,
                in_center=mu, in_invscale=1.0 / sd, mlp_coef=0.5, offset=0.0, plain_mode=0,
                box_penalty=1 if c.get("penalty") else 0, penalty_width=0.05)


def _points(p, rng, n, outside=0.0):
    """[d][n] draws of the target's Gaussian part (untwisted); a share of them far out."""
    ch = np.linalg.cholesky(p["gauss_cov"])
    y = p["gauss_mean"][:, None] + ch @ rng.standard_normal((p["d"], n))
    t = p["twist"]
    if t:
        y[t["v"]] -= t["beta"] * ((y[t["u"]] - t["center"]) ** 2 - t["kappa"])
    if outside:
        far = rng.random(n) < outside
        far[0] = False
        y[0, far] += 9.0 * p["sd"][0]
    return y


def _plain_problem(c, rng):
    """Spectrum of damped cosines against seeded noisy data."""
    d, nt = c["d"], N_TERMS
    center, w = rng.standard_normal(d), rng.uniform(0.5, 2.0, d)
    xg = np.arange(N_BINS) / (N_BINS - 1.0)
    m = np.arange(1, nt + 1, dtype=np.float64)
    a, g, ph = (rng.normal(0.0, 0.3, (nt, d)) for _ in range(3))
    star = rng.uniform(-0.5, 0.5, d)
    sigma = 0.05 * (1.0 + xg)
    s = (np.exp(a @ star)[:, None] * np.exp(-(0.5 * m * np.exp(g @ star))[:, None] * xg)
         * np.cos(6.0 * math.pi * m[:, None] * xg + math.pi * np.tanh(ph @ star)[:, None])).sum(0)
    plain = dict(n_bins=N_BINS, n_terms=nt, xgrid=xg, data=s + sigma * rng.standard_normal(N_BINS),
                 inv_sigma2=sigma ** -2, a=a, g=g, p=ph, k=3.0 * m, gamma0=0.5 * m,
                 center=center, invscale=1.0 / w)
    return dict(d=d, lower=center - w, upper=center + w, width=c["width"],
                n_hidden=c["n_hidden"], plain_mode=2, plain=plain,
                box=(center + w * (star - 0.1), center + w * (star + 0.1)))


def _gpu(a, dtype=torch.float64):
    return torch.tensor(np.ascontiguousarray(a), dtype=dtype, device="cuda")


def _inputs(c, seed):
    """The problem and host inputs of a case, from the seed alone."""
    rng = np.random.default_rng([seed, 0xCA5E])
    kind = c["kind"]
    if kind == "plain":
        p = _plain_problem(c, rng)
        lo, hi = p["box"]
        return p, lo[:, None] + (hi - lo)[:, None] * rng.random((c["d"], c["n"]))
    if kind == "train":
        # standardised targets of a smooth function over the unit box
        t = rng.uniform(-1.0, 1.0, (c["n"], c["d"]))
        w = rng.standard_normal(c["d"]) / math.sqrt(c["d"])
        y = np.sin(2.0 * t @ w) - (t @ np.roll(w, 1)) ** 2
        y = (y - y.mean()) / y.std()
        return _xavier(rng, c), t.astype(np.float32), y.astype(np.float32), \
            rng.permutation(c["n"]).astype(np.int32)
    p = _problem(c, rng)
    if kind == "eval":
        return p, _points(p, rng, c["n"], outside=0.05)
    if kind == "vjp":
        return p, _points(p, rng, c["n"]), rng.standard_normal(c["n"])
    return p, _points(p, rng, c["chains"])  # step, burnin


def _record(c, seed, T, shift=0.0):
    """[T][d][chains] stationary AR(1) chains with correlated components."""
    g = torch.Generator(device="cuda").manual_seed(seed * 7919 + 11)
    d, n, rho = c["d"], c["chains"], c["rho"]
    mix = torch.tril(torch.randn(d, d, generator=g, device="cuda") * 0.3) + torch.eye(d, device="cuda")
    e = torch.randn(T, d, n, generator=g, device="cuda")
    for t in range(1, T):
        e[t].mul_(math.sqrt(1.0 - rho * rho)).add_(e[t - 1], alpha=rho)
    if c["spread"]:  # chains that are not quite at the same mean, as after a short burn-in
        e += c["spread"] * torch.randn(1, d, n, generator=g, device="cuda")
    for t0 in range(0, T, 256):
        e[t0:t0 + 256] = torch.matmul(mix, e[t0:t0 + 256]) + shift
    return e, mix


def _records(c, seed):
    if c["kind"] == "ess":
        return _record(c, seed, c["T"])[0]
    rec, mix = _record(c, seed, c["T"])
    ref = _record(c, seed + 1000003, c["tail"], shift=0.1)[0]
    mu = rec.double().mean(dim=(0, 2)).cpu().numpy()
    L = mix.double().cpu().numpy()
    L = np.linalg.cholesky(L @ L.T + 1e-3 * np.eye(c["d"]))
    return rec, ref, mu, L


def _metrics_ctx(c):
    """A context of the record's dimension and chain count (a small network)."""
    cc = dict(d=c["d"], width=128, n_hidden=1)
    return B.best_init(_problem(cc, np.random.default_rng(1)), n_chains=c["chains"],
                       precision="fp32", seed=1)


def prepare(case, seed):
    c, kind = dict(case), case["kind"]
    s = dict(c=c)
    if kind in ("ess", "metrics"):
        r = _records(c, seed)
        s["ctx"] = _metrics_ctx(c)
        if kind == "ess":
            s["rec"] = r
        else:
            s["rec"], s["ref"], s["mu"], s["L"] = r
            s["tail"] = s["rec"][-c["tail"]:].contiguous()
        return s
    if kind == "train":
        params, t, y, perm = _inputs(c, seed)
        s.update(tr=B.Trainer(c["d"], c["width"], c["n_hidden"], params, precision=c["prec"]),
                 t=_gpu(t, torch.float32), y=_gpu(y, torch.float32), perm=_gpu(perm, torch.int32))
        return s
    got = _inputs(c, seed)
    p = got[0]
    s["ctx"] = ctx = B.best_init(p, n_chains=c["chains"], precision=c["prec"], seed=seed)
    if kind in ("eval", "plain", "vjp"):
        x = got[1].T if c.get("aos") else got[1]
        s["x"] = _gpu(x)
        if kind == "vjp":
            s["up"] = _gpu(got[2])
        return s
    # samplers: chains at the posterior, whitened with its covariance
    B.best_set_whitening(ctx, p["gauss_mean"], np.linalg.cholesky(
        p["gauss_cov"] if not p["twist"] else np.diag(p["sd"] ** 2)))
    B.best_set_state(ctx, got[1])
    cap = c["steps"] // c.get("thin", 1)
    s["rec"] = torch.zeros((max(cap, 1), c["d"], c["chains"]), dtype=torch.float32, device="cuda")
    if kind == "burnin":
        B.best_set_step_size(ctx, {"mala": 0.5, "hmc": 0.3}[c["sampler"]])
    return s


COUNTS = ("accepted", "evals", "n_nonfinite", "n_oob", "n_recorded", "sum_accept_prob", "eps")


def run(state):
    s, c = state, state["c"]
    kind = c["kind"]
    if kind in ("eval", "plain"):
        lp, g = B.best_logL_grad(s["ctx"], s["x"], want_grad=c["grad"], aos=c.get("aos", False))
        return {"logL": lp} if g is None else {"logL": lp, "grad": g}
    if kind == "vjp":
        lp, g = B.best_logL_grad(s["ctx"], s["x"])
        return {"logL": lp, "grad": g, "params": B.best_logL_param_grad(s["ctx"], s["x"], s["up"])}
    if kind == "step":
        st = B.best_step(s["ctx"], c["sampler"], c["steps"], eps=c["eps"], n_leapfrog=10,
                         mh_scale=2.4 / math.sqrt(c["d"]), thin=c["thin"], record=s["rec"],
                         max_depth=8)
        return {"record": s["rec"], **{k: st[k] for k in COUNTS}}
    if kind == "burnin":
        target = {"mala": 0.57, "hmc": 0.8}[c["sampler"]]
        st = B.best_step(s["ctx"], c["sampler"], c["steps"], record=s["rec"], adapt_eps=True,
                         target_accept=target)
        info = B.best_adapt(s["ctx"], samples=s["rec"][c["steps"] // 2:].contiguous(),
                            finalize_da=True, reset_da=True, target_accept=target)
        mu, L = B.best_get_whitening(s["ctx"])
        return {"record": s["rec"], "mu": mu, "L": L, "eps_new": info["eps"],
                **{k: st[k] for k in COUNTS}}
    if kind == "train":
        nb = c["n"] // c["batch"]
        loss = s["tr"].epoch(s["t"], s["y"], s["perm"], c["batch"], 1e-3, 1e-4, 0, nb)
        return {"loss": loss, "params": s["tr"].params()}
    if kind == "ess":
        e, flags = B.best_ess(s["ctx"], s["rec"], flags=True)
        return {"ess": e, "flags": flags}
    lo, hi, _ = B.best_credible(s["ctx"], s["rec"], CREDIBLE_LEVEL, whitening=(s["mu"], s["L"]))
    return {"rminus1": B.best_rhat(s["ctx"], s["rec"]), "lo": lo, "hi": hi,
            "sliced_w": B.best_sliced_wasserstein(s["ctx"], s["tail"], s["ref"], N_PROJ, PROJ_SEED,
                                                  whitening=(s["mu"], s["L"]))}


def work(case):
    """Inputs and weights read once, outputs written once; two operations per multiply-add of
    the layers, and one pass over the data for the statistics of a record."""
    c, kind = case, case["kind"]
    size = {"bf16": 2, "fp16": 2, "fp32": 4, "fp64": 8}.get(c.get("prec"), 8)
    if kind == "plain":
        # a decaying exponential, a cosine and the sums per bin and term
        ops = 2 * N_BINS * N_TERMS * (2 if c["grad"] else 1)
        return {"bytes": 8.0 * c["n"] * (c["d"] * (2 if c["grad"] else 1) + 1) + 24.0 * N_BINS,
                "flops": 5.0 * c["n"] * ops}
    if kind == "eval":
        return {"bytes": 8.0 * c["n"] * (c["d"] * (2 if c["grad"] else 1) + 1) + size * _nparams(c),
                "flops": c["n"] * _eval_flops(c, c["grad"])}
    if kind == "vjp":
        return {"bytes": 8.0 * c["n"] * (2 * c["d"] + 2) + (size + 8.0) * _nparams(c),
                "flops": c["n"] * 1.5 * _eval_flops(c, True)}
    if kind in ("step", "burnin"):
        per = {"hmc": 10, "nuts": 7}.get(c["sampler"], 1)
        grad = c["sampler"] in ("mala", "hmc", "nuts")
        rec = 4.0 * c["d"] * c["chains"] * (c["steps"] // c.get("thin", 1))
        return {"bytes": rec * (1.5 if kind == "burnin" else 1) + 16.0 * (2 * c["d"] + 1) * c["chains"]
                + size * _nparams(c),
                "flops": float(c["steps"]) * c["chains"] * per * _eval_flops(c, grad)}
    if kind == "train":
        nb = c["n"] // c["batch"]
        return {"bytes": nb * (56.0 * _nparams(c) + 4.0 * c["batch"] * (c["d"] + 1)),
                "flops": nb * c["batch"] * 1.5 * _eval_flops(c, True)}
    n = c["T"] * c["chains"]
    if kind == "ess":
        return {"bytes": 4.0 * n * c["d"], "flops": 2.0 * n * c["d"] * 32}
    return {"bytes": 4.0 * c["d"] * (n + 2 * c["tail"] * c["chains"]),
            "flops": n * c["d"] * (2.0 * c["d"] + 4.0) + 4.0 * c["tail"] * c["chains"] * N_PROJ * c["d"]}


# ---- FP64 values ---------------------------------------------------------------------------
def _unpack(theta, c):
    d, w, nh = c["d"], c["width"], c["n_hidden"]
    Ws, bs, o, fan = [], [], 0, d
    for _ in range(nh):
        Ws.append(theta[o:o + w * fan].view(w, fan))
        o += w * fan
        bs.append(theta[o:o + w])
        o, fan = o + w, w
    return Ws, bs, theta[o:o + w], theta[o + w]


def _mlp(theta, t, c, up=None, want_params=False, want_input=True):
    """Output, input gradient and (with upstream weights) parameter gradient in FP64."""
    Ws, bs, wo, bo = _unpack(theta, c)
    hs = [t]
    for W, b in zip(Ws, bs):
        hs.append(torch.tanh(hs[-1] @ W.T + b))
    out = hs[-1] @ wo + bo
    if not (want_input or want_params):
        return out, None, None
    u = torch.ones_like(out) if up is None else (up(out) if callable(up) else up)
    dl = u[:, None] * wo * (1.0 - hs[-1] ** 2)
    parts = [(u @ hs[-1]), u.sum().view(1)]
    for l in range(len(Ws) - 1, -1, -1):
        if want_params:
            parts = [(dl.T @ hs[l]).reshape(-1), dl.sum(0)] + parts
        dl = dl @ Ws[l]
        if l:
            dl = dl * (1.0 - hs[l] ** 2)
    return out, dl, torch.cat(parts) if want_params else None


def _exact_eval(p, x, c, grad):
    """log pi and its gradient of points x [n][d] in FP64."""
    t = p["twist"]
    lo, hi, mean, prec = (_gpu(p[k]) for k in ("lower", "upper", "gauss_mean", "gauss_prec"))
    out, dt, _ = _mlp(_gpu(p["mlp_params"]), (x - mean) * _gpu(p["in_invscale"]), c, want_input=grad)
    y = x.clone()
    if t:
        y[:, t["v"]] += t["beta"] * ((x[:, t["u"]] - t["center"]) ** 2 - t["kappa"])
    r = y - mean
    pr = r @ prec
    lp = -0.5 * (r * pr).sum(1) + p["mlp_coef"] * out
    inside = ((x >= lo) & (x <= hi)).all(1)
    width = hi - lo
    over = torch.clamp(x - hi, min=0.0) / width
    under = torch.clamp(lo - x, min=0.0) / width
    z = (over + under) / p["penalty_width"]
    if p["box_penalty"]:
        lp = lp - (torch.expm1(z) - z).sum(1)
    else:
        lp = torch.where(inside, lp, torch.full_like(lp, -math.inf))
    if not grad:
        return lp, None
    g = -pr
    if t:
        g = g.clone()
        g[:, t["u"]] -= pr[:, t["v"]] * 2.0 * t["beta"] * (x[:, t["u"]] - t["center"])
    g = g + p["mlp_coef"] * dt * _gpu(p["in_invscale"])
    if p["box_penalty"]:
        g = g - torch.expm1(z) / p["penalty_width"] / width * (torch.sign(over) - torch.sign(under))
    return lp, g


def _exact_plain(p, x, grad):
    """The spectrum log-likelihood of points x [n][d] (autograd for the gradient)."""
    q = {k: _gpu(v) for k, v in p["plain"].items() if isinstance(v, np.ndarray)}
    lps, gs = [], []
    for x0 in torch.split(x, 256):
        x0 = x0.clone().requires_grad_(grad)
        t = (x0 - q["center"]) * q["invscale"]
        s = 0.0
        for m in range(N_TERMS):
            s = s + torch.exp(t @ q["a"][m])[:, None] * torch.exp(
                -(q["gamma0"][m] * torch.exp(t @ q["g"][m]))[:, None] * q["xgrid"]) * torch.cos(
                2.0 * math.pi * q["k"][m] * q["xgrid"]
                + math.pi * torch.tanh(t @ q["p"][m])[:, None])
        lp = -0.5 * ((s - q["data"]) ** 2 * q["inv_sigma2"]).sum(1)
        if grad:
            gs.append(torch.autograd.grad(lp.sum(), x0)[0])
        lps.append(lp.detach())
    return torch.cat(lps), torch.cat(gs) if grad else None


def _exact_train(c, seed):
    params, t, y, perm = _inputs(c, seed)
    p, t, y = _gpu(params), _gpu(t), _gpu(y)
    m, v = torch.zeros_like(p), torch.zeros_like(p)
    nb, Bn = c["n"] // c["batch"], c["batch"]
    loss = 0.0
    for i in range(nb):
        idx = torch.tensor(perm[i * Bn:(i + 1) * Bn].astype(np.int64), device="cuda")
        out, _, g = _mlp(p, t[idx], c, up=lambda o: 2.0 * (o - y[idx]) / Bn, want_params=True)
        loss += float(((out - y[idx]) ** 2).mean())
        m = 0.9 * m + (1.0 - 0.9) * g
        v = 0.999 * v + (1.0 - 0.999) * g * g
        lr = 1e-4 + 0.5 * (1e-3 - 1e-4) * (1.0 + math.cos(math.pi * i / nb))
        p = p - lr * (m / (1.0 - 0.9 ** (i + 1))) / (torch.sqrt(v / (1.0 - 0.999 ** (i + 1))) + 1e-8)
    return {"loss": loss / nb, "params": p.cpu().numpy()}


def _exact_ess(rec):
    """Multi-chain ESS (Geyer's initial monotone sequence on the pair sums)."""
    T, d, n = rec.shape
    nfft = 1 << int(math.ceil(math.log2(2 * T)))
    ess, flags = np.empty(d), np.zeros(d, dtype=np.int32)
    for i in range(d):
        gam, means, ssq = torch.zeros(T, dtype=torch.float64, device="cuda"), [], 0.0
        for x in torch.split(rec[:, i, :], 1024, dim=1):
            x = x.double()
            mean = x.mean(0)
            means.append(mean)
            x = x - mean
            ssq += float((x * x).sum())
            f = torch.fft.rfft(x, n=nfft, dim=0)
            gam += torch.fft.irfft((f * f.conj()).real + 0j, n=nfft, dim=0)[:T].sum(1)
        mean = torch.cat(means)
        w = ssq / n / (T - 1)
        vp = (T - 1) / T * w + (float(mean.var()) if n > 1 else 0.0)
        rho = (1.0 - (w - gam / (n * T)) / vp).cpu().numpy()
        rho[0] = 1.0
        sums, flags[i] = [], 1
        for k in range(T // 2):
            pk = rho[2 * k] + rho[2 * k + 1]
            if not pk > 0.0:
                flags[i] = 0
                break
            sums.append(min(pk, sums[-1]) if sums else pk)
        ess[i] = n * T / max(-1.0 + 2.0 * sum(sums), 1.0 / math.log10(n * T))
    return {"ess": ess, "flags": flags}


def _philox_normals(seed, k, d):
    """Standard normals [k][d] of Philox4x32-10 (Salmon et al. 2011), counter (row, 0,
    6 << 24, block), two 52-bit uniforms per block through Box-Muller."""
    mask = np.uint64(0xFFFFFFFF)
    out = np.empty((k, d + d % 2))
    for b in range((d + 1) // 2):
        c = [np.arange(k, dtype=np.uint64), np.zeros(k, np.uint64),
             np.full(k, 6 << 24, np.uint64), np.full(k, b, np.uint64)]
        k0, k1 = seed & 0xFFFFFFFF, seed >> 32
        for _ in range(10):
            p0, p1 = np.uint64(0xD2511F53) * c[0], np.uint64(0xCD9E8D57) * c[2]
            c = [(p1 >> np.uint64(32)) ^ c[1] ^ np.uint64(k0), p1 & mask,
                 (p0 >> np.uint64(32)) ^ c[3] ^ np.uint64(k1), p0 & mask]
            k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
        u = [(((c[i] >> np.uint64(6)) << np.uint64(26) | (c[i + 1] >> np.uint64(6)))
              .astype(np.float64) + 0.5) * 2.0 ** -52 for i in (0, 2)]
        r = np.sqrt(-2.0 * np.log(u[0]))
        out[:, 2 * b], out[:, 2 * b + 1] = r * np.cos(2 * math.pi * u[1]), r * np.sin(2 * math.pi * u[1])
    return out[:, :d]


def _exact_metrics(c, rec, ref, mu, L):
    T, d, n = rec.shape
    x = rec.double()
    mean = x.mean(0)
    dev = (x - mean).transpose(0, 1).reshape(d, -1)
    W = (dev @ dev.T / (n * (T - 1))).cpu().numpy()
    mb = mean - mean.mean(1, keepdim=True)
    Bm = (mb @ mb.T / (n - 1)).cpu().numpy()
    s = np.sqrt(np.diag(Bm))
    lam = np.linalg.eigvals(np.linalg.solve(W / np.outer(s, s), Bm / np.outer(s, s)))
    Li = _gpu(np.linalg.inv(L))

    def whiten(r):
        return Li @ (r.double().transpose(0, 1).reshape(d, -1) - _gpu(mu)[:, None])

    z = whiten(rec)
    a = (1.0 - CREDIBLE_LEVEL) / 2.0
    lim = []
    for lev in (a, 1.0 - a):
        v = torch.sort(z, dim=1).values
        h = (v.shape[1] - 1) * lev
        k = int(math.floor(h))
        q = v[:, k] if k >= v.shape[1] - 1 else v[:, k] + (h - k) * (v[:, k + 1] - v[:, k])
        lim.append(q.cpu().numpy())
    w = _philox_normals(PROJ_SEED, N_PROJ, d)
    w = _gpu(w / np.linalg.norm(w, axis=1, keepdims=True))
    za, zb = whiten(rec[-c["tail"]:]), whiten(ref)  # equal counts: W1 is a mean difference
    tot = 0.0
    for wk in torch.split(w, 50):
        tot += float((torch.sort(wk @ za, dim=1).values - torch.sort(wk @ zb, dim=1).values)
                     .abs().mean(1).sum())
    return {"rminus1": float(np.max(np.abs(lam))), "lo": lim[0], "hi": lim[1], "sliced_w": tot / N_PROJ}


def exact(case, seed):
    """What run returns, in FP64.  The sampler cases have no such value: a chain's path turns
    on accept decisions, which another rounding of log pi decides otherwise."""
    c, kind = case, case["kind"]
    if kind in ("step", "burnin"):
        return None
    if kind == "train":
        return _exact_train(c, seed)
    if kind == "ess":
        return _exact_ess(_records(c, seed))
    if kind == "metrics":
        return _exact_metrics(c, *_records(c, seed))
    got = _inputs(c, seed)
    p, x = got[0], _gpu(got[1].T)
    if kind == "vjp":
        g = 0.0
        for x0, u0 in zip(torch.split(x, 8192), torch.split(_gpu(got[2]), 8192)):
            g = g + _mlp(_gpu(p["mlp_params"]), (x0 - _gpu(p["in_center"])) * _gpu(p["in_invscale"]),
                         c, up=p["mlp_coef"] * u0, want_params=True)[2]
    grad = c.get("grad", True)
    one = (lambda v: _exact_plain(p, v, grad)) if kind == "plain" else \
        (lambda v: _exact_eval(p, v, c, grad))
    parts = [one(x0) for x0 in torch.split(x, 8192)]
    out = {"logL": torch.cat([a for a, _ in parts])}
    if grad:
        gx = torch.cat([b for _, b in parts])
        out["grad"] = gx if c.get("aos") else gx.T.contiguous()
    if kind == "vjp":
        out["params"] = g
    return out
