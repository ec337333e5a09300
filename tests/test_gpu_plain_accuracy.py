"""Error of the plain model's log pi without its gradient (recurrence over the bins) against that of the
call with gradient (an exponential and a cosine per bin and term), both against extended precision of
the same expression (its constants pi and 2 pi k in FP64): ascending and descending grids, several
restarts of the recurrence, and an offset grid; two and three points per wave give the bits of one.

Tolerance: both forms are sums of bins with a handful of roundings each; their rms relative errors, over
192 points of three problems, are within a fourth of each other.  A factor of the recurrence whose own
rounding accumulates over a segment makes it several times larger."""
import numpy as np
import pytest
import torch

import paper_2606_04895_amd as B
from workloads import make_problem

pytestmark = pytest.mark.gpu


def _problem(xg, seed):
    p = make_problem("c4", seed=seed)
    pl = dict(p["plain"], n_bins=len(xg), xgrid=xg)
    rng = np.random.default_rng(seed)
    t = (pl["theta_star"] - pl["center"]) * pl["invscale"]
    s = (np.exp(pl["a"] @ t)[:, None] * np.exp(-(pl["gamma0"] * np.exp(pl["g"] @ t))[:, None] * xg)
         * np.cos(2 * np.pi * pl["k"][:, None] * xg + np.pi * np.tanh(pl["p"] @ t)[:, None])).sum(0)
    sd = 0.05 * (1.0 + rng.random(len(xg)))
    pl.update(data=s + sd * rng.normal(size=len(xg)), inv_sigma2=sd ** -2)
    return dict(p, plain=pl, plain_mode=2)


def _reference(pl, x):
    L = np.longdouble
    t = (x.astype(L) - pl["center"].astype(L)) * pl["invscale"].astype(L)
    xg, S = pl["xgrid"].astype(L), 0
    for m in range(pl["n_terms"]):
        gam = L(pl["gamma0"][m]) * np.exp(t @ pl["g"][m].astype(L))
        ph = L(2.0 * np.pi * pl["k"][m]) * xg + L(np.pi) * np.tanh(t @ pl["p"][m].astype(L))[:, None]
        S = S + np.exp(t @ pl["a"][m].astype(L))[:, None] * np.exp(-gam[:, None] * xg) * np.cos(ph)
    return -L(0.5) * ((S - pl["data"].astype(L)) ** 2 * pl["inv_sigma2"].astype(L)).sum(1)


@pytest.mark.parametrize("name,xg", [
    ("ascending", np.arange(2500) / 2499.0), ("descending", 1.0 - np.arange(2500) / 2499.0),
    ("several restarts", np.arange(9000) / 8999.0), ("offset", 10.0 + np.arange(2500) / 2499.0),
])
def test_error_of_the_values_is_that_of_the_call_with_gradient(name, xg):
    err = {False: [], True: []}
    for seed in (11, 12, 13):
        p = _problem(xg, seed)
        pl = p["plain"]
        rng = np.random.default_rng(seed)
        w = 1.0 / pl["invscale"]
        x = pl["theta_star"] + w * rng.uniform(-0.1, 0.1, (64, p["d"]))
        ref = _reference(pl, x)
        ctx = B.best_init(p, n_chains=16, precision="fp32", seed=1)
        for grad in err:
            lp = B.best_logL_grad(ctx, torch.tensor(x.T.copy(), device="cuda"), want_grad=grad)[0]
            err[grad].append(((lp.cpu().numpy() - ref) / ref).astype(np.float64))
    rms = {g: np.sqrt(np.mean(np.concatenate(e) ** 2)) for g, e in err.items()}
    print(name, "values %.2e with gradient %.2e" % (rms[False], rms[True]), flush=True)
    assert rms[False] <= 1.25 * rms[True]


def test_points_per_wave_do_not_change_the_bits():
    p = _problem(np.arange(700) / 699.0, 11)
    p["plain"]["gamma0"] = p["plain"]["gamma0"] * 40  # restarts at every chunk for some of the points
    p["plain"]["gamma0"][0] = 320.0                   # and some out of the recurrence's range
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    n = 16 * cu + 2
    rng = np.random.default_rng(1)
    x = torch.tensor(p["lower"][:, None] + (p["upper"] - p["lower"])[:, None] * rng.random((6, n)), device="cuda")
    ctx = B.best_init(p, n_chains=16, precision="fp32", seed=1)
    full = B.best_logL_grad(ctx, x, want_grad=False)[0]  # three per wave, a ragged last one
    for m in (1, 4 * cu, 4 * cu + 1, 16 * cu):           # one and two per wave
        part = B.best_logL_grad(ctx, x[:, :m].contiguous(), want_grad=False)[0]
        assert torch.equal(part, full[:m]), m
