"""Log pi of the plain model without its gradient (one wave per point, recurrence over the bins)
against an extended-precision evaluation of the same model and against the call with gradient: bins
short of, at and past the 64 lanes and the 4096 bins between restarts, fewer than eight terms, an
uneven grid (every bin evaluated directly), a Gaussian part with a twisted pair, points outside the
hard box and the smooth penalty, and a single point.

Tolerance: a residual S_j - data_j carries the rounding of the phase 2 pi k x + phi, half an ulp of
150 rad at k = 24 (1.4e-14) times the amplitudes over sigma, in a sum of squares: 1e-11 relative."""
import numpy as np
import pytest
import torch

import paper_2606_04895_amd as B
from workloads import make_problem

pytestmark = pytest.mark.gpu


def _problem(nb, nt, even, seed, gauss):
    p = make_problem("c4")
    rng = np.random.default_rng(seed)
    pl = dict(p["plain"], n_bins=nb, n_terms=nt)
    x = np.arange(nb) / max(nb - 1.0, 1.0)
    pl.update(xgrid=x if even else x ** 1.3, data=rng.normal(size=nb), inv_sigma2=1.0 + rng.random(nb))
    for k in ("a", "g", "p", "k", "gamma0"):
        pl[k] = pl[k][:nt]
    p = dict(p, plain=pl, plain_mode=2)
    if gauss:
        q = rng.normal(size=(6, 6))
        p.update(gauss_coef=0.7, gauss_mean=pl["center"], gauss_prec=q @ q.T + np.eye(6),
                 twist=dict(u=4, v=1, beta=0.3, center=0.1, kappa=0.2))
    return p


def _reference(p, x):
    L = np.longdouble
    pl = p["plain"]
    pi = L("3.14159265358979323846264338327950288")
    t = (x.astype(L) - pl["center"].astype(L)) * pl["invscale"].astype(L)
    xg, S = pl["xgrid"].astype(L), 0
    for m in range(pl["n_terms"]):
        gam = L(pl["gamma0"][m]) * np.exp(t @ pl["g"][m].astype(L))
        ph = 2 * pi * L(pl["k"][m]) * xg + pi * np.tanh(t @ pl["p"][m].astype(L))[:, None]
        S = S + np.exp(t @ pl["a"][m].astype(L))[:, None] * np.exp(-gam[:, None] * xg) * np.cos(ph)
    lp = -L(0.5) * ((S - pl["data"].astype(L)) ** 2 * pl["inv_sigma2"].astype(L)).sum(1)
    if p["gauss_coef"]:
        y, w = x.astype(L), p["twist"]
        y[:, w["v"]] += w["beta"] * ((y[:, w["u"]] - w["center"]) ** 2 - w["kappa"])
        r = y - p["gauss_mean"]
        lp = lp - L(p["gauss_coef"]) * L(0.5) * np.einsum("ni,ij,nj->n", r, p["gauss_prec"].astype(L), r)
    return lp


@pytest.mark.parametrize("nb,nt,even,n,gauss", [
    (1, 2, True, 5, False), (63, 3, True, 9, False), (64, 8, True, 4, True), (65, 1, True, 3, False),
    (2500, 8, True, 33, True), (4096, 8, True, 2, False), (4097, 5, True, 6, False),
    (9000, 8, True, 3, False), (300, 8, False, 7, True), (2500, 8, True, 1, False),
])
def test_plain_values(nb, nt, even, n, gauss):
    print(f"plain values nb={nb} nt={nt} even={even} n={n} gauss={gauss}", flush=True)
    p = _problem(nb, nt, even, nb + nt, gauss)
    rng = np.random.default_rng(n)
    x = p["lower"] + rng.random((n, 6)) * (p["upper"] - p["lower"])
    ctx = B.best_init(p, n_chains=16, precision="fp32", seed=1)
    xt = torch.tensor(x.T.copy(), device="cuda")
    lp = B.best_logL_grad(ctx, xt, want_grad=False)[0].cpu().numpy()
    ref = _reference(p, x)
    np.testing.assert_allclose(lp, ref.astype(np.float64), rtol=1e-11)
    np.testing.assert_allclose(lp, B.best_logL_grad(ctx, xt)[0].cpu().numpy(), rtol=1e-11)


def test_plain_values_outside_the_box_match_the_call_with_gradient():
    p = _problem(200, 8, True, 3, True)
    rng = np.random.default_rng(2)
    w = p["upper"] - p["lower"]
    x = torch.tensor((p["lower"] + rng.uniform(-0.2, 1.2, (40, 6)) * w).T.copy(), device="cuda")
    for pen in (0, 1):
        ctx = B.best_init(dict(p, box_penalty=pen, penalty_width=0.05), n_chains=16,
                          precision="fp32", seed=1)
        a = B.best_logL_grad(ctx, x, want_grad=False)[0].cpu().numpy()
        b = B.best_logL_grad(ctx, x)[0].cpu().numpy()
        assert np.isneginf(a).any() == (pen == 0)
        np.testing.assert_allclose(a, b, rtol=1e-11)
