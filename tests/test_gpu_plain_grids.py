"""Values of the plain model on every kind of grid that a problem may bring: descending grids and
negative damping, whose terms grow along the bins, damping that leaves the range of FP64 within the
grid (a term's first bin underflows or overflows), points on both sides of the recurrence's bound, and
a grid with a NaN.  Each through the batch kernel (plain_mode 2) and, for points outside the training
box, through the closing kernel of the layer-by-layer evaluation (FP32) and the tiles (FP64).

Tolerance: the exponent -gamma x is rounded to half an ulp of 1024 (5.7e-14 relative in its
exponential) and the phase to half an ulp of 150 rad, in a sum of squares: 1e-11 relative."""
import numpy as np
import pytest
import torch

import paper_2606_04895_amd as B
from workloads import make_problem
from workloads.synth import xavier_mlp

pytestmark = pytest.mark.gpu

ROUTES = [(2, "fp32"), (1, "fp32"), (1, "fp64")]


def _problem(xg, gamma0, mode, g_scale=0.0):
    p = make_problem("c4")
    rng = np.random.default_rng(len(xg))
    nb, nt = len(xg), len(gamma0)
    pl = dict(p["plain"], n_bins=nb, n_terms=nt, xgrid=np.asarray(xg, dtype=np.float64),
              data=rng.normal(size=nb), inv_sigma2=1.0 + rng.random(nb),
              gamma0=np.asarray(gamma0, dtype=np.float64))
    for k in ("a", "g", "p", "k"):
        pl[k] = pl[k][:nt]
    pl["g"] = g_scale * pl["g"]
    p = dict(p, plain=pl, plain_mode=mode)
    if mode == 1:
        w = p["upper"] - p["lower"]  # a training box that no test point lies in
        p.update(train_lo=p["upper"] - 1e-9 * w, train_hi=p["upper"])
        if p["mlp_params"] is None:
            p["mlp_params"] = xavier_mlp(np.random.default_rng(4), p["d"], p["width"], p["n_hidden"])
    return p


def _reference(p, x):
    """Extended precision, term by term; the exponential rounded to the range of FP64."""
    L = np.longdouble
    pl = p["plain"]
    pi = L("3.14159265358979323846264338327950288")
    t = (x.astype(L) - pl["center"].astype(L)) * pl["invscale"].astype(L)
    xg, S = pl["xgrid"].astype(L), 0
    for m in range(pl["n_terms"]):
        gam = L(pl["gamma0"][m]) * np.exp(t @ pl["g"][m].astype(L))
        ph = 2 * pi * L(pl["k"][m]) * xg + pi * np.tanh(t @ pl["p"][m].astype(L))[:, None]
        with np.errstate(over="ignore"):
            e = np.exp(-gam[:, None] * xg).astype(np.float64).astype(L)
        S = S + np.exp(t @ pl["a"][m].astype(L))[:, None] * (e * np.cos(ph))
    lp = -L(0.5) * ((S - pl["data"].astype(L)) ** 2 * pl["inv_sigma2"].astype(L)).sum(1)
    with np.errstate(over="ignore"):
        return lp.astype(np.float64)


GRIDS = {
    # name: grid, gamma0, scale of the damping's dependence on the parameters
    "descending": (np.linspace(1.0, 0.0, 2500), [0.5, 1.0, 4.0], 1.0),
    "descending, first bins underflow": (np.linspace(1.0, 0.0, 2500), [760.0, 1.0], 0.0),
    "descending, first bins subnormal": (np.linspace(1.0, 0.0, 700), [735.0, 2.0], 0.0),
    "negative damping, first bins underflow": (np.linspace(-1.0, 0.0, 2500), [-800.0, -3.0], 0.0),
    "first bins overflow": (np.linspace(-1.0, 1.0, 300), [760.0], 0.0),
    "last bins underflow": (np.linspace(0.0, 1.0, 2500), [5000.0, 1.0], 0.0),
    "both sides of the bound": (np.linspace(0.0, 1.0, 2500), [280.0, 300.0, 1.0], 1.0),
    "both sides of the bound, descending": (np.linspace(1.0, 0.0, 9000), [290.0, 1.0], 1.0),
}


@pytest.mark.parametrize("mode,prec", ROUTES)
@pytest.mark.parametrize("grid", GRIDS)
def test_plain_values_on_every_grid(grid, mode, prec):
    print(f"plain grid '{grid}' mode={mode} {prec}", flush=True)
    xg, gamma0, gs = GRIDS[grid]
    p = _problem(xg, gamma0, mode, gs)
    rng = np.random.default_rng(7)
    x = p["lower"] + rng.random((23, p["d"])) * 0.99 * (p["upper"] - p["lower"])
    ctx = B.best_init(p, n_chains=16, precision=prec, seed=1)
    got = B.best_logL_grad(ctx, torch.tensor(x.T.copy(), device="cuda"), want_grad=False)[0]
    ref = _reference(p, x)
    if grid == "first bins overflow":
        assert np.isneginf(ref).all()
    np.testing.assert_allclose(got.cpu().numpy(), ref, rtol=1e-11)


@pytest.mark.parametrize("mode,prec", ROUTES)
def test_a_nan_in_the_grid_gives_nan(mode, prec):
    xg = np.linspace(0.0, 1.0, 2500)
    xg[1234] = np.nan
    p = _problem(xg, [0.5, 1.0], mode)
    ctx = B.best_init(p, n_chains=16, precision=prec, seed=1)
    x = np.repeat(0.5 * (p["lower"] + p["upper"])[:, None], 5, axis=1)
    got = B.best_logL_grad(ctx, torch.tensor(x, device="cuda"), want_grad=False)[0]
    assert torch.isnan(got).all()


@pytest.mark.parametrize("nt", [1, 4, 5, 8])
@pytest.mark.parametrize("n", [1, 2, 3, 40])
@pytest.mark.parametrize("mode,prec", ROUTES)
def test_uneven_grids(mode, prec, n, nt):
    """One and two points go to a workgroup each, more to a wave each; up to four terms one by one,
    more together."""
    p = _problem(np.linspace(0.0, 1.0, 300) ** 1.3, 0.5 * np.arange(1, nt + 1), mode, 1.0)
    rng = np.random.default_rng(n)
    x = p["lower"] + rng.random((n, p["d"])) * 0.99 * (p["upper"] - p["lower"])
    ctx = B.best_init(p, n_chains=16, precision=prec, seed=1)
    got = B.best_logL_grad(ctx, torch.tensor(x.T.copy(), device="cuda"), want_grad=False)[0]
    np.testing.assert_allclose(got.cpu().numpy(), _reference(p, x), rtol=1e-11)
