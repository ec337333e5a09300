"""The plain model's values inside the tiles: Metropolis-Hastings, stretch and differential-evolution
steps on the plain model everywhere (plain_mode 2) and outside a training box that the chains cross
(plain_mode 1), step by step against the oracle; even and uneven grids, four and eight waves per tile.

Tolerance: log pi is about -1e4 and carries 1e-13 of it (1e-9), so a decision may differ only where
log alpha and log u are that close; proposals are FP64 sums of the same terms, 1e-10 relative."""
import numpy as np
import pytest

import paper_2606_04895_amd as B
from oracle import samplers as OS, target as OT
from workloads import make_problem
from workloads.synth import xavier_mlp

pytestmark = pytest.mark.gpu


def _problem(mode, even):
    p = make_problem("c4")
    rng = np.random.default_rng(3)
    nb, nt = 300, 3
    x = np.arange(nb) / (nb - 1.0)
    pl = dict(p["plain"], n_bins=nb, n_terms=nt, xgrid=x if even else x ** 1.3,
              data=rng.normal(size=nb), inv_sigma2=1.0 + rng.random(nb))
    for k in ("a", "g", "p", "k", "gamma0"):
        pl[k] = pl[k][:nt]
    return dict(p, plain=pl, plain_mode=mode, width=128, n_hidden=2,
                mlp_params=xavier_mlp(rng, p["d"], 128, 2))


@pytest.mark.parametrize("sampler,kw", [("mh", dict(mh_scale=0.7)), ("aies", dict(stretch_a=2.0)),
                                        ("de", dict(de_sigma=0.1))])
@pytest.mark.parametrize("mode,prec,even", [(1, "fp64", True), (1, "fp64", False), (2, "fp64", True),
                                            (2, "fp32", True), (2, "bf16", True), (2, "bf16", False)])
def test_steps_on_the_plain_model(mode, prec, even, sampler, kw):
    p, n, seed = _problem(mode, even), 70, 0xBE57
    mid = 0.5 * (p["train_lo"] + p["train_hi"])
    L = np.diag(p["train_hi"] - p["train_lo"])
    ctx = B.best_init(p, n_chains=n, precision=prec, seed=seed)
    B.best_set_whitening(ctx, mid, L)
    # in and around the training box
    B.best_set_state(ctx, mid[:, None] + L @ np.random.default_rng(8).uniform(-0.55, 0.55, (p["d"], n)))
    for s in range(3):
        t = B.best_get_step_counter(ctx)
        x0 = B.best_get_state(ctx)[0].T
        if mode == 1 and s == 0:
            inside = OT.in_box(p["train_lo"], p["train_hi"], x0)
            assert 0 < inside.sum() < n
        if sampler == "mh":
            W = dict(mu=mid, L=L)
            new, info = OS.mh_step(p, W, OS.init_state(p, W, x0), t, seed, kw["mh_scale"])
            want = mid[None, :] + new["z"] @ L.T
        else:
            st = dict(x=x0, lp=OT.log_target(p, x0)[0])
            new, info = (OS.aies_step(p, st, t, seed, kw["stretch_a"]) if sampler == "aies" else
                         OS.de_step(p, st, t, seed, kw["de_sigma"]))
            want = new["x"]
        B.best_step(ctx, sampler, 1, **kw)
        x1, lp1, _ = B.best_get_state(ctx)
        x1 = x1.T
        moved = np.any(x1 != x0, axis=1)
        bad = moved != info["accepted"]
        gap = np.abs(info["log_alpha"] - info["log_u"])[bad]
        assert np.all(gap < 1e-9), gap
        assert 0 < info["accepted"].sum() < n
        ok = ~bad
        rel = np.abs(x1[ok] - want[ok]) / (np.abs(want[ok]) + np.abs(want[ok] - x0[ok]) + 1e-12)
        assert rel.max() < 1e-10, rel.max()
        lo = OT.log_target(p, x1)[0]
        np.testing.assert_allclose(lp1, lo, rtol=1e-11, atol=1e-9)  # the FP64 network: 1e-9


@pytest.mark.parametrize("prec,n", [("fp32", 64), ("fp32", 5000), ("fp64", 64)])
def test_values_alone_with_the_plain_model_outside_the_training_box(prec, n):
    """Layer by layer (FP32, small n) and in tiles: the network's values inside the training box are
    the bits of the call with gradient, the plain model's outside it agree to rounding."""
    p = _problem(1, True)
    rng = np.random.default_rng(n)
    w = p["train_hi"] - p["train_lo"]
    x = (p["train_lo"] + rng.uniform(-0.1, 1.1, (n, p["d"])) * w).T.copy()
    inside = OT.in_box(p["train_lo"], p["train_hi"], x.T)
    assert 0 < inside.sum() < n
    ctx = B.best_init(p, n_chains=64, precision=prec, seed=3)
    a = B.best_logL_grad(ctx, x, want_grad=False)[0]
    b = B.best_logL_grad(ctx, x)[0]
    assert np.array_equal(a[inside], b[inside])
    np.testing.assert_allclose(a[~inside], b[~inside], rtol=1e-11)


@pytest.mark.parametrize("prec,cpb", [("bf16", 16), ("bf16", 32), ("bf16", 64), ("fp32", 16), ("fp64", 16)])
def test_kernels_without_the_plain_model_equal_those_with_it(prec, cpb):
    """plain_mode 0 has kernels of its own for values; with a training box as large as the prior box
    plain_mode 1 does the same work in the others: evaluations (layer by layer and in tiles) and the moves that
    need values alone, bit for bit."""
    base = _problem(0, True)
    base.update(train_lo=base["lower"], train_hi=base["upper"])
    rng = np.random.default_rng(cpb)
    w = base["upper"] - base["lower"]
    x = (base["lower"] + rng.random((5000, base["d"])) * w).T.copy()
    out = []
    for mode in (0, 1):
        p = dict(base, plain_mode=mode)
        ctx = B.best_init(p, n_chains=160, precision=prec, seed=5, chains_per_block=cpb)
        res = []
        for n in (64, 5000):
            for grad in (False, True):
                lp, g = B.best_logL_grad(ctx, x[:, :n].copy(), want_grad=grad)
                res += [lp] + ([g] if grad else [])
        B.best_set_whitening(ctx, 0.5 * (base["lower"] + base["upper"]), np.diag(0.2 * w))
        B.best_set_state(ctx, x[:, :160].copy())
        for s, kw in (("mh", dict(mh_scale=0.5)), ("aies", {}), ("de", {})):
            st = B.best_step(ctx, s, 3, **kw)
            assert st["accepted"] > 0
            res += [np.array(v) for v in B.best_get_state(ctx)[:2]]
        out.append(res)
    for a, b in zip(*out):
        assert np.array_equal(a, b)
