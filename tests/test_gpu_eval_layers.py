"""log pi and gradient of small batches, and of the last partly filled round of tiles of large ones,
are evaluated layer by layer; the points' results equal, bit for bit, those of the tiles.  A point's tile
results come from a batch of a whole round of tiles that holds it (256 CUs times a tile's chains), its
layer results from a batch of its own: one point, a ragged last column tile, the largest batch of the
route and one past it, a round of tiles plus a remainder, on networks of two to five hidden layers,
widths with one to eight row tiles per wave, inputs of one and two row tiles with and without a twisted
pair, training-box fallback to the plain model, and points outside the box."""
import numpy as np
import pytest
import torch

import paper_2606_04895_amd as B
from workloads import make_problem, small_problem
from workloads.synth import xavier_mlp

pytestmark = pytest.mark.gpu


def _points(prob, n, seed):
    rng = np.random.default_rng(seed)
    d = prob["d"]
    x = prob["gauss_mean"][:, None] + np.linalg.cholesky(prob["closed_cov"]) @ rng.normal(size=(d, n))
    lo, up = np.asarray(prob["lower"]), np.asarray(prob["upper"])
    x[:, 3::17] = (up + 0.01 * (up - lo))[:, None]  # outside
    return x


def _eval(ctx, x, grad=True):
    lp, g = B.best_logL_grad(ctx, torch.tensor(x, device="cuda").contiguous(), want_grad=grad)
    return lp.cpu().numpy(), g.cpu().numpy() if grad else None


@pytest.mark.parametrize("prec,d,width,nh,most", [
    ("bf16", 12, 512, 4, 1024), ("fp16", 27, 1024, 5, 2048), ("fp16", 5, 512, 2, 1024),
    ("fp32", 6, 128, 2, 1024), ("fp32", 9, 256, 3, 2048), ("fp32", 20, 512, 4, 2048),
    ("bf16", 7, 256, 3, 0),
])
def test_layers_equal_tiles(prec, d, width, nh, most):
    prob = small_problem(d=d, width=width, n_hidden=nh, twist=d >= 4)
    ctx = B.best_init(prob, n_chains=64, precision=prec, seed=3, chains_per_block=16)
    full = torch.cuda.get_device_properties(0).multi_processor_count * 32
    x = _points(prob, full + 37, 11)  # one or two workgroups per CU: full is whole rounds either way
    lp, g = _eval(ctx, x)
    rot = np.roll(x, -(full - 5), axis=1)  # the former remainder now inside a round
    lpr, gr = _eval(ctx, rot)
    assert np.array_equal(np.roll(lpr, full - 5), lp) and np.array_equal(np.roll(gr, full - 5, 1), g)
    for n in sorted({1, 16, 37, max(most, 64), most + 1}):
        a, b = _eval(ctx, x[:, :n])
        assert np.array_equal(a, lp[:n]) and np.array_equal(b, g[:, :n]), n
        v, _ = _eval(ctx, x[:, :n], grad=False)
        assert np.array_equal(v, lp[:n]), n


def test_layers_with_the_plain_model_outside_the_training_box():
    p = make_problem("c4")
    if p["mlp_params"] is None:
        p["mlp_params"] = xavier_mlp(np.random.default_rng(4), p["d"], p["width"], p["n_hidden"])
    q = dict(p, plain_mode=1)
    rng = np.random.default_rng(2)
    x = np.concatenate([rng.uniform(p["train_lo"], p["train_hi"], size=(32, p["d"])),
                        rng.uniform(p["lower"], p["upper"], size=(32, p["d"]))]).T
    ctx = B.best_init(q, n_chains=64, precision="fp32", seed=3)
    lo, hi = np.asarray(q["train_lo"])[:, None], np.asarray(q["train_hi"])[:, None]
    inside = np.all((x >= lo) & (x <= hi), axis=0)
    assert 0 < inside.sum() < 64
    lp, g = _eval(ctx, x)
    ref = B.best_init(dict(p, plain_mode=0), n_chains=64, precision="fp32", seed=3)
    pl = B.best_init(dict(p, plain_mode=2), n_chains=64, precision="fp32", seed=3)
    for c, m in ((ref, inside), (pl, ~inside)):
        a, b = _eval(c, x)
        assert np.array_equal(a[m], lp[m]) and np.array_equal(b[:, m], g[:, m])
