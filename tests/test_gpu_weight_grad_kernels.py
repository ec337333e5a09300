"""The weight-gradient launch at its edges, through the trainer's minibatch gradient, against
the FP64 oracle: batches shorter than the ring of k-steps in flight, equal to it, and with a
remainder; one and two tiles per wave on either side of the rule's threshold; no hidden GEMM
at all; input dimensions of one, one block of eight and several blocks.

Tolerance (per block of parameters, on the scale of its largest component): the network's
forward and reverse passes and the sums over the batch run in FP32, each layer sum of at most
1024 terms with a relative error of a few 2^-24 sqrt(1024), compounded over the layers: 2e-5."""
import numpy as np
import pytest
import torch

import paper_2606_04895_amd as B
from oracle import mlp as OM, target as OT, train as OTR
from workloads import small_problem
from workloads.synth import mlp_layout, xavier_mlp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,width,nh,batch", [
    (1, 128, 1, 16),     # no hidden GEMM
    (9, 128, 2, 16),     # one tile per wave, one k-step
    (32, 128, 2, 80),    # ring + 1 k-steps, four blocks of inputs
    (8, 256, 3, 64),     # exactly one ring
    (5, 512, 2, 96),     # 1024 tiles: one per wave
    (27, 512, 3, 48),    # 2048 tiles: two by two per wave, shorter than the ring
    (6, 1024, 2, 112),   # two by two, ring + remainder
])
def test_weight_gradients_at_the_edges(d, width, nh, batch):
    print(f"weight gradients d={d} width={width} nh={nh} batch={batch}", flush=True)
    rng = np.random.default_rng(d * 1000 + width + batch)
    p = xavier_mlp(rng, d, width, nh)
    p += 0.01 * rng.normal(size=p.size)
    t = rng.uniform(-1, 1, (batch, d)).astype(np.float32)
    y = rng.normal(size=batch).astype(np.float32)
    tr = B.Trainer(d, width, nh, p, precision="fp32")
    loss, g = tr.grad(torch.tensor(t, device="cuda"), torch.tensor(y, device="cuda"))
    loss_ref, ref = OTR.mse_loss_grad(p.astype(np.float32).astype(np.float64),
                                      t.astype(np.float64), y.astype(np.float64), d, width, nh)
    assert abs(loss - loss_ref) < 2e-5 * loss_ref
    for name, off, shape in mlp_layout(d, width, nh):
        n = int(np.prod(shape))
        a, b = g[off:off + n], ref[off:off + n]
        assert np.abs(a - b).max() < 2e-5 * np.abs(b).max() + 1e-12, (name, np.abs(a - b).max())


@pytest.mark.parametrize("prec,n", [
    ("fp32", 4100),    # one row and two columns of blocks per wave, the last column alone
    ("bf16", 8200),    # two by two, the last column alone
    ("fp16", 32769),   # two by four, a last column of one point
    ("fp16", 1),       # one block per wave, one point
])
def test_batch_passes_with_a_ragged_last_column(prec, n):
    """Tolerance on the scale of the largest component: 2e-5 in FP32; with 16-bit layer inputs
    (8 / 11 bits, rounding 2^-9 / 2^-12 relative through two layers and the deltas) 2^-7 / 2^-10."""
    print(f"batch passes {prec} n={n}", flush=True)
    prob = small_problem(d=5, width=128, n_hidden=3)
    ctx = B.best_init(prob, n_chains=64, precision=prec, seed=1)
    rng = np.random.default_rng(n)
    x = prob["gauss_mean"] + 1.5 * rng.normal(size=(n, 5)) * np.sqrt(np.diag(prob["closed_cov"]))
    w = rng.normal(size=n)
    g = B.best_logL_param_grad(ctx, torch.tensor(x.T.copy(), device="cuda"),
                               torch.tensor(w, device="cuda")).cpu().numpy()
    ref, _ = OM.param_grad(prob["mlp_params"], OT.normalise(prob, x), prob["mlp_coef"] * w, 5,
                           128, 3)
    tol = {"fp32": 2e-5, "fp16": 2.0 ** -10, "bf16": 2.0 ** -7}[prec]
    assert np.abs(g - ref).max() < tol * np.abs(ref).max()
