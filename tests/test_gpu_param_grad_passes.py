"""The parameter gradient of batches larger than one pass of 65536 points: passes are independent columns, so
a gradient whose upstream weights vanish outside one pass equals, bit for bit, that of the pass's points
alone; and the device memory of a call is what its documentation says."""
import numpy as np
import pytest
import torch

import paper_2606_04895_amd as B
from workloads import small_problem

pytestmark = pytest.mark.gpu

PASS = 65536


@pytest.mark.parametrize("prec,nh", [("fp32", 2), ("fp32", 1), ("bf16", 3), ("fp16", 1)])
def test_passes_are_independent(prec, nh):
    print(f"param grad passes {prec} nh={nh}", flush=True)
    prob = small_problem(d=5, width=128, n_hidden=nh)
    n, rng = PASS + 37, np.random.default_rng(nh)
    x = prob["gauss_mean"][:, None] + rng.normal(size=(5, n))
    u = rng.normal(size=n)
    ctx = B.best_init(prob, n_chains=64, precision=prec, seed=1)

    def grad(x, u):
        return B.best_logL_param_grad(ctx, torch.tensor(x.copy(), device="cuda"),
                                      torch.tensor(u.copy(), device="cuda")).cpu().numpy()

    head, tail = np.where(np.arange(n) < PASS, u, 0.0), np.where(np.arange(n) < PASS, 0.0, u)
    a, b = grad(x, head), grad(x[:, :PASS], u[:PASS])
    assert np.abs(b).max() > 0 and np.array_equal(a, b)
    a, b = grad(x, tail), grad(x[:, PASS:], u[PASS:])
    assert np.abs(b).max() > 0 and np.array_equal(a, b)


@pytest.mark.parametrize("prec,nh", [("bf16", 1), ("fp32", 2)])
def test_memory_per_point(prec, nh):
    d, width, n = 5, 128, 400000
    prob = small_problem(d=d, width=width, n_hidden=nh)
    ctx = B.best_init(prob, n_chains=64, precision=prec, seed=1)
    x = torch.tensor(np.repeat(prob["gauss_mean"][:, None], n, axis=1), device="cuda")
    B.best_logL_param_grad(ctx, x[:, :16].contiguous())
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    B.best_logL_param_grad(ctx, x)
    torch.cuda.synchronize()
    used = free - torch.cuda.mem_get_info()[0]
    size = 4 if prec == "fp32" else 2
    bound = 4 * n * (2 * nh * width + d + 1) + (2 * PASS * width * size if nh > 1 else 0)
    assert 0.9 * bound < used < bound + (16 << 20), (used, bound)
