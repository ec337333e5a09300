"""Widths whose row tiles per wave are neither 1, 2 nor a multiple of 4: the input layer covers all of
them.  log pi against the FP64 oracle at the precision's tolerance of the width 128 tests (FP32: 2e-5
relative to the size of log pi's terms, 16 bit: 2e-2)."""
import numpy as np
import pytest

import paper_2606_04895_amd as B
from oracle import target as OT
from workloads import small_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,width,tol", [("fp32", 384, 2e-5), ("fp32", 640, 2e-5), ("bf16", 384, 2e-2),
                                            ("fp16", 768, 2e-2), ("fp64", 384, 1e-9)])
def test_every_row_tile_of_the_input_layer(prec, width, tol):
    prob = small_problem(d=5, width=width, n_hidden=2)
    ctx = B.best_init(prob, n_chains=64, precision=prec, seed=3, chains_per_block=16)
    n = 2304  # more than the batches that are evaluated layer by layer
    rng = np.random.default_rng(1)
    x = prob["gauss_mean"][:, None] + np.linalg.cholesky(prob["closed_cov"]) @ rng.normal(size=(5, n))
    lp, _ = B.best_logL_grad(ctx, x, want_grad=False)
    ref, _ = OT.log_target(prob, np.ascontiguousarray(x.T))
    assert np.max(np.abs(lp - ref) / (1.0 + np.abs(ref))) < tol
