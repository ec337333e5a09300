"""Metropolis-Hastings on lane groups against the loop form: the same chains at a tile width that takes
the eight-lane form (d <= 8; with and without waves to spare for the draws), the sixteen-lane form
(8 < d <= 32 on 32-chain tiles) and the loops, in one launch of seven recorded steps and in seven
launches of one.  Every form keeps the order of the sums, so states, log pi, records and counts are
equal, bit for bit."""
import numpy as np
import pytest
import torch

import paper_2606_04895_amd as B
from workloads import small_problem

pytestmark = pytest.mark.gpu


def _run(prob, prec, cpb, launches):
    n, thin = 100, 2
    ctx = B.best_init(prob, n_chains=n, precision=prec, seed=21, init="gaussian",
                      init_point=prob["gauss_mean"], init_scale=0.3, chains_per_block=cpb)
    B.best_set_whitening(ctx, prob["gauss_mean"], 0.4 * np.linalg.cholesky(prob["closed_cov"]))
    rec = torch.zeros(4, prob["d"], n, dtype=torch.float32, device="cuda")
    acc = [B.best_step(ctx, "mh", k, mh_scale=1.0, thin=thin,
                       record=rec if len(launches) == 1 else None) for k in launches]
    x, lp, _ = B.best_get_state(ctx)
    sums = {k: sum(r[k] for r in acc) for k in ("accepted", "evals", "n_nonfinite", "n_oob")}
    return np.array(x), np.array(lp), rec.cpu().numpy(), sums


@pytest.mark.parametrize("prec,d,widths", [
    ("fp32", 1, (16, 32, 64)), ("fp32", 8, (16, 32, 64)), ("bf16", 5, (16, 32, 64)),
    ("fp64", 6, (16,)), ("fp64", 9, (16,)),
    ("bf16", 9, (32, 16)), ("fp16", 27, (32, 16)), ("bf16", 32, (32, 16)),
])
def test_lane_group_moves_equal_the_loops(prec, d, widths):
    prob = small_problem(d=d, width=128, n_hidden=2, twist=d >= 4)
    x0, lp0, rec0, s0 = _run(prob, prec, widths[0], [7])
    assert 0 < np.count_nonzero(np.diff(rec0[:3], axis=0)) < 2 * d * 100  # some moved, some stayed
    assert np.array_equal(rec0[3], np.zeros_like(rec0[3]))
    for cpb, launches in [(w, [7]) for w in widths[1:]] + [(w, [1] * 7) for w in widths]:
        x, lp, rec, s = _run(prob, prec, cpb, launches)
        assert np.array_equal(x, x0) and np.array_equal(lp, lp0) and s == s0, (cpb, launches)
        if len(launches) == 1:
            assert np.array_equal(rec, rec0), cpb
