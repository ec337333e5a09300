"""The metric kernels at their edges, against the oracle on the same records: sample sets around the
4096 keys of a sort tile, with several merge passes and runs of very different lengths; draws with
ties (more equal values than the selection gathers, so that it runs to the last bit); the smallest
sets; chain counts off the vector width and more than sixteen parameters for R - 1.

Tolerances as for the larger checks: sliced Wasserstein 1e-9 relative, limits 1e-12, R - 1 1e-9
(FP64 sums of the same floats in another order; the selected values are the sorted ones)."""
import numpy as np
import pytest
import torch

import paper_2606_04895_amd as B
from oracle import metrics as OM
from workloads import small_problem

pytestmark = pytest.mark.gpu


def _ctx(d):
    return B.best_init(small_problem(d=d, width=128, n_hidden=1), n_chains=16, precision="fp32")


def _dev(x):
    return torch.tensor(x, dtype=torch.float32, device="cuda")


@pytest.mark.parametrize("na,nb,K,grid", [
    (1, 1, 3, 0), (4095, 4097, 2, 0), (4096, 4096, 1, 4), (1, 12289, 2, 0), (20000, 8193, 5, 8),
    (3, 4096, 17, 1),
])
def test_sliced_wasserstein_at_the_tile_edges(na, nb, K, grid):
    print(f"sliced W na={na} nb={nb} K={K} grid={grid}", flush=True)
    rng = np.random.default_rng(na + nb)
    d = 3
    a, b = rng.normal(size=(1, d, na)), rng.normal(0.3, 1.2, size=(1, d, nb))
    if grid:  # ties
        a, b = np.round(a * grid) / grid, np.round(b * grid) / grid
    a, b = a.astype(np.float32), b.astype(np.float32)
    got = B.best_sliced_wasserstein(_ctx(d), _dev(a), _dev(b), K, 99)
    ref = OM.sliced_wasserstein(a, b, K, 99)
    assert abs(got - ref) <= 1e-9 * ref


@pytest.mark.parametrize("n,levels,d", [(1, 0, 2), (2, 0, 1), (5000, 3, 9), (70000, 0, 17),
                                        (40000, 5000, 2)])
def test_credible_limits_with_ties_and_small_sets(n, levels, d):
    print(f"credible n={n} levels={levels} d={d}", flush=True)
    rng = np.random.default_rng(n + levels)
    x = rng.normal(size=(1, d, n))
    if levels:
        x = np.round(x * levels / 4) / levels * 4
    x = x.astype(np.float32)
    for alpha in (0.1, 0.68, 0.999):
        lo, hi, _ = B.best_credible(_ctx(d), _dev(x), alpha)
        rlo, rhi = OM.credible_limits(x, alpha)
        np.testing.assert_allclose(lo, rlo, rtol=1e-12, atol=1e-12)
        np.testing.assert_allclose(hi, rhi, rtol=1e-12, atol=1e-12)


@pytest.mark.parametrize("T,d,N", [(2, 16, 40), (7, 17, 33), (5, 32, 70), (64, 1, 3)])
def test_rhat_off_the_vector_width(T, d, N):
    print(f"rhat T={T} d={d} N={N}", flush=True)
    rng = np.random.default_rng(T * d + N)
    x = (rng.normal(size=(T, d, N)) + 0.4 * rng.normal(size=(1, d, N))).astype(np.float32)
    got, ref = B.best_rhat(_ctx(d), _dev(x)), OM.rhat_minus_one(x)
    assert abs(got - ref) < 1e-9 * ref
