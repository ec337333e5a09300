"""Within-chain variance of chains that start far from where they settle (the first draw of a burn-in):
the ESS against the same estimator in extended precision.

Tolerance: two passes over T values carry a relative rounding of a few sqrt(T) 2^-53 (3e-13 for T =
200000) in W and in the lag sums, and tau is a short sum of their ratios: 1e-11 relative.  Squares about
the first value, reduced by S1^2 / T, carry T 2^-53 times the number of equal roundings instead."""
import numpy as np
import pytest
import torch

import paper_2606_04895_amd as B
from workloads import small_problem

pytestmark = pytest.mark.gpu


def _ess(x):
    """One chain's ESS (Geyer's initial monotone sequence) in extended precision."""
    x = x.astype(np.longdouble)
    T = len(x)
    y = x - x.mean()
    w = (y * y).sum() / (T - 1)
    var = (T - 1) / np.longdouble(T) * w
    sums = []
    for k in range(T // 2):
        rho = [np.longdouble(1) if t == 0 else 1 - (w - (y[:T - t] * y[t:]).sum() / T) / var
               for t in (2 * k, 2 * k + 1)]
        p = rho[0] + rho[1]
        if not p > 0:
            break
        sums.append(min(p, sums[-1]) if sums else p)
    return float(T / max(-1 + 2 * sum(sums), 1 / np.log10(np.longdouble(T))))


@pytest.mark.parametrize("T", [17, 255, 4097, 200003])
@pytest.mark.parametrize("far", [0.0, 1.0e3])
def test_ess_of_chains_that_start_far_out(T, far):
    print(f"ess outlier T={T} far={far}", flush=True)
    rng = np.random.default_rng(T)
    n = 3
    x = rng.normal(size=(T, 1, n)).astype(np.float32) * np.float32(0.01) + np.float32(5.0)
    x[:, 0, :] += (far * 0.8 ** np.arange(T))[:, None].astype(np.float32)
    for c in range(n):  # one chain per record: the chains' errors do not average out
        ctx = B.best_init(small_problem(d=1, width=128, n_hidden=1), n_chains=1, precision="fp32")
        rec = torch.tensor(x[:, :, c:c + 1].copy(), device="cuda")
        e, _ = B.best_ess(ctx, rec, flags=True)
        e2, _ = B.best_ess_noalloc(ctx, rec, flags=True)
        assert e[0] == e2[0]
        np.testing.assert_allclose(e[0], _ess(x[:, 0, c]), rtol=1e-11)
