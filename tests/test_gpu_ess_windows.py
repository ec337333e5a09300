"""The ESS at the edges of its lag windows, time segments and chain blocks, against the oracle's FFT
autocovariances: records shorter than a window of 32 lags, one step around it, several windows
(chains of different means never let the pair sums turn negative) with several time segments, and
chain counts around the 64 of a workgroup.

Tolerance: FP64 sums of the same floats in another order; tau is a sum of at most T / 2 pair sums
of size O(1), each with a relative rounding of about T 2^-53 < 1e-12, so 1e-9 relative."""
import numpy as np
import pytest
import torch

import paper_2606_04895_amd as B
from oracle import ess as OE
from workloads import ar1_chains, small_problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,n,spread", [
    (4, 64, 0.0), (31, 65, 0.0), (32, 1, 0.0), (33, 63, 1.0), (64, 130, 1.0), (161, 64, 1.0),
    (513, 65, 1.0), (700, 3, 0.3), (1100, 64, 0.0),
])
def test_ess_matches_the_oracle_at_the_window_edges(T, n, spread):
    print(f"ess T={T} n={n} spread={spread}", flush=True)
    rng = np.random.default_rng(T * 100 + n)
    d = 2
    x = np.stack([ar1_chains(rng, r, n, T) for r in (0.9, -0.4)])
    x += spread * rng.normal(size=(d, n, 1)) + 3.0
    rec = torch.tensor(x.transpose(2, 0, 1).copy(), dtype=torch.float32, device="cuda")
    ctx = B.best_init(small_problem(d=d, width=128, n_hidden=1), n_chains=n, precision="fp32")
    e, f = B.best_ess(ctx, rec, flags=True)
    e2, f2 = B.best_ess_noalloc(ctx, rec, flags=True)
    np.testing.assert_array_equal(e, e2)
    np.testing.assert_array_equal(f, f2)
    _, ref, rf = OE.min_ess(rec.cpu().numpy().transpose(0, 2, 1))
    np.testing.assert_array_equal(f, rf)
    np.testing.assert_allclose(e, ref, rtol=1e-9)
    if spread == 1.0 and T > 32:
        assert np.all(f == B.A.BEST_ESS_UNTRUNCATED)
