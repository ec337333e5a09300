"""The fused Adam update: after an epoch the packed weights the next pass uses are those of the
master parameters, in every precision.  A trainer created from the updated parameters packs them
with the stand-alone kernel; its minibatch gradient must be the running trainer's, bit for bit
(the same kernels on the same packed values), at shapes with and without hidden blocks and with
input components around the padding of 16."""
import numpy as np
import pytest
import torch

import paper_2606_04895_amd as B
from workloads.synth import xavier_mlp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp32", "fp16", "bf16"])
@pytest.mark.parametrize("d,width,nh", [(1, 128, 1), (16, 128, 2), (17, 256, 3)])
def test_updated_packs_match_a_fresh_pack(prec, d, width, nh):
    print(f"adam pack {prec} d={d} width={width} nh={nh}", flush=True)
    rng = np.random.default_rng(7)
    p = xavier_mlp(rng, d, width, nh)
    t = torch.tensor(rng.uniform(-1, 1, (96, d)).astype(np.float32), device="cuda")
    y = torch.tensor(rng.normal(size=96).astype(np.float32), device="cuda")
    perm = torch.tensor(rng.permutation(96).astype(np.int32), device="cuda")
    tr = B.Trainer(d, width, nh, p, precision=prec)
    tr.epoch(t, y, perm, 32, 1e-3, 1e-4, 0, 3)
    q = tr.params()
    assert np.all(q != p) or np.count_nonzero(q == p) < q.size // 100
    fresh = B.Trainer(d, width, nh, q, precision=prec)
    (l0, g0), (l1, g1) = tr.grad(t, y), fresh.grad(t, y)
    assert l0 == l1
    np.testing.assert_array_equal(g0, g1)
