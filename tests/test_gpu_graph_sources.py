"""More sources in turn than the library keeps graphs: each call drops the
oldest, whose replay may still be queued.  Every gradient is the eager one."""
import numpy as np
import pytest
import torch

import paper_2201_06914_amd as P
from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(60, 1, 70), (40, 44, 90)])
def test_more_sources_than_graphs(shape):
    nt, r, k, N = 64, 8, 16, int(np.prod(shape))
    rng = np.random.default_rng(2)
    say(f"case: graphs of twelve sources on {shape}")
    plan = P.Plan(P.PlanSpec(3 if shape[1] > 1 else 2, shape, 10.0, 1e-3, nt, 3, 2000.0, 1e-3,
                             2000.0, "f32", "bf16x2", r, k, 1, 9))
    m = torch.full((N,), 2.5e-7, device="cuda")
    q = torch.from_numpy(rng.standard_normal((nt, 1)).astype(np.float32)).cuda()
    d = torch.from_numpy(rng.standard_normal((nt, 9)).astype(np.float32)).cuda()
    Z = torch.from_numpy(rng.choice(np.array([-1, 1], np.int8), (nt, r))).cuda()
    rec = np.stack([np.full(9, 4.0), np.full(9, shape[1] // 2), 6.0 + np.arange(9)], 1)
    srcs = [np.array([[20.0, shape[1] // 2, 10.0 + 3 * i]]) for i in range(12)]
    work, bars = plan.workspace(), (plan.empty_bar(), None)

    def shots():                       # no wait between the calls
        return [P.fwi_gradient(plan, m, s, q, rec, d, Z, work=work, bars=bars, fused=True)["grad"]
                for s in srcs]
    want = shots()
    assert not torch.equal(want[0], want[1])
    P.set_graph(True)
    try:
        for _ in range(2):
            for a, b in zip(shots(), want):
                assert torch.equal(a, b)
            (torch.randn(1 << 20, device="cuda") * 2).sum().item()
    finally:
        P.set_graph(False)
