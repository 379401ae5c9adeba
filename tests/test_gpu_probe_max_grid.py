"""The probe kernels' launch at the largest grids a plan takes (below 2^31
cells): one workgroup per four tiles would be 2^32 work items."""
import numpy as np
import pytest
import torch

import paper_2201_06914_amd as P
from gpu_util import say

pytestmark = pytest.mark.gpu


def test_probe_launch_at_2_31_cells():
    """126 x 341 x 49981 = 2^31 - 2 cells, one block of two steps, the source
    on the last cell: the compressed field there is Z^T u_tt of the returned
    levels, to the operand's 16 bits (two products)."""
    shape, nt, r, dt = (126, 341, 49981), 2, 8, 1e-3
    N = int(np.prod(shape))
    assert N == 2**31 - 2
    say(f"case: forward probe at {shape}")
    plan = P.Plan(P.PlanSpec(3, shape, 10.0, dt, nt, 0, 2000.0, 1e-3, 2000.0, "f32", "bf16x2", r, 2,
                             1, 0))
    m = torch.full((N,), 2.5e-7, device="cuda")
    q = torch.tensor([[1.0], [-0.5]], device="cuda")
    Z = torch.tensor([[1] * 8, [1, -1] * 4], dtype=torch.int8, device="cuda")
    out = P.rtm_forward_probe(plan, m, np.array([[s - 1.0 for s in shape]]), q, Z=Z, want_d=False,
                              final=True)
    u2, u1 = (out["final"][i, -64:].double() for i in range(2))
    utt = torch.stack([u1, u2 - 2 * u1]) / dt**2
    want = Z.double().t() @ utt                                   # [r][64]
    tile = (N - 64) // 32
    i = torch.arange(N - 64, N, device="cuda")
    got = out["Ubar"][tile:].double()[(i // 32 - tile), :, i % 32].t()
    assert float(u1.abs().max()) > 0
    bound = 2.0**-14 * utt.abs().sum(0) + 2.0**-22 * (4 * u1.abs() + u2.abs()) / dt**2
    assert bool(((got - want).abs() <= bound).all())
    del out, m, u1, u2, got
    torch.cuda.empty_cache()
