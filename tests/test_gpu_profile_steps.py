"""rtm_profile_read counts steps, also where one 2D launch covers several."""
import numpy as np
import pytest
import torch

import paper_2201_06914_amd as P
from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,k,stride,want", [
    ((60, 1, 70), 32, 1, 70), ((60, 1, 70), 32, 50, 8),     # steps 0 and 50: launches of four
    ((60, 1, 70), 5, 7, 34),   # launches of 4 + 1: ten hold a multiple of 7, eight of them four steps
    ((20, 22, 24), 32, 1, 70), ((20, 22, 24), 32, 50, 2)])
def test_stencil_count_is_steps(shape, k, stride, want):
    say(f"case: {shape} k {k} stride {stride}")
    nt, N = 70, int(np.prod(shape))
    launches = []                                            # steps of each launch
    for b in range(0, nt, k):
        n = min(k, nt - b)
        launches += [1] * n if shape[1] > 1 else [4] * (n // 4) + [n % 4] * (n % 4 > 0)
    starts = np.concatenate([[0], np.cumsum(launches)[:-1]])
    assert want == sum(n for s, n in zip(starts, launches)
                       if any((s + i) % stride == 0 for i in range(n)))
    plan = P.Plan(P.PlanSpec(3 if shape[1] > 1 else 2, shape, 10.0, 1e-3, nt, 0, 2000.0, 1e-3,
                             2000.0, "f32", "bf16x2", 1, k, 1, 0))
    m = torch.full((N,), 2.5e-7, device="cuda")
    q = torch.ones((nt, 1), device="cuda")
    P.profile_read("stencil")
    P.profile_enable(stride)
    try:
        P.rtm_forward_probe(plan, m, np.array([[s // 2 for s in shape]], dtype=float), q,
                            want_d=False)
    finally:
        P.profile_enable(0)
    ms, n = P.profile_read("stencil")
    assert n == want and ms > 0
