"""The injection tables group entries by cell whatever the order of the points:
spreads off the grid, in rows and shuffled, over spans of cells below 2^11,
below 2^22 and beyond (one, two and three passes of the sort)."""
import numpy as np
import pytest
import torch

import paper_2201_06914_amd as P
from gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(9, 10, 12), (40, 50, 60), (170, 160, 180)])
def test_points_in_any_order(shape):
    rng = np.random.default_rng(1)
    step = 3 if shape[0] < 100 else 23
    g = np.stack(np.meshgrid(*[np.arange(0, n - 1, step) for n in shape], indexing="ij"), -1)
    pos = g.reshape(-1, 3) + [0.25, 0.5, 0.375]          # no two points share a cell
    n, nt, N = pos.shape[0], 3, int(np.prod(shape))
    span = int(np.ravel_multi_index(tuple(g[-1, -1, -1] + 1), shape))
    say(f"case: {n} points over {span} cells")
    q = torch.from_numpy(rng.standard_normal((nt, n)).astype(np.float32)).cuda()
    m = torch.full((N,), 2.5e-7, device="cuda")
    plan = P.Plan(P.PlanSpec(3, shape, 10.0, 1e-3, nt, 0, 2000.0, 1e-3, 2000.0, "f32", "bf16x2", 1,
                             2, n, 0))
    perm = rng.permutation(n)
    outs = [P.rtm_forward_probe(plan, m, pos[i], q[:, torch.from_numpy(i).cuda()].contiguous(),
                                want_d=False, final=True)["final"]
            for i in (np.arange(n), perm, np.arange(n)[::-1].copy())]
    # the first step leaves weight x value x dt^2 / m on each point's corners
    one = P.Plan(P.PlanSpec(3, shape, 10.0, 1e-3, 1, 0, 2000.0, 1e-3, 2000.0, "f32", "bf16x2", 1,
                            2, n, 0))
    u1 = P.rtm_forward_probe(one, m, pos[perm], q[:1, torch.from_numpy(perm).cuda()].contiguous(),
                             want_d=False, final=True)["final"][0].double().cpu().numpy()
    want = np.zeros(shape)
    for dz in (0, 1):
        for dy in (0, 1):
            for dx in (0, 1):
                w = (.25 if dz else .75) * .5 * (.375 if dx else .625)
                c = pos.astype(int) + [dz, dy, dx]
                want[tuple(c.T)] = w * q[0].double().cpu().numpy() * 1e-6 / np.float32(2.5e-7)
    assert np.abs(u1 - want.ravel()).max() <= 2.0**-21 * np.abs(want).max()
    assert float(outs[0].abs().max()) > 0
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
