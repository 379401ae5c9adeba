"""A batched window whose plane is 2 GiB or more, which the tiled kernel's
32-bit plane offsets do not reach, against the same shot by itself."""
import numpy as np
import pytest
import torch

import paper_2201_06914_amd as P
from gpu_util import say

pytestmark = pytest.mark.gpu


def test_batched_plane_beyond_tile_offsets():
    """One plane of 16416 x 32768 cells (2 GiB + 4 MiB): a source on the cell
    at byte 2^31 of the level, one at the grid's corner, and beside it an
    ordinary window of the same batch.  Bit for bit the single shots."""
    nt, k, r = 4, 2, 8
    shapes = [(1, 16416, 32768), (20, 18, 33)]
    specs, shots = [], []
    rng = np.random.default_rng(0)
    for i, shape in enumerate(shapes):
        src = np.array([[0, 16384, 0], [0, 0, 0], [0, shape[1] - 1, shape[2] - 1]],
                       dtype=float) if i == 0 else np.array([[9., 9., 9.]] * 3)
        rec = src[:2] + np.array([0.0, 1.0, 2.0])
        N = int(np.prod(shape))
        specs.append(P.PlanSpec(3, shape, 10.0, 1e-3, nt, 0, 2000.0, 1e-3, 2000.0, "f32", "bf16x2",
                                r, k, 3, 2))
        q = rng.standard_normal((nt, 3)).astype(np.float32)
        d = rng.standard_normal((nt, 2)).astype(np.float32)
        Z = rng.choice(np.array([-1, 1], dtype=np.int8), (nt, r))
        shots.append(dict(m=torch.full((N,), 2.5e-7, device="cuda"), src_pos=src,
                          q=torch.from_numpy(q).cuda(), rec_pos=rec,
                          d_obs=torch.from_numpy(d).cuda(), Z=torch.from_numpy(Z).cuda()))
    say(f"case: batch of {shapes}")
    outs, J = P.Batch(specs).fwi_gradient(shots)
    torch.cuda.synchronize()
    for i, (sp, sh) in enumerate(zip(specs, shots)):
        one = P.fwi_gradient(P.Plan(sp), sh["m"], sh["src_pos"], sh["q"], sh["rec_pos"],
                             sh["d_obs"], sh["Z"], fused=True)
        assert float(one["grad"].abs().max()) > 0
        for name in ("resid", "grad", "Ubar"):
            a, b = outs[i][name].reshape(-1), one[name].reshape(-1)
            assert all(torch.equal(x, y) for x, y in zip(a.split(1 << 28), b.split(1 << 28))), \
                (shapes[i], name)
        assert float(J[i].item()) == float(one["misfit"].item())
        del one
    del outs, shots
    torch.cuda.empty_cache()
