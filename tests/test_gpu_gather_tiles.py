"""Offset volumes staged by whole 32-cell tiles: rows that start inside a tile,
fields on and off 16-byte boundaries, the last probe rows of a chunk, and
neighbouring rows that hold no numbers."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import dev, host, require_gpu, say

pytestmark = pytest.mark.gpu

import paper_2201_06914_amd as P  # noqa: E402


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _tile_major(rows, Npad):
    r, N = rows.shape
    out = np.zeros((Npad // 32, r, 32), dtype=rows.dtype)
    x = np.arange(N)
    for i in range(r):
        out[x // 32, i, x % 32] = rows[i]
    return out.ravel()


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("nx,r,nh,nfield", [
    (31, 8, 3, 1), (33, 9, 0, 2), (128, 4, 40, 1), (160, 13, 64, 1), (129, 16, 8, 2),
    (400, 3, 40, 1), (255, 12, 56, 1)])
def test_tiles_of_a_row(nx, r, nh, nfield, shift):
    shape = (3, 3, nx)
    plan = P.Plan(P.PlanSpec(3, shape, 10.0, 1e-3, 16, 1, 3000.0, 1e-3, 3000.0, "f32", "f32", r,
                             16, 1, 1))
    N = 9 * nx
    rng = np.random.default_rng(nx + r)
    F = rng.standard_normal((2, nfield, r, N)).astype(np.float32)
    bad = np.zeros(N, bool)
    bad[nx:2 * nx] = True        # one row of every second holds no numbers
    bad[5 * nx:6 * nx] = True
    F[:, :, :, bad] = np.nan
    dt = torch.float32
    ptr = []
    for k in range(2):
        flat = np.concatenate([_tile_major(F[k, f], plan.Npad) for f in range(nfield)])
        buf = torch.zeros(flat.size + shift, device="cuda", dtype=dt)
        buf[shift:] = dev(flat, dt)
        ptr.append(buf[shift:])
    out = torch.full((2 * nh + 1, N), 7.0, device="cuda", dtype=dt)
    G = host(P.rtm_offset_gathers(plan, ptr[0], ptr[1], nh, scale=1.0, nfield=nfield, out=out))
    torch.cuda.synchronize()
    Fz = np.where(bad, 0.0, F.astype(np.float64))
    G0 = sum(oracle.offset_gathers(Fz[0, f], Fz[1, f], shape, nh, 1.0) for f in range(nfield))
    # FP32 products and a sum of nfield r of them in any order
    mag = sum(oracle.offset_gathers(abs(Fz[0, f]), abs(Fz[1, f]), shape, nh, 1.0)
              for f in range(nfield))
    tol = (nfield * r + 1) * 2.0 ** -24 * 1.01
    d = abs(G - np.asarray(G0).reshape(G.shape))[:, ~bad]
    mag = np.asarray(mag).reshape(G.shape)[:, ~bad]
    say(f"  nx={nx} r={r} nh={nh}: worst {np.max(d / (mag + 1e-30)):.2e} of {tol:.2e}")
    assert np.all(d <= tol * mag)
