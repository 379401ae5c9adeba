"""Which point sets the step kernels take and which inject with a launch of
their own, and that both give the same levels bit for bit: one more point far
away, with zero values, makes a set's box too large for the step."""
import numpy as np
import pytest
import torch

import paper_2201_06914_amd as P
from gpu_kernels import kernels, named
from gpu_util import say

pytestmark = pytest.mark.gpu


def _set(kind, shape):
    nz, ny, nx = shape
    z, y, x = np.arange(1.0, nz - 1), np.arange(0.0, ny - 1, 2), np.arange(0.0, nx - 1, 2)
    if kind.startswith("surface"):
        p = np.stack(np.meshgrid([3.0], y, x, indexing="ij"), -1).reshape(-1, 3)
    elif kind.startswith("dense"):                        # between all cells of a row
        y, x = np.arange(0.0, ny - 1), np.arange(0.0, nx - 1)
        p = np.stack(np.meshgrid([3.0], y, x, indexing="ij"), -1).reshape(-1, 3) - [0, 0.25, 0]
    elif kind.startswith("wall"):
        p = np.stack(np.meshgrid(z, y, [5.0], indexing="ij"), -1).reshape(-1, 3)
    elif kind.startswith("column"):
        p = np.stack([z, np.full(z.size, ny // 3), np.full(z.size, 5.0)], 1)
    else:                                                 # many points in one cell's corners
        p = np.tile([[3.0, ny // 2, 5.0]], (6, 1))
    if kind.endswith("off"):
        p = p + [0.5, 0.25 if ny > 1 else 0.0, 0.375]
    return np.minimum(p, np.array(shape) - 1.0)


SMALL, CACHED, STREAM = (30, 26, 44), (64, 50, 72), (200, 452, 452)
FOLDED = [(SMALL, "f32", k) for k in ("surface", "surface off", "wall off", "column off", "pile off")]
FOLDED += [(CACHED, f, k) for f in ("f32", "f64") for k in ("surface", "surface off", "column")]
FOLDED += [(STREAM, "f32", "surface"), (CACHED, "f64", "dense off")]
FOLDED += [((90, 1, 80), f, k) for f in ("f32", "f64") for k in ("column off", "pile off")]
LAUNCHED = [(CACHED, f, k) for f in ("f32", "f64") for k in ("wall", "wall off", "column off",
                                                              "pile off")]
LAUNCHED += [(CACHED, "f32", "dense off")]
LAUNCHED += [(STREAM, "f32", k) for k in ("surface off", "column", "wall")]
LAUNCHED += [((520, 1, 500), "f64", "pile off")]


@pytest.mark.parametrize("shape,field,kind,folded",
                         [c + (True,) for c in FOLDED] + [c + (False,) for c in LAUNCHED])
def test_injection_route(shape, field, kind, folded):
    nt, N = 5, int(np.prod(shape))
    T = torch.float32 if field == "f32" else torch.float64
    rng = np.random.default_rng(7)
    pos = _set(kind, shape)
    say(f"case: {kind} on {shape} {field}, {pos.shape[0]} points")
    m = torch.from_numpy(1.0 / rng.uniform(1500, 3500, N) ** 2).to("cuda", T)
    q = torch.from_numpy(rng.standard_normal((nt, pos.shape[0]))).to("cuda", T)
    ends = np.array([[s - 1.0 for s in shape], [0.0, 0.0, 0.0]])
    out = []
    for far in (False, True):
        p = np.concatenate([pos, ends]) if far else pos
        v = torch.cat([q, torch.zeros((nt, 2), device="cuda", dtype=T)], 1) if far else q
        plan = P.Plan(P.PlanSpec(3 if shape[1] > 1 else 2, shape, 10.0, 1e-3, nt, 0, 3500.0, 1e-3,
                                 3500.0, field, "f64" if field == "f64" else "bf16x2", 1, 4,
                                 p.shape[0], 0))
        v = v.contiguous()
        run = lambda: P.rtm_forward_probe(plan, m, p, v, want_d=False, final=True)["final"]
        out.append(run())
        n = named(kernels(run), "k_inject")
        assert n == (0 if folded and not far else nt), (far, n)
    assert float(out[0].abs().max()) > 0
    assert torch.equal(out[0], out[1])
