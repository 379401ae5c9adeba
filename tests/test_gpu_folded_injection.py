"""Injection folded into the step kernels against injection by a launch of its
own, bit for bit.  The step kernels take a point set whose cells' bounding box
is small against its point count; one more point far away, with zero values,
makes the box too large and changes nothing else."""
import numpy as np
import pytest
import torch

import paper_2201_06914_amd as P
from gpu_util import say

pytestmark = pytest.mark.gpu


def _points(kind, shape, rng):
    nz, ny, nx = shape
    two = ny == 1
    if kind == "one":
        p = np.array([[nz // 2, ny // 2, nx // 2]], dtype=float)
    elif kind == "plane":       # every cell of one plane, single entries of weight one
        y, x = np.meshgrid(np.arange(ny), np.arange(nx), indexing="ij")
        p = np.stack([np.full(y.size, 3.0), y.ravel(), x.ravel()], 1).astype(float)
    else:                       # off the grid, shared cells, one point twice
        p = rng.uniform(0, 1, (40, 3)) * [2.5, min(ny - 1, 6), min(nx - 1, 9)] + [2, 0, 0]
        p = np.concatenate([p, p[:1]])
    if two:
        p[:, 1] = 0.0
    return p


CASES = [((30, 26, 44), "f32", "one"), ((30, 26, 44), "f32", "plane"),
         ((31, 23, 45), "f32", "cloud"),        # one thread per cell
         ((64, 50, 70), "f32", "plane"), ((64, 50, 71), "f32", "cloud"),   # tiled
         ((64, 50, 72), "f32", "one"), ((60, 50, 71), "f64", "plane"), ((60, 50, 70), "f64", "cloud"),
         ((60, 1, 75), "f64", "cloud"), ((61, 1, 75), "f32", "plane")]


@pytest.mark.parametrize("shape,field,kind", CASES)
def test_folded_equals_launched(shape, field, kind):
    rng = np.random.default_rng(sum(shape))
    nt, two = 9, shape[1] == 1
    dt = torch.float32 if field == "f32" else torch.float64
    N = int(np.prod(shape))
    m = torch.from_numpy(1.0 / rng.uniform(1500, 3500, N) ** 2).to("cuda", dt)
    pos = _points(kind, shape, rng)
    vals = torch.from_numpy(rng.standard_normal((nt, pos.shape[0]))).to("cuda", dt)
    rec = np.array([[4.0, 0.0 if two else 2.5, 3.25]])
    far = np.array([[s - 1.0 for s in shape]])
    far[0, 1] = 0.0 if two else far[0, 1]
    say(f"case: folded injection {shape} {field} {kind} ({pos.shape[0]} points)")
    pr = "f64" if field == "f64" else "bf16x2"
    a = (2 if two else 3, shape, 12.5, 1e-3, nt, 3, 3500.0, 1e-3, 3500.0, field, pr, 2, 4)
    got = []
    for fold in (True, False):
        p = pos if fold else np.concatenate([pos, far, np.zeros((1, 3))])
        pad = torch.zeros((nt, p.shape[0] - pos.shape[0]), device="cuda", dtype=dt)
        v = torch.cat([vals, pad], 1).contiguous()
        plan = P.Plan(P.PlanSpec(*a, p.shape[0], 1))
        f = P.rtm_forward_probe(plan, m, p, v, rec, final=True)
        plan = P.Plan(P.PlanSpec(*a, 1, p.shape[0]))
        adj = P.rtm_adjoint_probe(plan, m, p, v, src_pos=rec, want_qadj=True)["qadj"]
        got.append((f["d"], f["final"], adj))
    assert float(got[0][1].abs().max()) > 0     # the levels; traces may see nothing yet
    for name, x, y in zip(("d", "final", "qadj"), *got):
        assert torch.equal(x, y), name


@pytest.mark.parametrize("shape", [(64, 50, 72), (64, 50, 71), (30, 26, 44)])
def test_folded_exact_gradient(shape):
    """The exact gradient's two epilogues: sources and receivers folded or not
    (the far points carry no signature and record zeros that d_obs repeats)."""
    rng = np.random.default_rng(5)
    nt = 9
    N = int(np.prod(shape))
    m = torch.from_numpy(1.0 / rng.uniform(1500, 3500, N) ** 2).to("cuda", torch.float32)
    src = _points("cloud", shape, rng)
    rec = _points("plane", shape, rng)
    q = torch.from_numpy(rng.standard_normal((nt, src.shape[0]))).to("cuda", torch.float32)
    d = torch.from_numpy(rng.standard_normal((nt, rec.shape[0]))).to("cuda", torch.float32)
    far = np.array([[s - 1.0 for s in shape], [0.0, 0.0, 0.0]])
    z = torch.zeros((nt, 2), device="cuda")
    say(f"case: folded injection, exact gradient {shape}")
    grads = []
    for fold in (True, False):
        s = src if fold else np.concatenate([src, far])
        r = rec if fold else np.concatenate([rec, far])
        a = (3, shape, 12.5, 1e-3, nt, 3, 3500.0, 1e-3, 3500.0, "f32", "bf16x2", 2, 4)
        plan = P.Plan(P.PlanSpec(*a, s.shape[0], r.shape[0]))
        qq = q if fold else torch.cat([q, z], 1).contiguous()
        dd = d if fold else torch.cat([d, z], 1).contiguous()
        if not fold:        # what the far receivers record, so that they inject zeros
            dd[:, -2:] = P.rtm_forward_probe(plan, m, s, qq, r)["d"][:, -2:]
        grads.append(P.fwi_gradient_exact(plan, m, s, qq, r, dd, checkpoint_every=4)["grad"])
    assert float(grads[0].abs().max()) > 0
    assert torch.equal(grads[0], grads[1])
