"""The tiled stencil kernels at the edges of their tiles, vectors and z chunks:
every variant, in both z-marching directions, gives the levels of the
one-thread-per-cell kernel bit for bit, and so does the automatic choice over a
whole sweep."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2201_06914_amd as P
from paper_2201_06914_amd import _lib
from gpu_util import say

pytestmark = pytest.mark.gpu


def _plan(shape, field, nt=8):
    return P.Plan(P.PlanSpec(3, shape, 12.5, 1e-3, nt, 1, 4500.0, 1e-3, 4500.0, field,
                             "f32" if field == "f32" else "f64", 1, 4, 1, 0))


def _m(plan, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    v = 1500.0 + 2500.0 * torch.rand(plan.N, generator=g, device="cuda", dtype=torch.float64)
    return (1.0 / v ** 2).to(plan.dtype)


# x: one vector, a cut vector of each length, whole tiles, one cell more; y: below,
# at and past a tile; z: fewer planes than the queue, whole and cut ring trips
@pytest.mark.parametrize("field", ["f32", "f64"])
@pytest.mark.parametrize("shape", [(3, 3, 4), (5, 9, 5), (13, 16, 64), (12, 17, 65), (19, 31, 66),
                                   (7, 33, 67), (25, 8, 128), (6, 70, 31), (41, 12, 131)])
def test_tiled_variants_equal_simple(shape, field):
    plan = _plan(shape, field)
    m, w = _m(plan, sum(shape)), plan.workspace()
    say(f"case: stencil variants {shape} {field}")
    for blocks in (1, 64, 100000):      # one chunk; some; chunks of four planes
        P.set_stencil_blocks(blocks)
        try:
            best = ctypes.c_int32()
            mism = (ctypes.c_int64 * 14)()
            code = _lib.load().rtm_autotune_stencil(
                plan.handle, ctypes.c_void_p(m.data_ptr()), ctypes.c_void_p(w.data_ptr()),
                w.numel(), 1, ctypes.byref(best), None, mism,
                ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        finally:
            P.set_stencil_blocks(0)
        assert code == 0
        assert list(mism) == [0] * 14, (shape, field, blocks, list(mism))


# either side of the automatic rule's cell threshold, whole and cut rows
@pytest.mark.parametrize("shape,field", [((40, 50, 99), "f32"), ((40, 50, 101), "f32"),
                                         ((64, 52, 76), "f32"), ((41, 52, 95), "f64")])
def test_automatic_choice_equals_simple(shape, field):
    plan = _plan(shape, field, nt=11)
    m = _m(plan, 3)
    q = torch.full((11, 1), 1e-3, device="cuda", dtype=plan.dtype)
    src = np.array([[shape[0] / 2, shape[1] / 2, shape[2] / 2]])
    say(f"case: automatic stencil {shape} {field}")
    got = P.rtm_forward_probe(plan, m, src, q, want_d=False, final=True)["final"]
    P.set_stencil_variant(0)
    try:
        ref = P.rtm_forward_probe(plan, m, src, q, want_d=False, final=True)["final"]
    finally:
        P.set_stencil_variant(-1)
    assert float(ref.abs().max()) > 0
    assert torch.equal(got, ref)


# 2D, several steps per launch: fewer cells than a tile, one column more than a
# tile, both tile heights; blocks that end on and off a launch's four steps
@pytest.mark.parametrize("shape,field,k", [((9, 1, 11), "f32", 3), ((16, 1, 33), "f64", 4),
                                           ((50, 1, 97), "f32", 7), ((17, 1, 32), "f64", 1),
                                           ((1060, 1, 260), "f64", 6), ((70, 1, 64), "f32", 2)])
def test_2d_steps_equal_single_steps(shape, field, k):
    nt = 11
    plan = P.Plan(P.PlanSpec(2, shape, 10.0, 1e-3, nt, 2, 4500.0, 1e-3, 4500.0, field,
                             "f32" if field == "f32" else "f64", 3, k, 2, 3))
    m = _m(plan, 3)
    q = torch.tensor([[1e-3, -2e-3]], device="cuda", dtype=plan.dtype).repeat(nt, 1)
    src = np.array([[shape[0] / 2, 0, shape[2] / 2], [shape[0] / 2 + 0.5, 0, shape[2] / 2 + 0.25]])
    rec = np.array([[3.0, 0, 4.5], [shape[0] / 2, 0, shape[2] / 2], [shape[0] - 1, 0, 0]])
    Z = torch.ones((nt, 3), device="cuda", dtype=torch.int8)
    say(f"case: 2D steps {shape} {field} k={k}")

    def run():
        f = P.rtm_forward_probe(plan, m, src, q, rec, Z, final=True)
        res = f["d"] + 1e-6
        b = P.rtm_adjoint_probe(plan, m, rec, res, Z, src_pos=src, want_qadj=True)
        return f["final"], f["d"], f["Ubar"], b["Vbar"], b["qadj"]
    got = run()
    P.set_stencil_variant(0)
    try:
        ref = run()
    finally:
        P.set_stencil_variant(-1)
    assert float(ref[0].abs().max()) > 0
    for x, y in zip(got, ref):
        assert torch.equal(x, y)
