"""Which kernel the automatic choice runs a step with, and that its levels are
the one-thread-per-cell kernel's bit for bit."""
import numpy as np
import pytest
import torch

import paper_2201_06914_amd as P
from gpu_kernels import kernels, named
from gpu_util import say

pytestmark = pytest.mark.gpu


def _levels(shape, field, nt=5, k=4):
    T = torch.float32 if field == "f32" else torch.float64
    rng = np.random.default_rng(3)
    N = int(np.prod(shape))
    plan = P.Plan(P.PlanSpec(3 if shape[1] > 1 else 2, shape, 10.0, 1e-3, nt, 0, 3500.0, 1e-3,
                             3500.0, field, "f64" if field == "f64" else "bf16x2", 1, k, 1, 0))
    m = torch.from_numpy(1.0 / rng.uniform(1500, 3500, N) ** 2).to("cuda", T)
    q = torch.from_numpy(rng.standard_normal((nt, 1))).to("cuda", T)
    src = np.array([[s // 2 for s in shape]], dtype=float)
    return lambda: P.rtm_forward_probe(plan, m, src, q, want_d=False, final=True)["final"]


@pytest.mark.parametrize("field", ["f32", "f64"])
@pytest.mark.parametrize("shape,tiled", [((300, 250, 3), False), ((60, 700, 12), False),
                                         ((500, 301, 1), False), ((400, 24, 16), None),
                                         ((100, 100, 20), True), ((60, 50, 70), True)])
def test_thin_grids_run_a_thread_per_cell(shape, tiled, field):
    """3D grids whose planes fill less than a fifth of the lanes of the tiles
    over them (64 x 16 cells, FP64 64 x 8: 24 x 16 cells fill 19 % and 25 %)."""
    if tiled is None:
        tiled = field == "f64"
    say(f"case: {shape} {field}")
    run = _levels(shape, field)
    names = kernels(run)
    got = run()
    P.set_stencil_variant(0)
    try:
        assert torch.equal(got, run())
    finally:
        P.set_stencil_variant(-1)
    assert (named(names, "k_stencil3d_tiled") == 5) == tiled, names
    assert (named(names, "k_stencil_simple") == 5) != tiled, names


# (grid, steps per block, launches of four, three, two and one steps by k_stencil2d_steps,
# launches of one step by a thread per cell); 9 steps
@pytest.mark.parametrize("field,shape,k,multi,simple", [
    ("f32", (120, 1, 130), 1, 9, 0), ("f64", (120, 1, 130), 1, 9, 0),
    ("f32", (300, 1, 310), 1, 0, 9), ("f64", (300, 1, 310), 2, 4, 1),
    ("f32", (300, 1, 310), 5, 2, 1),                    # 4 + 1, 4
    ("f32", (1010, 1, 1000), 2, 0, 9), ("f64", (520, 1, 500), 2, 0, 9),
    ("f32", (1010, 1, 1000), 3, 3, 0), ("f32", (2010, 1, 2000), 3, 0, 9),
    ("f32", (2010, 1, 2000), 4, 2, 1), ("f32", (4010, 1, 4000), 4, 0, 9),
    ("f64", (1250, 1, 1500), 3, 3, 0), ("f64", (1450, 1, 1400), 4, 0, 9)])
def test_2d_steps_per_launch(field, shape, k, multi, simple):
    """2D launches of several steps only where they beat a launch per step."""
    say(f"case: {shape} {field} k {k}")
    run = _levels(shape, field, nt=9, k=k)
    names = kernels(run)
    got = run()
    P.set_stencil_variant(0)
    try:
        assert torch.equal(got, run())
    finally:
        P.set_stencil_variant(-1)
    assert named(names, "k_stencil2d_steps") == multi, names
    assert named(names, "k_stencil_simple") == simple, names


@pytest.mark.parametrize("variant,kernel", [(9, "float, 64, 16, 2, true"), (10, "float, 64, 8, 1, true"),
                                            (11, "float, 128, 8, 1, true"),
                                            (12, "float, 128, 8, 1, true"),
                                            (13, "float, 128, 8, 1, true")])
def test_ids_of_the_streaming_tiles(variant, kernel):
    """Ids 11 and 13 run the 128 x 8 non-temporal tiles."""
    say(f"case: variant {variant}")
    run = _levels((40, 37, 70), "f32")
    want = run()
    P.set_stencil_variant(variant)
    try:
        names = kernels(run)
        assert named(names, f"k_stencil3d_tiled<{kernel},") == 5, names
        assert torch.equal(run(), want)
    finally:
        P.set_stencil_variant(-1)
