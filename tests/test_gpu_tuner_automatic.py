"""The tuners against the automatic choice: it is a candidate, in 2D it wins
(several steps per launch), and nothing else stays set."""
import ctypes
import json

import numpy as np
import pytest
import torch

import paper_2201_06914_amd as P
from gpu_kernels import kernels, named
from gpu_util import say
from paper_2201_06914_amd import _lib
from paper_2201_06914_amd.tune import autotune_batch

pytestmark = pytest.mark.gpu


def _plan(shape, field, k):
    return P.Plan(P.PlanSpec(3 if shape[1] > 1 else 2, shape, 10.0, 1e-3, 12, 2, 2000.0, 1e-3,
                             2000.0, field, "f64" if field == "f64" else "bf16x2", 1, k, 1, 0))


def _m(plan):
    return torch.full((plan.N,), 2.5e-7, device="cuda", dtype=plan.dtype)


@pytest.mark.parametrize("field,k", [("f32", 12), ("f64", 4)])
def test_2d_tuning_keeps_several_steps_per_launch(field, k, tmp_path):
    """221 x 221: the sweep takes four steps in a launch after tuning, directly
    and from the cache (us a step 1.9 and 2.3 against 3.4 and 3.5)."""
    say(f"case: tuning 2D {field} k {k}")
    plan = _plan((221, 1, 221), field, k)
    m, w, cache = _m(plan), plan.workspace(), str(tmp_path / "tune.json")
    best = ctypes.c_int32(7)
    code = _lib.load().rtm_autotune_stencil(
        plan.handle, ctypes.c_void_p(m.data_ptr()), ctypes.c_void_p(w.data_ptr()), w.numel(), 40,
        ctypes.byref(best), None, None, ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert code == 0 and best.value == -1
    run = lambda: P.rtm_forward_probe(plan, m, np.array([[110., 0., 110.]]),
                                      torch.ones((12, 1), device="cuda", dtype=plan.dtype),
                                      want_d=False)
    try:
        for cached in (False, True):
            res = P.autotune_stencil(plan, m, work=w, steps=40, cache=cache)
            assert res["cached"] == cached and res["best"] == -1, res
            assert res["us"][2048 if not cached else "2048"][-1] > 0
            assert P.api.get_stencil_variant() == -1 and P.api.get_stencil_blocks() == 2048
            assert named(kernels(run), "k_stencil2d_steps") == 3
    finally:
        P.set_stencil_variant(-1)
        P.set_stencil_blocks(0)
    assert all("tiles3" in key for key in json.load(open(cache)))


def test_tuning_times_the_automatic_choice_in_3d():
    """The pick is the fastest entry, the automatic choice's among them, and
    apply=False leaves the settings alone."""
    say("case: tuning 3D")
    plan = _plan((64, 60, 64), "f32", 4)
    P.set_stencil_variant(5)
    P.set_stencil_blocks(1024)
    try:
        res = P.autotune_stencil(plan, _m(plan), steps=20, apply=False, blocks=(1024, 4096))
        assert P.api.get_stencil_variant() == 5 and P.api.get_stencil_blocks() == 1024
        names = kernels(lambda: P.rtm_forward_probe(plan, _m(plan), np.array([[9., 9., 9.]]),
                                                    torch.ones((12, 1), device="cuda"), want_d=False))
        assert named(names, "k_stencil3d_tiled<float, 32, 32,") == 12
    finally:
        P.set_stencil_variant(-1)
        P.set_stencil_blocks(0)
    assert [len(res["us"][b]) for b in (1024, 4096, 2048)] == [14, 14, 1]
    assert res["us"][res["blocks"]][res["best"]] == min(min(u) for u in res["us"].values())
    assert res["us"][1024][11] == res["us"][1024][13] == res["us"][1024][12]


def test_batch_tuning_leaves_the_variant():
    say("case: batch tuning")
    shape, nt, r = (24, 22, 40), 32, 8
    sp = P.PlanSpec(3, shape, 10.0, 1e-3, nt, 2, 2000.0, 1e-3, 2000.0, "f32", "bf16x2", r, 16, 1, 1)
    N = int(np.prod(shape))
    sh = dict(m=torch.full((N,), 2.5e-7, device="cuda"), src_pos=np.array([[9., 9., 9.]]),
              q=torch.ones((nt, 1), device="cuda"), rec_pos=np.array([[4., 5., 6.]]),
              d_obs=torch.zeros((nt, 1), device="cuda"),
              Z=torch.ones((nt, r), dtype=torch.int8, device="cuda"))
    P.set_stencil_variant(0)
    try:
        res = autotune_batch([sp, sp], [sh, sh], steps=32, k_blocks=(16, 32))
        assert P.api.get_stencil_variant() == 0
    finally:
        P.set_stencil_variant(-1)
    assert sorted(res["ms_per_step"]) == sorted(f"{v}/{b}" for v in (1, 7)
                                                for b in (2048, 4096, 8192))
