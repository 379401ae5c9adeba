"""Which kernel a probe block runs, and its result against the sum of products
in 64 bits.  Probes that select one step each return the probed values
themselves (1 x value, nothing added), from which the reference is formed."""
import numpy as np
import pytest
import torch

import paper_2201_06914_amd as P
from gpu_kernels import kernels, named
from gpu_util import say
from paper_2201_06914_amd.autograd import _adjoint_image_fused

pytestmark = pytest.mark.gpu

SHAPE = (13, 22, 35)                       # 10010 cells: 312 whole tiles and 26 cells
# unit roundoff of a product's operand and of the sums
EPS = {"f64": (0.0, 2.0**-53), "f32": (0.0, 2.0**-24), "bf16x2": (2.0**-16, 2.0**-24),
       "bf16": (2.0**-8, 2.0**-24), "f16s": (2.0**-10, 2.0**-24)}


def _plan(probe, r, k, nt):
    return P.Plan(P.PlanSpec(3, SHAPE, 10.0, 1e-3, nt, 0, 2000.0, 1e-3, 2000.0,
                             "f64" if probe == "f64" else "f32", probe, r, k, 1, 1))


def _inputs(T, nt, r, rng):
    N = int(np.prod(SHAPE))
    return dict(m=torch.full((N,), 2.5e-7, device="cuda", dtype=T),
                src=np.array([[6., 11., 17.]]),
                q=torch.from_numpy(rng.standard_normal((nt, 1))).to("cuda", T),
                Z=torch.from_numpy(rng.choice(np.array([-1, 1], np.int8), (nt, r))).cuda())


ROUTES = [  # probe, r, k, kernel of the blocks
    ("f64", 1, 1, "k_probe_vec<double"), ("f64", 7, 8, "k_probe_vec<double"),
    ("f64", 8, 8, "k_probe_mfma_f64<1"), ("f64", 3, 9, "k_probe_mfma_f64<1"),
    ("f32", 1, 1, "k_probe_vec<float"), ("f32", 16, 12, "k_probe_vec<float"),
    ("f32", 17, 12, "k_probe_mfma_edge<1"), ("f32", 8, 16, "k_probe_mfma_fast<1"),
    ("f32", 40, 20, "k_probe_mfma_fast<2"), ("f32", 32, 50, "k_probe_mfma_edge<4"),
    ("f32", 32, 70, "k_probe_mfma_fast<8"), ("f32", 40, 70, "k_probe_mfma_edge<8"),
    ("bf16x2", 24, 20, "k_probe_mfma_fast<2"), ("bf16x2", 32, 50, "k_probe_mfma_fast<4"),
    ("bf16x2", 40, 50, "k_probe_mfma_edge<4"), ("bf16x2", 8, 70, "k_probe_mfma_fast<8"),
    ("bf16x2", 96, 70, "k_probe_mfma_edge<8"), ("bf16x2", 64, 64, "k_probe_mfma_fast<4"),
    ("f16s", 40, 50, "k_probe_mfma_fast<4"), ("f16s", 96, 70, "k_probe_mfma_fast<8"),
    ("bf16", 12, 16, "k_probe_mfma_edge<1"), ("bf16", 40, 50, "k_probe_mfma_edge<4")]


@pytest.mark.parametrize("probe,r,k,kernel", ROUTES)
def test_update_block_route(probe, r, k, kernel):
    say(f"case: {probe} r {r} k {k}")
    nt, rng = 2 * k, np.random.default_rng(4)
    T = torch.float64 if probe == "f64" else torch.float32
    x = _inputs(T, nt, r, rng)
    plan = _plan(probe, r, k, nt)
    run = lambda: P.rtm_forward_probe(plan, x["m"], x["src"], x["q"], Z=x["Z"], want_d=False)["Ubar"]
    names = kernels(run)
    # every block's whole tiles by that kernel (the others only beside it, for the last cells)
    assert named(names, kernel) == 2, names
    assert named(names, "k_queue_reset") == (2 if (probe, r, k) == ("bf16x2", 64, 64) else 0), names
    # the probed values: real probes of the field's type, one step each
    sel = "f64" if probe == "f64" else "f32"
    S = P.rtm_forward_probe(_plan(sel, nt, k, nt), x["m"], x["src"], x["q"],
                            Z=torch.eye(nt, device="cuda", dtype=T), want_d=False)["Ubar"]
    S = S.double().permute(1, 0, 2).reshape(nt, -1)
    got = run().double().permute(1, 0, 2).reshape(r, -1)
    want = x["Z"].double().t() @ S
    op, acc = EPS[probe]
    size = S.abs().sum(0)                              # |Z|^T |S|
    if probe == "f16s":                                # a chunk's scale is its tile's largest value
        tile = S.reshape(nt, -1, 32).abs().amax((0, 2)).repeat_interleave(32)
        size = torch.maximum(size, nt * tile)
    bound = (op + (nt + 2) * acc) * size
    N = x["m"].numel()
    assert float(want.abs().max()) > 0
    assert bool(((got - want).abs() <= bound)[:, :N].all())
    assert float(got[:, N:].abs().max()) == 0          # padding cells


FUSED = [("bf16x2", 32, 12, "k_probe_mfma_edge<1"), ("bf16x2", 32, 20, "k_probe_mfma_fast<2"), ("bf16x2", 96, 20, "k_probe_mfma_fast<2"),
         ("bf16x2", 32, 50, "k_probe_mfma_edge<4"), ("bf16x2", 32, 70, "k_probe_mfma_fast<8"),
         ("bf16x2", 64, 70, "k_probe_mfma_fast<8"), ("f16s", 64, 70, "k_probe_mfma_edge<8"),
         ("bf16x2", 96, 70, "k_probe_mfma_edge<8"), ("f16s", 96, 50, "k_probe_mfma_edge<4"),
         ("bf16", 32, 20, "k_probe_mfma_fast<2"), ("bf16", 96, 50, "k_probe_mfma_fast<4")]


@pytest.mark.parametrize("probe,r,k,kernel", FUSED)
def test_fused_block_route(probe, r, k, kernel):
    """Fused imaging against the imaging condition on the two fields (their
    operands are rounded alike; 2 x 2^-24 a product and sum, r nt terms)."""
    say(f"case: fused {probe} r {r} k {k}")
    nt, rng = 2 * k, np.random.default_rng(4)
    x = _inputs(torch.float32, nt, r, rng)
    plan = _plan(probe, r, k, nt)
    rec = np.array([[5., 9., 14.]])
    res = torch.from_numpy(rng.standard_normal((nt, 1)).astype(np.float32)).cuda()
    U = P.rtm_forward_probe(plan, x["m"], x["src"], x["q"], Z=x["Z"], want_d=False)["Ubar"]
    V = P.rtm_adjoint_probe(plan, x["m"], rec, res, Z=x["Z"])["Vbar"]
    run = lambda: _adjoint_image_fused(plan, x["m"], rec, res, x["Z"], U)
    names = kernels(run)
    assert named(names, kernel) == 2, names
    N = x["m"].numel()
    rows = lambda F: F.double().permute(1, 0, 2).reshape(r, -1)[:, :N]
    # the adjoint's probed values, for the size of the sums
    S = P.rtm_adjoint_probe(_plan("f32", nt, k, nt), x["m"], rec, res,
                            Z=torch.eye(nt, device="cuda"))["Vbar"]
    S = S.double().permute(1, 0, 2).reshape(nt, -1)[:, :N].abs().sum(0)
    want = (rows(U) * rows(V)).sum(0)
    size = rows(U).abs().sum(0) * S
    got = -r * run().double().reshape(-1)          # the call's scale is -1 / r
    assert float(want.abs().max()) > 0
    assert bool(((got - want).abs() <= 2.0**-23 * (nt + r + 4) * size).all())


@pytest.mark.parametrize("probe,r,k,fused", [("bf16x2", 128, 16, False), ("bf16x2", 64, 32, False),
                                             ("bf16", 128, 64, True), ("f16s", 64, 16, True)])
def test_hint_off_keeps_the_kernel(probe, r, k, fused):
    """rtm_set_probe_nt(0): the wide fast kernels with ordinary loads and
    stores, not another kernel; the same bits."""
    say(f"case: no hint, {probe} r {r} k {k}")
    nt, rng = 2 * k, np.random.default_rng(4)
    x = _inputs(torch.float32, nt, r, rng)
    plan = _plan(probe, r, k, nt)
    rec = np.array([[5., 9., 14.]])
    d = torch.from_numpy(rng.standard_normal((nt, 1)).astype(np.float32)).cuda()
    bars = (plan.empty_bar(), None if fused else plan.empty_bar())
    run = lambda: P.fwi_gradient(plan, x["m"], x["src"], x["q"], rec, d, x["Z"], bars=bars,
                                 fused=fused)
    out = []
    try:
        for on in (True, False):
            P.set_probe_nt(on)
            names = kernels(run)
            o = run()
            out.append((o["Ubar"].clone(), o["grad"]))
            assert named(names, "k_probe_mfma_fast") == 4, names
            hint = {k_.rstrip(">").split(", ")[-1] for k_ in names if "mfma_fast" in k_}
            assert hint == {"true" if on else "false"}, names
    finally:
        P.set_probe_nt(True)
    assert float(out[0][1].abs().max()) > 0
    assert torch.equal(out[0][0], out[1][0]) and torch.equal(out[0][1], out[1][1])
