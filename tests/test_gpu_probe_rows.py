"""The probe GEMM at the edges of its row groups and step chunks: the kernels
chosen from r and the block length equal the masked kernel bit for bit, the
FP32 operand's sums stay within FP32 rounding of the FP64 sums of the same
levels, and the padding cells of a compressed field are zeros."""
import numpy as np
import pytest
import torch

import paper_2201_06914_amd as P
from gpu_util import say

pytestmark = pytest.mark.gpu
SHAPE = (9, 10, 17)     # 1530 cells: 47 whole 32-cell tiles and one of 26 cells
N = int(np.prod(SHAPE))


def _run(r, k, nt, probe, real=False, what="u"):
    field = "f64" if probe == "f64" else "f32"
    dt = torch.float64 if probe == "f64" else torch.float32
    rng = np.random.default_rng(r * 1000 + k)
    m = torch.from_numpy(1.0 / rng.uniform(1500, 3500, N) ** 2).to("cuda", dt)
    q = torch.from_numpy(rng.standard_normal((nt, 1))).to("cuda", dt)
    Z = (torch.from_numpy(rng.standard_normal((nt, r))).to("cuda", dt) if real else
         torch.from_numpy(rng.integers(0, 2, (nt, r)).astype(np.int8) * 2 - 1).cuda())
    cells = np.stack(np.meshgrid(*[np.arange(s) for s in SHAPE], indexing="ij"), -1).reshape(-1, 3)
    plan = P.Plan(P.PlanSpec(3, SHAPE, 12.5, 1e-3, nt, 2, 3500.0, 1e-3, 3500.0, field, probe, r, k,
                             1, N))
    o = P.rtm_forward_probe(plan, m, np.array([[4.0, 5.0, 8.0]]), q, cells.astype(float), Z, what=what)
    return plan, o["d"], o["Ubar"], Z


# r: below, at and past a group of 8, one to four row tiles; k: a cut chunk, one,
# two, four and eight chunks; nt: a short last block
@pytest.mark.parametrize("probe,real", [("f32", False), ("f32", True), ("bf16x2", False),
                                        ("bf16x2", True), ("f16s", False)])
@pytest.mark.parametrize("r,k,nt", [(7, 16, 21), (8, 16, 35), (24, 20, 45), (32, 32, 70),
                                    (40, 64, 90), (48, 32, 64), (96, 128, 150), (128, 32, 41)])
def test_rows_and_chunks(r, k, nt, probe, real):
    say(f"case: probe rows r={r} k={k} nt={nt} {probe} {'real' if real else '+-1'}")
    for what in ("u", "utt"):
        plan, d, U, Z = _run(r, k, nt, probe, real, what)
        P.set_probe_nt(False)
        try:
            ref = _run(r, k, nt, probe, real, what)[2]
        finally:
            P.set_probe_nt(True)
        assert torch.equal(U, ref), what
        pad = U.view(-1, r, 32)[-1, :, N % 32:]
        assert torch.equal(pad, torch.zeros_like(pad))
        if probe == "f32" and what == "u":
            h = torch.zeros((nt, N), device="cuda", dtype=torch.float64)
            h[1:] = d.double()[:-1]                       # d[n] = u^{n+1} at every cell
            zt = Z.double().t()
            want = zt @ h
            # nt FP32 additions of products rounded once: nt ulps of the sum of magnitudes
            bound = nt * 2.0 ** -23 * (zt.abs() @ h.abs())
            err = (P.rtm_bar_to_rows(plan, U).double() - want).abs()
            assert bool((err <= bound + 1e-300).all())


# FP64: row tiles of 16 (below, at, past one; many), chunks of 16 steps (cut, one
# to eight), and the vector kernel where the operand exceeds LDS
@pytest.mark.parametrize("real", [False, True])
@pytest.mark.parametrize("r,k,nt", [(1, 5, 12), (16, 16, 40), (17, 20, 45), (33, 64, 70),
                                    (64, 128, 150), (48, 130, 140), (128, 32, 41), (260, 32, 33)])
def test_f64_rows_and_chunks(r, k, nt, real):
    say(f"case: FP64 probe rows r={r} k={k} nt={nt} {'real' if real else '+-1'}")
    plan, d, U, Z = _run(r, k, nt, "f64", real, "u")
    h = torch.zeros((nt, N), device="cuda", dtype=torch.float64)
    h[1:] = d[:-1]
    zt = Z.double().t()
    bound = 2 * nt * 2.0 ** -52 * (zt.abs() @ h.abs())    # both sums round
    assert bool(((P.rtm_bar_to_rows(plan, U) - zt @ h).abs() <= bound + 1e-300).all())
    pad = U.view(-1, r, 32)[-1, :, N % 32:]
    assert torch.equal(pad, torch.zeros_like(pad))
    plan, d, U, Z = _run(r, k, nt, "f64", real, "utt")
    h = torch.zeros((nt + 1, N), device="cuda", dtype=torch.float64)
    h[1:] = d
    um = torch.cat([torch.zeros_like(h[:1]), h[:-2]])
    utt = ((h[1:] - 2.0 * h[:-1]) + um) * 1e6
    bound = 4 * nt * 2.0 ** -52 * (zt.abs() @ (h[1:].abs() + 2.0 * h[:-1].abs() + um.abs())) * 1e6
    assert bool(((P.rtm_bar_to_rows(plan, U) - zt @ utt).abs() <= bound + 1e-300).all())
