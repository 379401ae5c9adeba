"""Grids whose levels stream from HBM and whose rows are no multiple of the
vector: the automatic choice of the tile (128 x 8 cells where that covers the
row as tightly as 64-cell tiles, two rows per thread elsewhere; batches that
take 128 x 8 tiles) changes no bit."""
import numpy as np
import pytest
import torch

import paper_2201_06914_amd as P
from gpu_util import say

pytestmark = pytest.mark.gpu


def _spec(shape, nt, nrec, r=1):
    return P.PlanSpec(3, shape, 12.5, 1e-3, nt, 10, 4500.0, 1e-3, 4500.0, "f32", "bf16x2", r, 4, 1,
                      nrec)


def _shot(shape, nt, seed, r=1):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    n = shape[0] * shape[1] * shape[2]
    m = 1.0 / (1500.0 + 2500.0 * torch.rand(n, generator=g, device="cuda")) ** 2
    q = torch.full((nt, 1), 1e-3, device="cuda")
    src = np.array([[shape[0] / 2, shape[1] / 2, shape[2] / 2 + 0.5]])
    rec = src + np.array([[1.0, 0.0, 0.0], [0.0, 1.5, 1.0]])[:, None].reshape(2, 3)
    Z = (2 * torch.randint(0, 2, (nt, r), generator=g, device="cuda") - 1).to(torch.int8)
    return dict(m=m, src_pos=src, q=q, rec_pos=rec, Z=Z,
                d_obs=torch.zeros((nt, 2), device="cuda"))


@pytest.mark.parametrize("shape", [(256, 320, 501), (251, 411, 393), (300, 1050, 129)])
def test_streaming_cut_rows_equal_simple(shape):
    nt = 5
    plan = P.Plan(_spec(shape, nt, 0))
    s = _shot(shape, nt, sum(shape))
    say(f"case: streaming cut rows {shape}")

    def run():
        return P.rtm_forward_probe(plan, s["m"], s["src_pos"], s["q"], want_d=False,
                                   final=True)["final"]
    got = run()
    P.set_stencil_variant(0)
    try:
        ref = run()
    finally:
        P.set_stencil_variant(-1)
    assert float(ref.abs().max()) > 0
    assert torch.equal(got, ref)


@pytest.mark.parametrize("shapes", [[(128, 350, 379), (150, 397, 500)], [(24, 39, 130), (340, 401, 353)]])
def test_streaming_batch_equals_single_shots(shapes):
    nt, r = 8, 4
    specs = [_spec(s, nt, 2, r) for s in shapes]
    shots = [_shot(s, nt, k + 1, r) for k, s in enumerate(shapes)]
    say(f"case: streaming batch {shapes}")
    outs, J = P.Batch(specs).fwi_gradient(shots)
    torch.cuda.synchronize()
    for i, (sp, sh) in enumerate(zip(specs, shots)):
        one = P.fwi_gradient(P.Plan(sp), sh["m"], sh["src_pos"], sh["q"], sh["rec_pos"],
                             sh["d_obs"], sh["Z"], fused=True)
        torch.cuda.synchronize()
        assert float(one["resid"].abs().max()) > 0
        for k in ("grad", "resid", "Ubar"):
            assert torch.equal(outs[i][k], one[k]), (i, k)
        assert float(J[i].item()) == float(one["misfit"].item()), i
