"""The scalar coefficient's gradient in both forms of its sum, at sizes where the
tile form runs (few levels on many tiles, or a workspace of one sum per tile) and
where the row walk does, ragged tiles and a single level among them: against the
oracle, and the full workspace against the least."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_2311_08322_amd import api, fields, inputs

from .helpers import TOL, round_f32

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("damping", [False, True], ids=["stated", "damping"])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("dims", [(512, 512, 20), (999, 501, 8), (57, 111, 66), (65, 5, 61), (1, 3, 9), (1500, 1501, 1)],
                         ids=lambda d: "x".join(map(str, d)))
def test_coeff_forms(dims, dtype, damping):
    ni, nj, nk = dims
    print(f"coeff forms {dims} {dtype} damping={damping}", flush=True)
    f = inputs.fields_sized(ni, nj, nk, seed=680)
    lam = inputs.cotangent(ni, nj, nk)
    f32 = dtype == torch.float32
    u, lm = (round_f32(a) if f32 else a for a in (f.u, lam))
    ud, ld = fields.from_padded(f.u, dtype, DEV), fields.from_interior(lam, dtype, DEV)
    mx, my = orc.hdiff_masks(u, decide_f32=f32, damping=damping)
    want = orc.coeff_grad(u, lm, mx, my, damping=damping)
    scale = float(np.sum(np.abs(orc.coeff_field_grad(u, lm, mx, my, damping=damping)))) or 1.0
    least = (((ni + 63) // 64) * ((nj + 3) // 4) * 8 + 255) // 256 * 256
    got = []
    for n in (api.stencil_param_workspace_bytes(dtype, dims), least):
        cb = torch.full((1,), 9.0, dtype=torch.float64, device=DEV)
        api.stencil_step_param_adjoint(ud, None, None, ld, None, cb, dims, inputs.DT_DZ,
                                       ws=torch.empty(n, dtype=torch.uint8, device=DEV),
                                       opts=api.Options(hdiff_form=api.HDIFF_DAMPING if damping else api.HDIFF_STATED))
        torch.cuda.synchronize()
        got.append(float(cb.item()))
        assert abs(got[-1] - want) <= TOL[dtype] * scale
    # the sum's order shows in FP64 by its last rounding alone, in FP32 (plain sums of
    # exact products, ni nj nk of them at most in a row) by theirs
    eps = np.finfo(np.float64).eps
    assert abs(got[0] - got[1]) <= (2 * eps if not f32 else ni * nj * nk * eps) * scale
