"""The row walk of the generalised diffusion and of the coefficient's gradients
at its strips' edges (56 columns, 120 in FP32, by 16 rows), in rows that keep
8-byte alignment and rows that do not, over runs of levels with a remainder,
against the oracle."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_2311_08322_amd import api, fields, inputs

from .helpers import TOL, c_scalar, host, rel_err, round_f32, unpack_mask

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("aligned", [True, False], ids=["aligned", "packed"])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("dims", [(56, 16, 3), (57, 17, 5), (120, 15, 2), (121, 33, 7), (240, 64, 29), (2, 1, 1)],
                         ids=lambda d: "x".join(map(str, d)))
def test_general_strips(dims, dtype, aligned):
    ni, nj, nk = dims
    print(f"strips {dims} {dtype} aligned={aligned}", flush=True)
    f = inputs.fields_sized(ni, nj, nk, seed=650)
    kap, lam = inputs.coeff_field(ni, nj, nk), inputs.cotangent(ni, nj, nk)
    f32 = dtype == torch.float32
    u, k, lm = (round_f32(a) if f32 else a for a in (f.u, kap, lam))
    ud = fields.from_padded(f.u, dtype, DEV, aligned=aligned)
    kd, ld = (fields.from_interior(a, dtype, DEV, aligned=aligned) for a in (kap, lam))
    for damping in (False, True):
        form = api.HDIFF_DAMPING if damping else api.HDIFF_STATED
        mx, my = orc.hdiff_masks(u, decide_f32=f32, damping=damping)
        for field in (True, False):
            out = fields.alloc(ni, nj, nk, dtype, DEV, halo=0, aligned=aligned, fill=-3.0)
            mask = fields.mask_tensor(dims, DEV)
            api.stencil_hdiff(ud, out, dims, inputs.COEFF, mask=mask,
                              opts=api.Options(hdiff_form=form, coeff_field=kd if field else None))
            torch.cuda.synchronize()
            want, _, _ = orc.hdiff(u, c_scalar(inputs.COEFF, dtype), decide_f32=f32, kappa=k if field else None,
                                   damping=damping)
            assert rel_err(host(fields.interior(out, ni, nj, nk)), want[:, 2:-2, 2:-2]) <= TOL[dtype]
            gx, gy = unpack_mask(mask, ni, nj, nk)
            assert np.array_equal(gx, mx) and np.array_equal(gy, my)
        o = api.Options(hdiff_form=form)
        kb = fields.alloc(ni, nj, nk, dtype, DEV, halo=0, aligned=aligned, fill=5.0)
        api.stencil_coeff_field_adjoint(ud, ld, kb, dims, opts=o)
        cb = torch.full((1,), 9.0, dtype=torch.float64, device=DEV)
        n = api.stencil_param_workspace_bytes(dtype, dims)
        api.stencil_step_param_adjoint(ud, None, None, ld, None, cb, dims, inputs.DT_DZ,
                                       ws=torch.empty(n, dtype=torch.uint8, device=DEV), opts=o)
        torch.cuda.synchronize()
        want = orc.coeff_field_grad(u, lm, mx, my, damping=damping)
        assert rel_err(host(fields.interior(kb, ni, nj, nk)), want) <= TOL[dtype]
        scale = float(np.sum(np.abs(want))) or 1.0
        assert abs(float(cb.item()) - orc.coeff_grad(u, lm, mx, my, damping=damping)) <= TOL[dtype] * scale
