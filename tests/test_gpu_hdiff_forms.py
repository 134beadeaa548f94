"""The horizontal diffusion on both sides of the lines between its row walk and its
tile kernel: strips and tiles by width (56 columns a strip, 120 in FP32; 32 a tile),
and masked domains of just over 2^22 points, where strips end one column or row past a
whole one, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_2311_08322_amd import api, fields, inputs

from .helpers import TOL, c_scalar, host, rel_err, round_f32, unpack_mask

pytestmark = pytest.mark.gpu
DEV = "cuda"
DIMS = [(1, 1, 1), (33, 9, 5), (62, 17, 3), (64, 8, 7), (73, 9, 2), (121, 11, 3), (250, 7, 5), (302, 17, 9),
        (62, 700, 98), (128, 301, 110), (1009, 65, 64), (1081, 33, 118), (1082, 49, 81)]


@pytest.mark.parametrize("aligned", [True, False], ids=["aligned", "packed"])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("dims", DIMS, ids=lambda d: "x".join(map(str, d)))
def test_forms(dims, dtype, aligned):
    ni, nj, nk = dims
    print(f"hdiff {dims} {dtype} aligned={aligned}", flush=True)
    f, kap = inputs.fields_sized(ni, nj, nk, seed=653), inputs.coeff_field(ni, nj, nk)
    f32 = dtype == torch.float32
    u, k = (round_f32(a) if f32 else a for a in (f.u, kap))
    ud = fields.from_padded(f.u, dtype, DEV, aligned=aligned)
    kd = fields.from_interior(kap, dtype, DEV, aligned=aligned)
    for damping, field in ((False, False), (True, False), (False, True)):
        mx, my = orc.hdiff_masks(u, decide_f32=f32, damping=damping)
        want, _, _ = orc.hdiff(u, c_scalar(inputs.COEFF, dtype), decide_f32=f32, kappa=k if field else None,
                               damping=damping)
        o = api.Options(hdiff_form=api.HDIFF_DAMPING if damping else api.HDIFF_STATED,
                        coeff_field=kd if field else None)
        for masked in (True, False):
            out = fields.alloc(ni, nj, nk, dtype, DEV, halo=0, aligned=aligned, fill=-3.0)
            mask = fields.mask_tensor(dims, DEV) if masked else None
            api.stencil_hdiff(ud, out, dims, inputs.COEFF, mask=mask, opts=o)
            torch.cuda.synchronize()
            assert rel_err(host(fields.interior(out, ni, nj, nk)), want[:, 2:-2, 2:-2]) <= TOL[dtype]
            if masked:
                gx, gy = unpack_mask(mask, ni, nj, nk)
                assert np.array_equal(gx, mx) and np.array_equal(gy, my)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
def test_byte_aligned_mask(dtype):
    dims = (62, 17, 3)
    f = inputs.fields_sized(*dims, seed=654)
    u = fields.from_padded(f.u, dtype, DEV)
    out = fields.alloc(*dims, dtype, DEV, halo=0, fill=0.0)
    want = fields.mask_tensor(dims, DEV)
    mask = torch.zeros(want.numel() + 4, dtype=torch.uint8, device=DEV)[3:-1]
    assert mask.data_ptr() % 4 == 3
    for m in (want, mask):
        api.stencil_hdiff(u, out, dims, inputs.COEFF, mask=m)
    torch.cuda.synchronize()
    assert torch.equal(mask, want)
