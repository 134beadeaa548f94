"""The untuned step's tile: on both sides of the rule (domains that fit half the
last-level cache or all of it, whole rounds of workgroups or partly idle ones, the generalised step's spilling
class) the default equals the 64 x 4 tile bit for bit, masks included."""
import pytest
import torch

from paper_2311_08322_amd import api, fields, inputs

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("dims", [(1, 1, 1), (17, 9, 31), (130, 61, 96), (33, 20, 144), (256, 256, 80), (300, 300, 60),
                                  (384, 384, 64), (512, 512, 48)],
                         ids=lambda d: "x".join(map(str, d)))
def test_default_tile(dims, dtype):
    ni, nj, nk = dims
    print(f"default tile {dims} {dtype}", flush=True)
    api.stencil_clear_tuning()
    g = torch.Generator(device=DEV)
    g.manual_seed(7)

    def draw(halo, lo, hi, kextra=0):
        f = fields.alloc(ni, nj, nk, dtype, DEV, halo=halo, kextra=kextra, fill=0.0)
        f.tensor.uniform_(lo, hi, generator=g)
        return f
    u, data, w = draw(2, 0, 1), draw(0, -0.1, 0.1), draw(0, -1, 1, 1)
    kap = draw(0, 0.0125, 0.0375)
    for field in (None, kap):
        for saves in (True, False):
            res = []
            for kw in (dict(), dict(tile_i=64, tile_j=4)):
                out, mask = draw(0, 0, 1), fields.mask_tensor(dims, DEV)
                api.stencil_step(u, data, w, out, dims, inputs.COEFF, inputs.DT_DZ, mask=mask if saves else None,
                                 opts=api.Options(coeff_field=field, **kw))
                torch.cuda.synchronize()
                res.append((fields.interior(out, *dims).clone(), mask.clone()))
            assert torch.equal(res[0][0], res[1][0])
            assert not saves or torch.equal(res[0][1], res[1][1])
