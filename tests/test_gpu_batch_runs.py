"""Batched forward step: workgroups take their items in runs per XCD, 128 items a
round.  Launches of fewer items than a round, whole rounds and remainders give every
item to one workgroup: bit for bit the single-field call, mask included."""
import pytest
import torch

from paper_2311_08322_amd import api, fields, inputs

pytestmark = pytest.mark.gpu
DEV = "cuda"


def _field(dom, dtype, halo, seed, kextra=0):
    f = fields.alloc(*dom, dtype, DEV, halo=halo, kextra=kextra, fill=0.0)
    f.tensor.uniform_(-1, 1, generator=torch.Generator(DEV).manual_seed(seed))
    return f


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("nk", [12, 100, 140])
@pytest.mark.parametrize("tiles", [(1,), (127,), (128,), (129,), (250, 6), (200, 185)])
def test_items(dtype, nk, tiles):
    items, want = [], []
    wide = 128 if nk > (80 if dtype == torch.float32 else 96) else 256  # columns of a tile
    for q, n in enumerate(tiles):
        dom = (61, n * (wide // 64), nk)
        u, data, w = _field(dom, dtype, 2, q), _field(dom, dtype, 0, q + 7), _field(dom, dtype, 0, q + 9, 1)
        out, ref = (fields.alloc(*dom, dtype, DEV, halo=0, fill=5.0) for _ in range(2))
        mask, mref = (fields.mask_tensor(dom, DEV) for _ in range(2))
        args = dict(coeff=inputs.COEFF, dt_dz=inputs.DT_DZ)
        items.append(dict(u=u, data=data, w=w, out=out, domain=dom, mask=mask, **args))
        api.stencil_step(u, data, w, ref, dom, inputs.COEFF, inputs.DT_DZ, mask=mref)
        want.append((out, ref, mask, mref))
    ws = torch.empty(api.stencil_batch_workspace_bytes(dtype, items), dtype=torch.uint8, device=DEV)
    api.stencil_step_batched(dtype, items, ws, opts=api.Options(tile_i=64))
    torch.cuda.synchronize()
    for out, ref, mask, mref in want:
        assert torch.equal(out.tensor, ref.tensor) and torch.equal(mask, mref)
