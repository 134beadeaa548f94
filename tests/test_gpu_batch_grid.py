"""Batches of more workgroups than one grid holds (2^32 lanes): one field of a
single column of points, 64-wide tiles of four rows and one more tile than fits,
equal bit for bit to calls that run it in wider rows.  On one level T = 1, so the
column adjoint is the identity."""
import pytest
import torch

from paper_2311_08322_amd import api, fields, inputs

pytestmark = pytest.mark.gpu
DEV = "cuda"
TILES = (1 << 32) // 512 + 1  # 512 lanes a workgroup
DOM = (1, 4 * TILES - 3, 1)


def _field(halo, lo, hi, kextra=0):
    n = (DOM[2] + kextra, DOM[1] + 2 * halo, DOM[0] + 2 * halo)
    return api.Field(torch.empty(n, dtype=torch.float32, device=DEV).uniform_(lo, hi), (halo, halo, 0))


def test_step():
    print(f"batched step of {TILES} tiles", flush=True)
    torch.manual_seed(31)
    u, data, w = _field(2, 0, 1), _field(0, -0.1, 0.1), _field(0, -1, 1, 1)
    out, want = _field(0, 5, 6), _field(0, 7, 8)
    mask, mask1 = (fields.mask_tensor(DOM, DEV) for _ in range(2))
    items = [dict(u=u, data=data, w=w, out=out, domain=DOM, coeff=inputs.COEFF, dt_dz=inputs.DT_DZ, mask=mask)]
    ws = torch.empty(api.stencil_batch_workspace_bytes(torch.float32, items), dtype=torch.uint8, device=DEV)
    api.stencil_step_batched(torch.float32, items, ws, opts=api.Options(tile_i=64))
    api.stencil_step(u, data, w, want, DOM, inputs.COEFF, inputs.DT_DZ, mask=mask1,
                     opts=api.Options(tile_i=16, tile_j=16))
    torch.cuda.synchronize()
    assert torch.equal(out.tensor, want.tensor) and torch.equal(mask, mask1)


def test_adjoint():
    print(f"batched adjoint of {TILES} tiles", flush=True)
    torch.manual_seed(32)
    x, w, ub, db, want = _field(0, -1, 1), _field(0, -1, 1, 1), _field(2, 5, 6), _field(0, 5, 6), _field(2, 7, 8)
    mask = torch.randint(0, 256, fields.mask_tensor(DOM, DEV).shape, dtype=torch.uint8, device=DEV)
    items = [dict(x_bar=x, w=w, mask=mask, u_bar=ub, data_bar=db, domain=DOM, coeff=inputs.COEFF, dt_dz=inputs.DT_DZ)]
    ws = torch.empty(api.stencil_batch_adjoint_workspace_bytes(torch.float32, items), dtype=torch.uint8, device=DEV)
    api.stencil_step_adjoint_batched(torch.float32, items, ws)
    api.stencil_hdiff_adjoint(x, mask, want, DOM, inputs.COEFF)
    torch.cuda.synchronize()
    assert torch.equal(db.tensor, x.tensor) and torch.equal(ub.tensor, want.tensor)
