"""The column solves at the edges of their register classes: the shortest and
the longest column of each class, odd and even, on ragged tiles (one column
past a tile in i and in j), against the oracle with the suite's per-dtype
tolerance (helpers.TOL)."""
import pytest
import torch

from oracle import oracle as orc
from paper_2311_08322_amd import api, fields, inputs

from .helpers import TOL, dev_fields, host, rel_err, round_f32

pytestmark = pytest.mark.gpu
DEV = "cuda"
# 16 | 24 | 40 (FP32) | 48 | 72 | 80 (FP32) levels per half column
CLASS_EDGES = [2, 31, 32, 33, 47, 48, 49, 79, 80, 81, 95, 96, 97, 98, 143, 144, 145, 159, 160]


def _fields(ni, nj, nk, dtype):
    f = inputs.fields_sized(ni, nj, nk, seed=700 + nk)
    xb = inputs.cotangent(ni, nj, nk)
    if dtype == torch.float32:
        f = inputs.Fields(u=round_f32(f.u), w=round_f32(f.w), data=round_f32(f.data))
        xb = round_f32(xb)
    return f, xb


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("nk", CLASS_EDGES)
def test_column_class_edges(nk, dtype):
    ni, nj = 65, 5
    dom = (ni, nj, nk)
    print(f"column classes {dom} {dtype}", flush=True)
    f, xb = _fields(ni, nj, nk, dtype)
    uin = f.u[:, 2:-2, 2:-2].copy()
    _, data, w = dev_fields(f, dtype, DEV)
    u = fields.from_interior(uin, dtype, DEV)
    out, lam = (fields.alloc(ni, nj, nk, dtype, DEV, halo=0, fill=7.0) for _ in range(2))
    api.stencil_vadv(u, data, w, out, dom, inputs.DT_DZ)
    api.stencil_vadv_adjoint(fields.from_interior(xb, dtype, DEV), w, lam, dom, inputs.DT_DZ)
    torch.cuda.synchronize()
    assert rel_err(host(fields.interior(out, *dom)), orc.vadv(uin, f.data, f.w, inputs.DT_DZ)) <= TOL[dtype]
    assert rel_err(host(fields.interior(lam, *dom)), orc.vadv_adjoint(xb, f.w, inputs.DT_DZ)) <= TOL[dtype]
    # nothing is written outside the domain (the row pitch is padded)
    for g in (out, lam):
        pad = g.tensor[:, :, ni:]
        assert torch.equal(pad, torch.full_like(pad, 7.0))


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
def test_batch_class_edges(dtype):
    """Batches whose fields sit on both sides of every class edge equal the
    separate calls bit for bit (forward with mask, adjoint)."""
    items, adj = [], []
    for n, nk in enumerate([1, 80, 81, 96, 97, 112, 113, 144]):
        ni, nj = (33, 9) if n % 2 else (65, 17)
        dom = (ni, nj, nk)
        f, xb = _fields(ni, nj, nk, dtype)
        u, data, w = dev_fields(f, dtype, DEV)
        items.append(dict(u=u, data=data, w=w, out=fields.alloc(ni, nj, nk, dtype, DEV, fill=0.0), domain=dom,
                          coeff=inputs.COEFF, dt_dz=inputs.DT_DZ, mask=fields.mask_tensor(dom, DEV)))
        adj.append(dict(x_bar=fields.from_interior(xb, dtype, DEV), w=w, mask=items[-1]["mask"],
                        u_bar=fields.alloc(ni, nj, nk, dtype, DEV, fill=0.0),
                        data_bar=fields.alloc(ni, nj, nk, dtype, DEV, halo=0, fill=0.0), domain=dom,
                        coeff=inputs.COEFF, dt_dz=inputs.DT_DZ))
    print(f"batch classes {dtype}", flush=True)
    ws = torch.empty(api.stencil_batch_workspace_bytes(dtype, items), dtype=torch.uint8, device=DEV)
    api.stencil_step_batched(dtype, items, ws)
    ws2 = torch.empty(api.stencil_batch_adjoint_workspace_bytes(dtype, adj), dtype=torch.uint8, device=DEV)
    api.stencil_step_adjoint_batched(dtype, adj, ws2)
    for it, a in zip(items, adj):
        dom = it["domain"]
        out = fields.alloc(*dom, dtype, DEV, fill=0.0)
        mask = fields.mask_tensor(dom, DEV)
        ub, db = fields.alloc(*dom, dtype, DEV, fill=0.0), fields.alloc(*dom, dtype, DEV, halo=0, fill=0.0)
        api.stencil_step(it["u"], it["data"], it["w"], out, dom, inputs.COEFF, inputs.DT_DZ, mask=mask)
        api.stencil_step_adjoint(a["x_bar"], a["w"], mask, ub, db, dom, inputs.COEFF, inputs.DT_DZ)
        assert torch.equal(out.tensor, it["out"].tensor), dom
        assert torch.equal(mask, it["mask"]), dom
        assert torch.equal(ub.tensor, a["u_bar"].tensor) and torch.equal(db.tensor, a["data_bar"].tensor), dom
