"""The gradient of w in runs of two levels (large FP64 fields), three and four,
with every remainder of the nk + 1 levels, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_2311_08322_amd import api, fields, inputs

from .helpers import TOL, host, rel_err, round_f32

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("dims", [(65, 5, n) for n in (1, 2, 3, 4, 5, 7, 8, 9, 10, 13, 14)] + [(701, 600, 30), (701, 600, 31)],
                         ids=lambda d: "x".join(map(str, d)))
def test_w_grad(dims, dtype):
    ni, nj, nk = dims
    print(f"w grad {dims} {dtype}", flush=True)
    r = np.random.default_rng(690 + nk)
    w, x, lam = (r.uniform(-1, 1, (n, nj, ni)) for n in (nk + 1, nk, nk))
    w[:, 0, 0] = 0.0  # no sign
    wf, xf, lf = (fields.from_interior(a, dtype, DEV) for a in (w, x, lam))
    wb = fields.alloc(ni, nj, nk, dtype, DEV, halo=0, kextra=1, fill=7.0)
    api.stencil_step_param_adjoint(None, wf, xf, lf, wb, None, dims, inputs.DT_DZ, dtype=dtype)
    torch.cuda.synchronize()
    if dtype == torch.float32:
        w, x, lam = map(round_f32, (w, x, lam))
    assert rel_err(host(fields.interior(wb, ni, nj, nk + 1)), orc.w_grad(w, x, lam, inputs.DT_DZ)) <= TOL[dtype]
