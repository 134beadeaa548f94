"""A stencil's variables may have any name: one called `cond` is a value of the
fields' type in the generated kernel, not a truth value."""
import re

import numpy as np
import pytest
import torch

from paper_2311_08322_amd import fields
from paper_2311_08322_amd.frontend import PARALLEL, Field, computation, interval, stencil


@stencil
def named(u: Field, out: Field):
    with computation(PARALLEL), interval(...):
        cond = u * 0.5
        if u[1, 0, 0] > 0.25:
            cond = cond + 3.0
        out = cond - cond[-1, 0, 0]


@pytest.mark.parametrize("dtype", ["float64", "float32"])
def test_only_the_condition_is_a_truth_value(dtype):
    src = named.source(dtype)
    assert "gts_g0" in src and "P_u_p0" in src  # evaluated point by point
    exprs = re.findall(r"const bool \w+ = \(bool\)\((.*)\);", src)
    assert len(exprs) == 2 and all(" > " in e for e in exprs)  # at the point and at its west neighbour


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
def test_values(dtype):
    ni, nj, nk = 67, 5, 6
    print(f"names {dtype}", flush=True)
    npd = np.float64 if dtype == torch.float64 else np.float32
    u = np.random.default_rng(1200).uniform(-1, 1, (nk, nj + 4, ni + 4)).astype(npd)
    out = fields.alloc(ni, nj, nk, dtype, "cuda", halo=0, fill=0.0)
    named(fields.from_padded(u, dtype, "cuda"), out, domain=(ni, nj, nk))
    torch.cuda.synchronize()
    c = u[:, 2:-2, :-1] * npd(0.5)
    c = np.where(u[:, 2:-2, 1:] > 0.25, c + npd(3), c)
    assert np.array_equal(fields.interior(out, ni, nj, nk).cpu().numpy(), c[:, :, 2:-1] - c[:, :, 1:-2])
