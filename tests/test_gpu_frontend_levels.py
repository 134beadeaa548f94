"""Generated kernels that load levels ahead: columns and chunks shorter than, as long
as and around multiples of the four (two, with many inputs) levels in flight.  The
arithmetic is exact up to one rounding per sum, so the results equal NumPy's."""
import numpy as np
import pytest
import torch

from paper_2311_08322_amd import fields
from paper_2311_08322_amd.frontend import BACKWARD, FORWARD, PARALLEL, Field, computation, interval, stencil

DEV = "cuda"


@stencil
def cross(u: Field, v: Field, out: Field):
    with computation(PARALLEL), interval(...):
        out = ((u[-1, 0, 0] + u[1, 0, 0]) + (u[0, -1, 0] + u[0, 1, 0])) - v


@stencil
def nine(a: Field, b: Field, c: Field, d: Field, e: Field, f: Field, g: Field, h: Field, m: Field, out: Field):
    with computation(PARALLEL), interval(...):
        out = ((((((((a + b) + c) + d) + e) + f) + g) + h) + m)


@stencil
def forward(u: Field, out: Field):
    with computation(FORWARD):
        with interval(0, 1):
            out = u
        with interval(1, None):
            out = u + 0.5 * out[0, 0, -1]


@stencil
def backward(u: Field, out: Field):
    with computation(BACKWARD):
        with interval(-1, None):
            out = u
        with interval(0, -1):
            out = u[0, 0, 1] + 0.5 * out[0, 0, 1]


def test_point_form():
    for s in (cross, nine, forward, backward):
        assert "auto issue" in s.source("float64"), s  # evaluated point by point


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("nk", [1, 2, 3, 4, 5, 7, 8, 9, 13, 33])
def test_levels(nk, dtype):
    ni, nj = 67, 5
    print(f"levels {nk} {dtype}", flush=True)
    npd = np.float64 if dtype == torch.float64 else np.float32
    r = np.random.default_rng(nk)
    a = r.uniform(-1, 1, (10, nk, nj + 4, ni + 4)).astype(npd)
    x = [fields.from_padded(q, dtype, DEV) for q in a]
    p = a[:, :, 2:-2, 2:-2]

    def run(s, *ins):
        out = fields.alloc(ni, nj, nk, dtype, DEV, halo=0, fill=0.0)
        s(*ins, out, domain=(ni, nj, nk))
        torch.cuda.synchronize()
        return fields.interior(out, ni, nj, nk).cpu().numpy()

    u = a[0]
    want = ((u[:, 2:-2, 1:-3] + u[:, 2:-2, 3:-1]) + (u[:, 1:-3, 2:-2] + u[:, 3:-1, 2:-2])) - p[1]
    assert np.array_equal(run(cross, x[0], x[1]), want)
    want = p[0]
    for q in p[1:9]:
        want = want + q
    assert np.array_equal(run(nine, *x[:9]), want)
    want = p[0].copy()
    for k in range(1, nk):
        want[k] = p[0][k] + npd(0.5) * want[k - 1]
    assert np.array_equal(run(forward, x[0]), want)
    want = p[0].copy()
    for k in range(nk - 2, -1, -1):
        want[k] = p[0][k + 1] + npd(0.5) * want[k + 1]
    assert np.array_equal(run(backward, x[0]), want)
