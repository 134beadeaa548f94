"""The training calls behind autograd: a scalar coefficient on the device (either
type) gives what the same number given from the host gives, bit for bit, also
when the tensor changes before the backward or the saved tensors leave the
device meanwhile; a larger u takes the general route to the same values."""
import numpy as np
import pytest
import torch

from paper_2311_08322_amd import autograd, inputs

pytestmark = pytest.mark.gpu
DEV = "cuda"
C = float(np.float32(0.025))  # the same in both types


def _inputs(dims, dtype):
    f = inputs.fields_sized(*dims, seed=660)
    t = [torch.tensor(a, dtype=dtype, device=DEV) for a in (f.u, f.data, f.w, inputs.cotangent(*dims))]
    return [x.requires_grad_() for x in t[:3]], t[3]


def _run(leaves, xbar, coeff, damping, column, after=lambda: None, hooks=None):
    args = leaves if column else leaves[:1]
    with hooks or torch.enable_grad():
        out = (autograd.step if column else autograd.hdiff)(*args, coeff, damping=damping)
    after()
    wanted = list(args) + ([coeff] if torch.is_tensor(coeff) else [])
    return [out.detach(), *torch.autograd.grad(out, wanted, xbar)]


@pytest.mark.parametrize("column", [True, False], ids=["step", "hdiff"])
@pytest.mark.parametrize("damping", [False, True], ids=["stated", "damping"])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("dims", [(67, 45, 7), (1, 1, 1), (130, 20, 100), (33, 17, 144)],
                         ids=lambda d: "x".join(map(str, d)))
def test_device_coefficient(dims, dtype, damping, column):
    print(f"train {dims} {dtype} damping={damping} column={column}", flush=True)
    leaves, xbar = _inputs(dims, dtype)
    want = _run(leaves, xbar, torch.tensor(C, dtype=dtype, requires_grad=True), damping, column)  # read on the host
    plain = _run(leaves, xbar, C, damping, column)
    assert all(torch.equal(a, b) for a, b in zip(plain, want))
    for cdtype in (torch.float64, torch.float32):
        c = torch.tensor(C, dtype=cdtype, device=DEV, requires_grad=True)
        got = _run(leaves, xbar, c, damping, column, after=lambda: c.detach().fill_(7.0))
        assert all(torch.equal(a, b.to(DEV)) for a, b in zip(got[:-1], want))
        assert got[-1].dtype == cdtype and float(got[-1]) == float(want[-1].to(cdtype))
    c = torch.tensor(C, dtype=dtype, device=DEV, requires_grad=True)
    got = _run(leaves, xbar, c, damping, column, hooks=torch.autograd.graph.save_on_cpu())
    assert all(torch.equal(a, b.to(DEV)) for a, b in zip(got, want))


def test_larger_field_takes_the_general_route():
    """u with rows beyond the halo is read at its own strides."""
    (u, data, w), _ = _inputs((40, 12, 6), torch.float64)
    big = torch.zeros(6, 20, 44, dtype=torch.float64, device=DEV)
    big[:, :16] = u.detach()
    with torch.no_grad():
        c = torch.tensor(C, device=DEV)
        assert torch.equal(autograd.step(big, data, w, c), autograd.step(u, data, w, c))
