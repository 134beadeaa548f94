"""Argument checks of the training calls, which need no GPU: every buffer that a
call writes is refused where it overlaps one that it reads or another output, and
scalars and workspaces where they are missing or misaligned.  The pointers are
never dereferenced."""
import pytest

from paper_2311_08322_amd import _lib

BASE = 0x7F0000000000
NI, NJ, NK = 16, 12, 8
DOM = (NI, NJ, NK)
NAMES = ["x_bar", "mask", "u", "w", "x", "coeff_copy", "u_bar", "data_bar", "w_bar", "kappa_bar", "coeff_bar", "ws"]
INPUTS, OUTPUTS = NAMES[:6], NAMES[6:]
AT = {n: BASE + (i << 32) for i, n in enumerate(NAMES + ["kappa", "out", "data", "coeff_dev"])}


@pytest.fixture(scope="module")
def L():
    return _lib.lib()


def code(name):
    return _lib.CODES[name]


def backward(L, dtype=_lib.F64, column=True, nbytes=None, form=0, **at):
    p = {**{n: AT[n] for n in NAMES}, "kappa": None, **at}
    if not column:
        p.update(w=None, data_bar=None, w_bar=None, x=None)
    n = L.stencil_param_workspace_bytes(dtype, _lib.domain3(DOM)) if nbytes is None else nbytes
    return L.stencil_train_backward(dtype, p["x_bar"], p["mask"], p["u"], p["w"], p["x"], p["kappa"], 0.0,
                                    p["coeff_copy"], p["u_bar"], p["data_bar"], p["w_bar"], p["kappa_bar"],
                                    p["coeff_bar"], p["ws"], n, *DOM, 0.5, form, None)


def forward(L, dtype=_lib.F64, column=True, coeff_dtype=_lib.F64, **at):
    p = {**AT, "kappa": None, **at}
    if not column:
        p.update(w=None, data=None)
    return L.stencil_train_forward(dtype, p["u"], p["data"], p["w"], p["out"], p["mask"], p["kappa"], 0.0,
                                   p["coeff_dev"], coeff_dtype, p["coeff_copy"], *DOM, 0.5, 0, None)


@pytest.mark.parametrize("out", OUTPUTS)
@pytest.mark.parametrize("other", NAMES)
def test_backward_overlaps(L, out, other):
    if other == out:
        return
    for dtype in (_lib.F64, _lib.F32):
        assert backward(L, dtype, **{out: AT[other]}) == code("STENCIL_E_ALIAS")
    if out in ("u_bar", "kappa_bar", "coeff_bar", "ws") and other not in ("w", "x", "data_bar", "w_bar"):
        assert backward(L, column=False, **{out: AT[other]}) == code("STENCIL_E_ALIAS")


def test_backward_kappa_overlaps(L):
    for out in ("u_bar", "data_bar", "w_bar", "kappa_bar"):
        assert backward(L, kappa=AT[out], coeff_copy=None, coeff_bar=None) == code("STENCIL_E_ALIAS")


def test_backward_scalars_and_workspace(L):
    assert backward(L, kappa=AT["kappa"], coeff_bar=None) == code("STENCIL_E_ARG")  # both kinds of coefficient
    assert backward(L, kappa=AT["kappa"], coeff_copy=None) == code("STENCIL_E_ARG")
    need = L.stencil_param_workspace_bytes(_lib.F64, _lib.domain3(DOM))
    assert backward(L, ws=None) == code("STENCIL_E_WORKSPACE")
    assert backward(L, nbytes=need - 1) == code("STENCIL_E_WORKSPACE")
    assert backward(L, ws=AT["ws"] + 4) == code("STENCIL_E_WORKSPACE")
    for n in ("coeff_copy", "coeff_bar", "u", "x", "w_bar", "kappa_bar"):
        assert backward(L, **{n: AT[n] + 4}) == code("STENCIL_E_DTYPE")
        assert backward(L, _lib.F32, **{n: AT[n] + 2}) == code("STENCIL_E_DTYPE")
    assert backward(L, u=None) == code("STENCIL_E_NULL") and backward(L, x=None) == code("STENCIL_E_NULL")
    assert backward(L, data_bar=None) == code("STENCIL_E_NULL") and backward(L, u_bar=None) == code("STENCIL_E_NULL")
    assert backward(L, form=9, ws=AT["ws"]) == code("STENCIL_E_ARG")


@pytest.mark.parametrize("column", [True, False], ids=["step", "hdiff"])
def test_forward(L, column):
    ins = ["u", "coeff_dev"] + (["data", "w"] if column else [])
    for out in ("out", "mask", "coeff_copy"):
        for other in ins + [o for o in ("out", "mask", "coeff_copy") if o != out]:
            assert forward(L, column=column, **{out: AT[other]}) == code("STENCIL_E_ALIAS"), (out, other)
    n = L.stencil_mask_bytes(_lib.domain3(DOM))
    assert forward(L, column=column, coeff_copy=AT["mask"] + n - 8) == code("STENCIL_E_ALIAS")
    assert forward(L, column=column, coeff_dev=AT["coeff_dev"] + 4) == code("STENCIL_E_DTYPE")
    assert forward(L, column=column, coeff_copy=AT["coeff_copy"] + 4) == code("STENCIL_E_DTYPE")
    assert forward(L, _lib.F32, column, _lib.F32, coeff_dev=AT["coeff_dev"] + 2) == code("STENCIL_E_DTYPE")
    assert forward(L, column=column, kappa=AT["kappa"]) == code("STENCIL_E_ARG")
    assert forward(L, column=column, mask=None) == code("STENCIL_E_NULL")
    assert forward(L, column=column, coeff_copy=None) == code("STENCIL_E_NULL")
