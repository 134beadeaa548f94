"""A coefficient on the device under a tuning table whose column store is one of
the one-lane forms, which take their coefficient from the host: output and
gradients are those of the untuned call with the same number given from the host,
bit for bit."""
import json

import pytest
import torch

from paper_2311_08322_amd import api

from .test_gpu_train import C, DEV, _inputs, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("damping", [False, True], ids=["stated", "damping"])
@pytest.mark.parametrize("store", [api.COLUMN_REGISTERS, api.COLUMN_OUTBUF], ids=["registers", "outbuf"])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("dims", [(67, 45, 40), (130, 20, 100)], ids=lambda d: "x".join(map(str, d)))
def test_tuned_column_store(dims, dtype, store, damping, tmp_path):
    print(f"train tuned {dims} {dtype} store={store} damping={damping}", flush=True)
    api.stencil_clear_tuning()
    leaves, xbar = _inputs(dims, dtype)
    want = _run(leaves, xbar, torch.tensor(C, dtype=dtype, requires_grad=True), damping, True)
    path = tmp_path / "tuning.json"
    path.write_text(json.dumps({"arch": "gfx950", "entries": [
        {"dtype": int(dtype == torch.float64), "op": api.OP_STEP, "nk_class": (dims[2] + 15) // 16, "area_class": 0,
         "tile_i": 32, "tile_j": 8, "column_store": store}]}))
    api.stencil_load_tuning(str(path))
    try:
        assert api.stencil_tuning_lookup(dtype, api.OP_STEP, dims)[2] == store
        c = torch.tensor(C, dtype=dtype, device=DEV, requires_grad=True)
        got = _run(leaves, xbar, c, damping, True, after=lambda: c.detach().fill_(7.0))
        assert all(torch.equal(a, b.to(DEV)) for a, b in zip(got, want))
    finally:
        api.stencil_clear_tuning()
