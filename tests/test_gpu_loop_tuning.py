"""A periodic loop captured while another thread changes the tuning table: all its
steps take the entry that the capture found, so the replay is that of a capture
under one of the two tables, bit for bit."""
import json
import threading

import pytest
import torch

from paper_2311_08322_amd import api, fields, inputs

from .helpers import dev_fields

pytestmark = pytest.mark.gpu
DEV = "cuda"
DIMS, STEPS = (20, 6, 8), 300


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
def test_loop_keeps_its_tuning(dtype, tmp_path):
    print(f"loop under changing tuning {dtype}", flush=True)
    u0, data, w = dev_fields(inputs.fields_sized(*DIMS, seed=512), dtype, DEV)
    path = tmp_path / "tuning.json"
    path.write_text(json.dumps({"arch": "gfx950", "entries": [
        {"dtype": int(dtype == torch.float64), "op": api.OP_STEP, "nk_class": 1, "area_class": 0, "tile_i": 64,
         "tile_j": 4, "column_store": api.COLUMN_REGISTERS}]}))
    opts, s = api.Options(boundary=api.BOUNDARY_PERIODIC), torch.cuda.Stream()
    a, b = (fields.alloc(*DIMS, dtype, DEV, fill=0.0) for _ in range(2))

    def loop():
        fields.padded(a, *DIMS).copy_(fields.padded(u0, *DIMS))
        fields.padded(b, *DIMS).fill_(-5.0)
        torch.cuda.synchronize()
        graph = api.stencil_graph_capture_steps(STEPS, a, b, data, w, DIMS, inputs.COEFF, inputs.DT_DZ, opts=opts,
                                                stream=s)
        api.stencil_graph_launch(graph, stream=s)
        s.synchronize()
        api.stencil_graph_destroy(graph)
        return fields.padded(a, *DIMS).clone(), fields.padded(b, *DIMS).clone()

    changes, stop = 0, threading.Event()

    def change():
        nonlocal changes
        while not stop.is_set():
            api.stencil_load_tuning(str(path))
            api.stencil_clear_tuning()
            changes += 1

    api.stencil_clear_tuning()
    try:
        wanted = [loop()]
        api.stencil_load_tuning(str(path))
        wanted.append(loop())
        t = threading.Thread(target=change)
        t.start()
        try:
            got = [loop() for _ in range(8)]
        finally:
            stop.set()
            t.join()
        assert changes > 0
        for g in got:
            assert any(torch.equal(g[0], x[0]) and torch.equal(g[1], x[1]) for x in wanted)
    finally:
        api.stencil_clear_tuning()
