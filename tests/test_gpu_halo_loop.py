"""Periodic loops whose steps read the halo from the state's interior: after 1 to
5 captured steps both buffers, halos included, equal eager periodic steps bit for
bit, at tile edges, in every register class, from a state whose halo is not
periodic, over several replays."""
import pytest
import torch

from paper_2311_08322_amd import api, fields, inputs

from .helpers import dev_fields

pytestmark = pytest.mark.gpu
DEV = "cuda"
DIMS = [(2, 2, 3), (1, 5, 2), (3, 9, 4), (64, 4, 80), (65, 9, 17), (66, 7, 33), (67, 33, 96), (34, 20, 144), (20, 6, 150)]


@pytest.mark.parametrize("damping", [False, True], ids=["stated", "damping"])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("dims", DIMS, ids=lambda d: "x".join(map(str, d)))
def test_periodic_loop(dims, dtype, damping):
    ni, nj, nk = dims
    if damping and nk > 144:
        pytest.skip("the generalised step's longest column")
    print(f"periodic loop {dims} {dtype} damping={damping}", flush=True)
    f = inputs.fields_sized(ni, nj, nk, seed=511)
    u0, data, w = dev_fields(f, dtype, DEV)  # u0's halo is not its interior's period
    opts = api.Options(boundary=api.BOUNDARY_PERIODIC, hdiff_form=api.HDIFF_DAMPING if damping else api.HDIFF_STATED)
    for nsteps in (1, 2, 3, 5):
        e, g = ([fields.alloc(ni, nj, nk, dtype, DEV, fill=-5.0) for _ in range(2)] for _ in range(2))
        s = torch.cuda.Stream()
        torch.cuda.synchronize()
        graph = api.stencil_graph_capture_steps(nsteps, g[0], g[1], data, w, dims, inputs.COEFF, inputs.DT_DZ,
                                                opts=opts, stream=s)
        try:
            for replay in range(3):
                for x in (e, g):
                    fields.padded(x[0], *dims).copy_(fields.padded(u0, *dims))
                    fields.padded(x[1], *dims).fill_(-5.0)
                for n in range(nsteps):
                    api.stencil_step(e[n % 2], data, w, e[(n + 1) % 2], dims, inputs.COEFF, inputs.DT_DZ, opts=opts)
                torch.cuda.synchronize()
                api.stencil_graph_launch(graph, stream=s)
                s.synchronize()
                for a, b in zip(e, g):
                    assert torch.equal(fields.padded(a, *dims), fields.padded(b, *dims)), (nsteps, replay)
        finally:
            api.stencil_graph_destroy(graph)
