"""The untuned step's tile where 128-column tiles do not pay: long FP64 columns
whose 64x2 tiles fit one round, domains that 64x4 fills (more than a workgroup per
CU, a quarter or 0.4 of the last-level cache, more than three 16x8 tiles per CU), and
the long generalised class.  The default equals the 64 x 4 tile bit for bit, masks
included."""
import pytest
import torch

from .test_gpu_default_tile import test_default_tile as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("dims", [(763, 42, 113), (771, 141, 61), (256, 200, 80), (252, 470, 17), (626, 59, 107),
                                  (320, 491, 32), (300, 300, 45), (300, 320, 30), (305, 320, 30)], ids=lambda d: "x".join(map(str, d)))
def test_default_tile_rounds(dims, dtype):
    check(dims, dtype)
