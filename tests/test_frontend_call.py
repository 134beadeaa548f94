"""What a stencil call hands to its generated library, without a GPU: a stand-in
library records the field descriptions."""
import ctypes

import pytest
import torch

from paper_2311_08322_amd import api
from paper_2311_08322_amd.frontend import PARALLEL, Field, computation, interval, stencil


@stencil
def shift(u: Field, v: Field, out: Field):
    with computation(PARALLEL), interval(...):
        out = u[1, 0, 0] + v


class Library:
    def gts_workspace_bytes(self, dom):
        return 0

    def gts_run(self, fields, n, scalars, ns, dom, ws, nbytes, stream):
        words = ctypes.cast(fields, ctypes.POINTER(ctypes.c_int64))
        self.fields = [words[10 * f:10 * f + 10] for f in range(n)]
        return 0


def _words(t, o):
    st, shape = t.stride()[::-1], t.shape[::-1]
    return [t.data_ptr() + sum(a * b for a, b in zip(o, st)) * t.element_size(), *st, *o,
            *(n - a for n, a in zip(shape, o))]


@pytest.mark.parametrize("longer", [(), (7,), (7, 8)], ids=["3", "4", "5"])
def test_field_descriptions(longer, monkeypatch):
    """An origin's first three entries count, as they are."""
    L = Library()
    monkeypatch.setattr(shift, "build", lambda dtype: L)
    u, v, out = (torch.zeros(n, dtype=torch.float64) for n in ((6, 9, 12), (5, 8, 11), (4, 7, 10)))
    at = [(1, 2, 0), (3, 1, 1), (0, 2, 0)]
    want = [_words(t, o) for t, o in zip((u, v, out), at)]
    shift(*(api.Field(t, o + longer) for t, o in zip((u, v, out), at)), domain=(4, 3, 4))
    assert L.fields == want
    shift(u, v, out, origin=dict(zip("uv", (o + longer for o in at)), out=at[2] + longer), domain=(4, 3, 4))
    assert L.fields == want
    shift(u, v, out, origin=(1, 1, 0) + longer, domain=(4, 3, 4))
    assert L.fields == [_words(t, (1, 1, 0)) for t in (u, v, out)]
    with pytest.raises(IndexError):
        shift(u, v, out, origin=(1, 1), domain=(4, 3, 4))
