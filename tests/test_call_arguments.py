"""Arguments of the binding, without a GPU: a domain may be any iterable of three
numbers, also one that can be read only once."""
import numpy as np
import pytest

from paper_2311_08322_amd import _lib


@pytest.mark.parametrize("numbers", [(4, 5, 6), (4.0, 5.9, 6.0), ("4", "5", "6"), np.array([4, 5, 6]),
                                     np.array([4.0, 5.0, 6.0])], ids=["int", "float", "text", "int64", "float64"])
@pytest.mark.parametrize("once", [tuple, iter, lambda x: (v for v in x), lambda x: map(lambda v: v, x)],
                         ids=["tuple", "iter", "generator", "map"])
def test_domain(numbers, once):
    assert tuple(_lib.domain3(once(numbers))) == (4, 5, 6)


def test_domain_refused():
    with pytest.raises((IndexError, ValueError)):
        _lib.domain3((1, 2, 3, 4))
    with pytest.raises(ValueError):
        _lib.domain3(("x", 2, 3))
