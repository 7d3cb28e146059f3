"""What the binding takes for an address (CPU)."""
import numpy as np
import pytest

from paper_2510_14686_amd.binding import _ptr


class Tensor:
    def __init__(self, address):
        self.address = address

    def data_ptr(self):
        return self.address


@pytest.mark.parametrize("given,address", [(None, None), (0, 0), (4096, 4096), (Tensor(64), 64), (Tensor(np.int64(128)), 128)])
def test_addresses(given, address):
    assert _ptr(given) == address and type(_ptr(given)) is type(address)


@pytest.mark.parametrize("given", ["4096", 1.5, np.int64(4096), [4096]])
def test_anything_else_is_refused(given):
    with pytest.raises(TypeError):
        _ptr(given)
