"""What the binding takes for a scale (CPU): a number, or TypeError before anything is called."""
import numpy as np
import pytest

import paper_2510_14686_amd as xa

CALLS = [lambda scale: xa.xattn_decode(None, None, None, None, 1, 1, 8, 8, 128, scale, None, None),
         lambda scale: xa.xattn_decode_noalloc(None, None, None, None, 1, 1, 8, 8, 128, scale, None, None),
         lambda scale: xa.xattn_mla_decode(None, None, None, 1, 1, 16, 512, 64, scale, None, None)]


@pytest.mark.parametrize("call", CALLS, ids=["decode", "decode_noalloc", "mla_decode"])
@pytest.mark.parametrize("scale", ["0.1", None, [0.1], 1j])
def test_no_number_is_a_type_error(call, scale):
    with pytest.raises(TypeError):
        call(scale)


@pytest.mark.parametrize("call", CALLS, ids=["decode", "decode_noalloc", "mla_decode"])
@pytest.mark.parametrize("scale", [0.1, 1, True, np.float32(0.1), np.float64(0.1)])
def test_a_number_reaches_the_call(call, scale):
    with pytest.raises(xa.XattnError):       # refused there: the addresses are NULL
        call(scale)
