"""How the KV heads of a call are grouped on the matrix path: every head has a wave, and most of the chip has work (CPU)."""
import ctypes

import numpy as np
import pytest

import host_lib

N_CU, MAX_WAVES = 256, 8


def call_share(n_kv_heads, row_groups):
    runs = np.zeros(MAX_WAVES + 1, np.int32)
    got = host_lib.load().xattn_test_call_share(N_CU, row_groups, n_kv_heads, MAX_WAVES, ctypes.c_void_p(runs.ctypes.data))
    return got // 16, got % 16, runs


@pytest.mark.parametrize("row_groups", [1, 2, 4])
@pytest.mark.parametrize("n_kv_heads", list(range(1, 65)) + [100, 128, 1000, 100000])
def test_waves_per_head(n_kv_heads, row_groups):
    heads, parts, runs = call_share(n_kv_heads, row_groups)
    assert 1 <= heads <= n_kv_heads and parts in (1, 2, 4, 8) and heads * parts <= MAX_WAVES < heads * parts * 2 + heads
    assert runs[0] == runs[heads]


@pytest.mark.parametrize("row_groups", [1, 2])
@pytest.mark.parametrize("n_kv_heads", range(1, 65))
def test_most_of_the_chip_has_work(n_kv_heads, row_groups):
    """One workgroup per compute unit, eight waves each, would cut a head's keys into MAX_WAVES * N_CU / (groups * heads) runs.
    With more than 32 query rows no other group of 2, 4 or 8 heads would give more."""
    _, _, runs = call_share(n_kv_heads, row_groups)
    assert runs[0] >= 0.6 * 64 * MAX_WAVES * N_CU / (row_groups * n_kv_heads)
    if row_groups > 1:
        assert all(runs[0] >= runs[h] for h in (1, 2, 4, 8) if h < n_kv_heads)
