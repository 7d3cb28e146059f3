"""Which merges deal their rows out round robin, on the code the kernel runs (CPU): those of calls where an eighth of the
sequences holds much more than an eighth of the keys."""
import ctypes

import numpy as np
import pytest

import host_lib


def spread(lens, seq_rows=32, n_pieces=256, cost=16):
    kv = np.asarray(lens, np.int32)
    chunk = 1
    while 64 * chunk < len(kv):
        chunk *= 2
    return host_lib.load().xattn_test_spread_rows(ctypes.c_void_p(kv.ctypes.data), len(kv), cost, chunk, n_pieces, seq_rows)


_rng = np.random.RandomState(5)


@pytest.mark.parametrize("seq_rows", [8, 64, 256, 4096])
@pytest.mark.parametrize("lens", [[1000] * 8, [30000] * 8, [0] * 9, list(_rng.randint(1024, 8192, size=64)),
                                  list(_rng.randint(30, 200, size=300)), [100] * 4096, list(_rng.randint(1, 60, size=3000))], ids=range(7))
def test_about_even_lengths_keep_their_order(lens, seq_rows):
    assert spread(lens, seq_rows) == 0


@pytest.mark.parametrize("seq_rows", [8, 32, 4096])
@pytest.mark.parametrize("lens", [[30000] + [100] * 7, [100] * 15 + [30000], [100] * 31 + [30000] + [100] * 31, [4000] * 8 + [100] * 56,
                                  [20] * 8 + [4000] + [20] * 7, [1] * 4000 + [9000] * 96], ids=range(6))
def test_uneven_lengths_are_dealt_out(lens, seq_rows):
    assert spread(lens, seq_rows) == 1


@pytest.mark.parametrize("lens,seq_rows", [([20] * 8 + [4000] + [20] * 7, 7), ([0] * 11 + [500], 60), ([1000] + [50] * 31, 32)])
def test_few_partial_rows_keep_their_order(lens, seq_rows):
    assert spread(lens, seq_rows) == 0


@pytest.mark.parametrize("lens", [[4000] * 32 + [100] * 32, [400] * 4 + [900] * 2 + [400] * 6], ids=range(2))
def test_a_quarter_of_the_keys_counts_where_partial_rows_are_many(lens):
    assert [spread(lens, rows, 128) for rows in (8, 127, 128, 1000)] == [0, 0, 1, 1]


@pytest.mark.parametrize("at", range(0, 64, 7))
def test_a_sequence_of_half_the_keys_is_seen_anywhere(at):
    lens = [100] * 64
    lens[at] = 64 * 116
    assert spread(lens) == 1


def test_the_largest_total_does_not_overflow():
    assert spread([2**27 - 16] * 15 + [2**27 - 17]) == 0 and spread([2**31 - 17 - 7 * 17] + [1] * 7) == 1
