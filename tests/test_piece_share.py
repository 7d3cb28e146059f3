"""A piece shared by the waves of a workgroup: which of their segments join, on the code the kernel runs (CPU)."""
import ctypes

import numpy as np
import pytest

import host_lib

COST = 16
_rng = np.random.RandomState(3)
CASES = [[1], [16], [17, 64, 100, 256], [0, 0, 5, 0, 3000], [3] * 50 + [5000] + [2] * 50, list(_rng.randint(1, 700, size=40)),
         list(1 + _rng.randint(0, 40, size=900))]


@pytest.mark.parametrize("parts", [1, 2, 4, 8])
@pytest.mark.parametrize("n_pieces,min_piece,few", [(256, 64, (256, 16)), (7, 16, (0, 1)), (1, 16, (0, 1)), (64, 512, (16, 16))])
@pytest.mark.parametrize("lens", CASES, ids=range(len(CASES)))
def test_joined_parts_are_the_pieces_segments(lens, n_pieces, min_piece, few, parts):
    """Following each segment that joins none before it through the parts it says hold more gives the segments of the
    pieces themselves, each once, and `ends` says which reach the sequence's end; all others join the part before."""
    kv = np.asarray(lens, np.int32)
    out = np.zeros((sum(lens) // 16 + 16 * len(lens) + 65536, 8), np.int32)
    n = host_lib.load().xattn_test_part_runs(ctypes.c_void_p(kv.ctypes.data), len(kv), n_pieces, min_piece, COST, 0, *few, parts,
                                             ctypes.c_void_p(out.ctypes.data), len(out))
    assert 0 < n <= len(out)
    rows = [tuple(map(int, r)) for r in out[:n]]
    first = {}                                   # (piece, part): its first segment
    for r in rows:
        first.setdefault(r[:2], r)
    led, joined = [], set()
    for p, part, b, j0, j1, prev, nxt, ends in rows:
        if prev:
            assert first[p, part][2:5] == (b, j0, j1), "only a part's first segment joins the part before"
            continue
        end = j1
        for q in range(part + 1, part + 1 + nxt):
            _, _, b2, k0, k1, prev2, _, _ = first[p, q]
            assert (b2, k0, prev2) == (b, end, 1)
            end = k1
            joined.add((p, q))
        assert bool(ends) == (end == lens[b])
        led.append((p, b, j0, end))
    assert joined == {r[:2] for r in rows if r[5]}
    used = host_lib.plan(kv, n_pieces, min_piece, COST, 0, few)[1]
    assert led == [(p, b, j0, j1) for p in range(used) for b, j0, j1, _, _ in host_lib.piece_segments(kv, n_pieces, min_piece, COST, p, few=few)]


def test_every_kv_head_has_a_wave():
    for n in range(1, 200):
        heads, parts = divmod(host_lib.load().xattn_test_piece_share(n, 8), 16)
        assert 1 <= heads <= n and parts >= 1 and heads * parts <= 8
        if n <= 4 or n % 4 == 0 or n % 3 == 0:
            assert n % heads == 0 and (parts > 1 or heads > 4)
