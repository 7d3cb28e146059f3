"""The plan's quotients, which are products with an inverse: the integers they stand for (CPU)."""
import numpy as np
import pytest

import host_lib

COST = 16
_rng = np.random.RandomState(11)


def _exact_bounds(total, n, skew):
    def rounded(x):
        return min(total, (x + 8) // 16 * 16)
    if not skew:
        return [rounded(p * total // n) for p in range(n)] + [total]
    starts = [(total // 8) * x + (total % 8) * x // 8 + ((total // 8000) * skew + total % 8000 * skew // 8000 if x & 1 else 0) for x in range(9)]
    m = n // 8
    return [rounded(starts[p // m] + p % m * (starts[p // m + 1] - starts[p // m]) // m) for p in range(n)] + [total]


@pytest.mark.parametrize("n_pieces", [1, 7, 8, 96, 256, 1000, 65536])
@pytest.mark.parametrize("total", [17, 4097, 156169, 1 << 20, (1 << 24) - 3, 2**31 - 1] + [int(x) for x in _rng.randint(2000, 2**31 - 1, size=6)])
@pytest.mark.parametrize("skew", [0, 32])
def test_piece_bounds_are_the_exact_quotients(total, n_pieces, skew):
    lens = [total - COST]
    got = host_lib.piece_bounds(lens, n_pieces, 64, COST, skew)
    n = len(got) - 1
    assert n == max(1, min(n_pieces, total // 64))
    used = skew if n % 8 == 0 and total // n >= 512 else 0
    assert list(map(int, got)) == _exact_bounds(total, n, used)


@pytest.mark.parametrize("steps", [-2, -1, 0, 1, 2])
def test_an_inverse_two_units_off_still_gives_the_integer(steps):
    """What the device's inverse may differ by from the host's division, at quotients just at and just below an integer."""
    m = np.concatenate([np.arange(1, 300), _rng.randint(300, 65537, size=3000), [65535, 65536]]).astype(np.int64)
    inv = 1.0 / m
    for _ in range(abs(steps)):
        inv = np.nextafter(inv, np.inf if steps > 0 else 0.0)
    for span in [int(x) for x in _rng.randint(1, 2**31 - 1, size=40)] + [2**31 - 1, 65536, 1]:
        for i in (m, m - 1, m // 2, _rng.randint(0, 65537, size=len(m)) % m):
            assert np.array_equal(np.floor((i * float(span) + 0.25) * inv).astype(np.int64), i * span // m)
    for a in (2**31 - 1, 2**31 - 2, 123456789):
        near = np.concatenate([a // m * m, np.maximum(a // m * m - 1, 0)])
        assert np.array_equal(np.floor((near + 0.25) * np.concatenate([inv, inv])).astype(np.int64), near // np.concatenate([m, m]))
