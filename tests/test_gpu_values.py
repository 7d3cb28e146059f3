"""Grouped-query decode on values at the edge of what the types hold, against the oracle: sums that must not leave
the fp32 range, weights that must be exact, infinities and NaN among the cached values."""
import math

import numpy as np
import pytest

import oracle
from workloads import bf16_to_f32, normal_bf16

pytestmark = pytest.mark.gpu
D = 128
SCALE = float(np.float32(1.0 / math.sqrt(D)))
# rows per KV head: 1 and 3 (weights in three parts), 4 and 16 (one tile), 32 (two tiles)
ROWS = [(1, 1), (3, 1), (1, 4), (4, 4), (4, 8)]


def _bf16(x):
    """fp32 -> bf16 bits of values that bf16 holds exactly."""
    bits = np.ascontiguousarray(x, dtype=np.float32).view(np.uint32)
    assert not np.any(bits & 0xffff)
    return (bits >> 16).astype(np.uint16)


@pytest.fixture(autouse=True)
def configure():
    import paper_2510_14686_amd as xa
    keys = (xa.XATTN_CFG_PIECES, xa.XATTN_CFG_MIN_PIECE_TOKENS, xa.XATTN_CFG_PATH, xa.XATTN_CFG_PV_MODE)

    def set_all(*values):
        for key, value in zip(keys, values + (0,) * (len(keys) - len(values))):
            xa.xattn_configure(key, value)
    set_all()
    yield set_all
    set_all()


def _scores_case(T, group, Hkv, scores):
    """q = e0, K's first column = the scores of one sequence's keys (bf16 values), scale 1."""
    L, Hq = len(scores), group * Hkv
    q = np.zeros((1, T, Hq, D), np.float32)
    q[..., 0] = 1.0
    k = np.zeros((L, Hkv, D), np.float32)
    k[:, :, 0] = np.asarray(scores, np.float32)[:, None]
    return _bf16(q), [_bf16(k)]


@pytest.mark.parametrize("pv_mode", [0, 1, 2])
@pytest.mark.parametrize("T,group", ROWS)
def test_weights_do_not_exceed_one(configure, T, group, pv_mode):
    """One key a little above an earlier block's maximum, values of 2^122: the sum of at most 48 weights of at most
    1 stays below 2^128, a weight of 2^7 does not."""
    from gpu_util import gpu_attn
    configure(1, 16, 0, pv_mode)
    L = 48
    scores = np.zeros(L)
    scores[20] = 5.0                          # 2^7.2 times the weight of the others
    q, ks = _scores_case(T, group, 2, scores)
    vs = [_bf16(np.full((L, 2, D), 2.0 ** 122, np.float32))]
    out_bits, lse = gpu_attn(q, ks, vs, [L], 1.0)
    ref_out, ref_lse = oracle.attn(q, ks, vs, [L], 1.0)
    # a weighted mean of one value: 2^-8 is half a bf16 ulp below a power of two, and 2^-8 the one-bf16 weights' rounding
    got = bf16_to_f32(out_bits).astype(np.float64)
    assert np.all(np.abs(got / 2.0 ** 122 - 1.0) <= 2.0 ** -8 + (2.0 ** -8 if pv_mode == 2 else 0.0))
    assert np.max(np.abs(lse - ref_lse)) < 1e-5


@pytest.mark.parametrize("T,group", ROWS)
def test_the_largest_key_has_an_exact_weight(configure, T, group):
    """With one bf16 per weight a row that one key carries is as exact as its output's rounding, wherever the key's
    score lies against those of earlier blocks.  The scale of a row (its projection on the exact one) averages the
    rounding of 128 normal outputs, 1.66e-3 each, to 1.66e-3 sqrt(3 / 128) = 2.5e-4; a rounded weight is off by up
    to 2^-8 = 3.9e-3 of itself."""
    from gpu_util import gpu_attn
    configure(1, 16, 0, 2)
    L, Hkv = 32, 8
    worst = 0.0
    for case in range(8):
        scores = np.full(L, -40.0)
        scores[3] = 0.0                                       # the first block's maximum
        scores[19] = 4.0 + case * 0.1875                      # 2^5.8 to 2^7.7 times its weight
        q, ks = _scores_case(T, group, Hkv, np.round(scores * 32) / 32)
        vs = [normal_bf16(60 + case, 1, L * Hkv * D).reshape(L, Hkv, D)]
        out_bits, _ = gpu_attn(q, ks, vs, [L], 1.0)
        ref, _ = oracle.attn(q, ks, vs, [L], 1.0)
        got = bf16_to_f32(out_bits).astype(np.float64).reshape(ref.shape)
        worst = max(worst, float(np.max(np.abs(np.sum(got * ref, -1) / np.sum(ref * ref, -1) - 1.0))))
    # 4.5 standard deviations for the output, and the smaller key's weight: 2^-5.8 of the row, off by 2^-8 of itself
    assert worst <= 4.5 * 2.5e-4 + 2.0 ** -13.8, worst


@pytest.mark.parametrize("pv_mode", [0, 1])
@pytest.mark.parametrize("pieces", [1, 2])
@pytest.mark.parametrize("T,group", ROWS)
def test_weights_have_more_than_sixteen_bits(configure, T, group, pieces, pv_mode):
    """Two keys whose values cancel to about 2^-15 of themselves, in one segment and in two: 16-bit weights are off by
    up to 2^-17, a sixteenth of the result on average."""
    from gpu_util import gpu_attn
    configure(pieces, 16, 0, pv_mode)
    L, Hkv = 32, 8
    delta = 0.25 + np.arange(Hkv) / 16.0                      # second key's score below the first's, per KV head
    Hq = group * Hkv
    q = np.zeros((1, T, Hq, D), np.float32)
    q[..., 0] = 1.0
    k = np.zeros((L, Hkv, D), np.float32)
    k[:, :, 0] = -200.0                                       # no weight
    k[3, :, 0] = 0.0
    k[20, :, 0] = -delta
    v = np.zeros((L, Hkv, D), np.float32)
    a, b = np.meshgrid(np.arange(128, 256), np.arange(128, 256), indexing="ij")
    for h in range(Hkv):
        diff = np.abs(a - b * math.exp(-delta[h])).ravel()
        best = np.argsort(diff)[:D]                           # the 128 closest pairs of 8-bit values
        v[3, h], v[20, h] = a.ravel()[best], -b.ravel()[best]
    out_bits, _ = gpu_attn(_bf16(q), [_bf16(k)], [_bf16(v)], [L], 1.0)
    ref, _ = oracle.attn(_bf16(q), [_bf16(k)], [_bf16(v)], [L], 1.0)
    got = bf16_to_f32(out_bits).astype(np.float64).reshape(ref.shape)
    # the output's rounding; and of the summands, below 256: exp2 (2^-23), its argument (up to 1: twice 2^-24), the
    # weights of a merge (2^-23) and the sums (2^-24)
    assert np.all(np.abs(got - ref) <= 2.0 ** -8 * np.abs(ref) + 256 * 2.0 ** -21)


# rows 1 to 3 per KV head; merges of 16, 4 and 1 waves per row; segments from one to 64
@pytest.mark.parametrize("T,group,Hkv", [(1, 1, 2), (1, 2, 8), (3, 1, 3), (1, 1, 600), (1, 3, 700)])
@pytest.mark.parametrize("pieces", [1, 3, 20, 64])
def test_infinite_values_below_four_rows(configure, T, group, Hkv, pieces):
    """An infinity or NaN among the values reaches its own column of the rows that see its key, as what the sum
    makes of it, and nothing else."""
    from gpu_util import TOL_LSE, TOL_MAX_ABS, gpu_attn
    configure(pieces, 16)
    L, Hq = 16 * 20 - 16, group * Hkv         # a sequence counts as its keys + 16: pieces end at whole blocks
    q = normal_bf16(61, 0, T * Hq * D).reshape(1, T, Hq, D)
    k = normal_bf16(61, 1, L * Hkv * D).reshape(L, Hkv, D)
    v = normal_bf16(61, 2, L * Hkv * D).reshape(L, Hkv, D).copy()
    inf, minus_inf, nan = 0x7F80, 0xFF80, 0x7FC0
    for col, (key, value) in enumerate([(0, inf), (5, minus_inf), (16, inf), (47, inf), (100, minus_inf), (163, inf), (200, nan),
                                        (299, inf)]):
        v[key, :, 3 + 11 * col] = value
    v[20, :, 127] = inf
    v[220, :, 127] = minus_inf                # in different segments, or in one
    out_bits, lse = gpu_attn(q, [k], [v], [L], SCALE)
    ref_out, ref_lse = oracle.attn(q, [k], [v], [L], SCALE)
    got = bf16_to_f32(out_bits).astype(np.float64).reshape(ref_out.shape)
    assert np.array_equal(np.isnan(got), np.isnan(ref_out))
    assert np.array_equal(np.isposinf(got), np.isposinf(ref_out)) and np.array_equal(np.isneginf(got), np.isneginf(ref_out))
    finite = np.isfinite(ref_out)
    assert np.max(np.abs(got[finite] - ref_out[finite])) <= TOL_MAX_ABS and np.max(np.abs(lse - ref_lse)) <= TOL_LSE


@pytest.mark.parametrize("T,group", [(1, 1), (1, 3), (3, 1)])
def test_weight_modes_do_not_apply_below_four_rows(configure, T, group):
    from gpu_util import gpu_attn
    L, Hkv = 700, 2
    Hq = group * Hkv
    q = normal_bf16(62, 0, T * Hq * D).reshape(1, T, Hq, D)
    kv = [normal_bf16(62, 1 + i, L * Hkv * D).reshape(L, Hkv, D) for i in range(2)]
    want = gpu_attn(q, [kv[0]], [kv[1]], [L], SCALE)
    for pv_mode in (1, 2):
        configure(0, 0, 0, pv_mode)
        got = gpu_attn(q, [kv[0]], [kv[1]], [L], SCALE)
        np.testing.assert_array_equal(got[0], want[0])
        np.testing.assert_array_equal(got[1], want[1])
