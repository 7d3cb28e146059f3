"""The merge kernels against the oracle, at the slot counts and row counts where their split over waves changes."""
import math

import numpy as np
import pytest

import oracle
from workloads import normal_bf16

pytestmark = pytest.mark.gpu


@pytest.fixture
def pieces_of_16():
    """set(n): n pieces of 16 keys, so that a sequence of 16 n keys has n partial results."""
    import paper_2510_14686_amd as xa

    def set_pieces(n):
        xa.xattn_configure(xa.XATTN_CFG_PIECES, n)
        xa.xattn_configure(xa.XATTN_CFG_MIN_PIECE_TOKENS, 16 if n else 0)
    yield set_pieces
    set_pieces(0)


# one long sequence (16 keys per slot) and short ones: rows per call 8 (16 waves per row), 640 (4), 2240 (1)
@pytest.mark.parametrize("B,Hq", [(1, 8), (20, 32), (70, 32)])
@pytest.mark.parametrize("slots", [2, 8, 9, 17, 64, 65, 300])
def test_gqa_merge_over_waves(pieces_of_16, B, Hq, slots):
    from gpu_util import check_against_oracle
    pieces_of_16(slots + 2 * B)              # a sequence counts as its keys + 16
    lens = [16 * slots - 3] + [1 + b % 5 for b in range(B - 1)]
    D, Hkv = 128, 2
    q = normal_bf16(31, 0, B * Hq * D).reshape(B, 1, Hq, D)
    ks = [normal_bf16(31, 1 + 2 * b, L * Hkv * D).reshape(L, Hkv, D) for b, L in enumerate(lens)]
    vs = [normal_bf16(31, 2 + 2 * b, L * Hkv * D).reshape(L, Hkv, D) for b, L in enumerate(lens)]
    check_against_oracle(q, ks, vs, lens, float(np.float32(1.0 / math.sqrt(D))), what="B=%d slots=%d" % (B, slots))


@pytest.mark.parametrize("B,H", [(1, 16), (40, 16), (140, 16)])
@pytest.mark.parametrize("slots", [2, 8, 9, 65])
def test_latent_kv_merge_over_waves(pieces_of_16, B, H, slots):
    from gpu_util import assert_parity
    from test_gpu_mla import gpu_mla
    pieces_of_16(slots + 14 * B)             # a sequence counts as its keys + 192
    lens = [16 * slots - 3] + [16 + b % 5 for b in range(B - 1)]
    q = normal_bf16(32, 0, B * H * 576).reshape(B, 1, H, 576)
    cs = [normal_bf16(32, 1 + b, L * 576).reshape(L, 576) for b, L in enumerate(lens)]
    scale = float(np.float32(1.0 / math.sqrt(576.0)))
    out_bits, lse = gpu_mla(q, cs, lens, scale)
    ref_out, ref_lse = oracle.mla(q, cs, lens, 512, scale)
    assert_parity(out_bits, lse, ref_out, ref_lse, what="B=%d slots=%d" % (B, slots))
