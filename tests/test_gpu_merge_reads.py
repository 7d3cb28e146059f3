"""The merge kernels on calls of fewer and more sequences than XCDs: their forms by row count, against the oracle."""
import math

import numpy as np
import pytest

import oracle
from test_gpu_merge import pieces_of_16  # noqa: F401
from workloads import normal_bf16

pytestmark = pytest.mark.gpu


# rows 252 and 256 (16 waves per row, through the L2 and past it), 896 (4), 3584 (1); 8 sequences
@pytest.mark.parametrize("B,T,Hq,Hkv", [(3, 1, 84, 2), (4, 1, 64, 2), (7, 4, 32, 2), (7, 16, 32, 8), (8, 1, 84, 2)])
@pytest.mark.parametrize("slots", [2, 9, 70])
def test_gqa_merge_of_few_sequences(pieces_of_16, B, T, Hq, Hkv, slots):  # noqa: F811
    from gpu_util import check_against_oracle
    pieces_of_16(slots + 2 * B)              # a sequence counts as its keys + 16
    D, lens = 128, [16 * slots + T - 3] + [T + b % 5 for b in range(B - 1)]
    q = normal_bf16(33, 0, B * T * Hq * D).reshape(B, T, Hq, D)
    ks = [normal_bf16(33, 1 + 2 * b, L * Hkv * D).reshape(L, Hkv, D) for b, L in enumerate(lens)]
    vs = [normal_bf16(33, 2 + 2 * b, L * Hkv * D).reshape(L, Hkv, D) for b, L in enumerate(lens)]
    check_against_oracle(q, ks, vs, lens, float(np.float32(1.0 / math.sqrt(D))), what="B=%d slots=%d" % (B, slots))


@pytest.mark.parametrize("B,T,H", [(1, 1, 16), (7, 2, 128), (7, 3, 128), (8, 1, 16)])
@pytest.mark.parametrize("slots", [2, 9, 70])
def test_latent_kv_merge_of_few_sequences(pieces_of_16, B, T, H, slots):  # noqa: F811
    from gpu_util import assert_parity
    from test_gpu_mla import gpu_mla
    pieces_of_16(slots + 14 * B)             # a sequence counts as its keys + 192
    lens = [16 * slots + T - 3] + [15 + T + b % 5 for b in range(B - 1)]
    q = normal_bf16(34, 0, B * T * H * 576).reshape(B, T, H, 576)
    cs = [normal_bf16(34, 1 + b, L * 576).reshape(L, 576) for b, L in enumerate(lens)]
    scale = float(np.float32(1.0 / math.sqrt(576.0)))
    out_bits, lse = gpu_mla(q, cs, lens, scale)
    ref_out, ref_lse = oracle.mla(q, cs, lens, 512, scale)
    assert_parity(out_bits, lse, ref_out, ref_lse, what="B=%d slots=%d" % (B, slots))
