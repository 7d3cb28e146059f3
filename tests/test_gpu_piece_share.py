"""Grouped-query decode whose waves share a piece: sequences cut among them, at a piece's ends and at both, against the oracle."""
import math

import numpy as np
import pytest

from workloads import normal_bf16

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def restore():
    import paper_2510_14686_amd as xa
    yield
    xa.xattn_configure(xa.XATTN_CFG_PIECES, 0)
    xa.xattn_configure(xa.XATTN_CFG_MIN_PIECE_TOKENS, 0)


# 1 and 2 pieces: runs of up to 8 parts; 9: parts of one or two blocks, some without any.  One tile, two, and two groups of rows.
@pytest.mark.parametrize("pieces", [1, 2, 9])
@pytest.mark.parametrize("T,group", [(1, 2), (4, 4), (3, 7), (5, 12)])
@pytest.mark.parametrize("Hkv", [1, 2, 3, 4, 6, 7, 8, 12])
@pytest.mark.parametrize("lens", [(700, 16, 37, 300), (5, 1, 1203), (16, 17, 15, 33, 1, 64, 40)])
def test_sequences_cut_among_waves(lens, Hkv, T, group, pieces):
    import paper_2510_14686_amd as xa
    from gpu_util import check_against_oracle
    xa.xattn_configure(xa.XATTN_CFG_PIECES, pieces)
    xa.xattn_configure(xa.XATTN_CFG_MIN_PIECE_TOKENS, 16)
    D = 128
    lens = [L + T - 1 for L in lens]
    q = normal_bf16(43, 0, len(lens) * T * group * Hkv * D).reshape(len(lens), T, group * Hkv, D)
    ks = [normal_bf16(43, 1 + 2 * b, L * Hkv * D).reshape(L, Hkv, D) for b, L in enumerate(lens)]
    vs = [normal_bf16(43, 2 + 2 * b, L * Hkv * D).reshape(L, Hkv, D) for b, L in enumerate(lens)]
    check_against_oracle(q, ks, vs, lens, float(np.float32(1.0 / math.sqrt(D))), what="T=%d group=%d Hkv=%d" % (T, group, Hkv))
