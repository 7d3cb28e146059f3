"""Grouped-query decode with KV head counts that leave a workgroup's last group of heads partly empty, against the oracle."""
import math

import numpy as np
import pytest

from workloads import normal_bf16

pytestmark = pytest.mark.gpu


# 1 and 2 query tokens of 2 rows; 40 rows, two groups; 64.  Sequences split over pieces, cut among waves, and short ones.
@pytest.mark.parametrize("T,group", [(1, 2), (5, 8), (8, 8)])
@pytest.mark.parametrize("Hkv", [5, 7, 10, 11, 13, 18, 27, 36, 41])
@pytest.mark.parametrize("lens", [(700, 16, 37, 300), (2100, 33, 5)])
def test_uneven_groups_of_heads(lens, Hkv, T, group):
    from gpu_util import check_against_oracle
    D = 128
    lens = [L + T - 1 for L in lens]
    q = normal_bf16(57, 0, len(lens) * T * group * Hkv * D).reshape(len(lens), T, group * Hkv, D)
    ks = [normal_bf16(57, 1 + 2 * b, L * Hkv * D).reshape(L, Hkv, D) for b, L in enumerate(lens)]
    vs = [normal_bf16(57, 2 + 2 * b, L * Hkv * D).reshape(L, Hkv, D) for b, L in enumerate(lens)]
    check_against_oracle(q, ks, vs, lens, float(np.float32(1.0 / math.sqrt(D))), what="T=%d group=%d Hkv=%d" % (T, group, Hkv))
