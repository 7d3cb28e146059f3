"""The table of segments that the merge kernel works from, written by a decode workgroup that may have keys of its own."""
import math

import numpy as np
import pytest

from workloads import normal_bf16

pytestmark = pytest.mark.gpu


# one KV head: 8 waves share a piece; 8: 2; 3: a workgroup with fewer waves; 5 and 12: several workgroups per piece.  65 and 130
# sequences: a second and third group of 64 in the table.  Both inner loops.
@pytest.mark.parametrize("Hkv", [1, 3, 5, 8, 12])
@pytest.mark.parametrize("B,lo,hi", [(3, 200, 900), (65, 60, 150), (130, 1, 90)])
@pytest.mark.parametrize("path", [0, 1])
def test_segments_of_every_sequence_reach_the_merge(Hkv, B, lo, hi, path):
    import paper_2510_14686_amd as xa
    from gpu_util import check_against_oracle
    D, group = 128, 2
    rng = np.random.RandomState(B)
    lens = [int(n) for n in rng.randint(lo, hi, size=B)]
    q = normal_bf16(35, 0, B * group * Hkv * D).reshape(B, 1, group * Hkv, D)
    ks = [normal_bf16(35, 1 + 2 * b, L * Hkv * D).reshape(L, Hkv, D) for b, L in enumerate(lens)]
    vs = [normal_bf16(35, 2 + 2 * b, L * Hkv * D).reshape(L, Hkv, D) for b, L in enumerate(lens)]
    xa.xattn_configure(xa.XATTN_CFG_PATH, path)
    try:
        check_against_oracle(q, ks, vs, lens, float(np.float32(1.0 / math.sqrt(D))), what="B=%d Hkv=%d path=%d" % (B, Hkv, path))
    finally:
        xa.xattn_configure(xa.XATTN_CFG_PATH, 0)
