"""Grouped-query decode where a workgroup holds several pieces (few KV heads) and where a wave or several
workgroups share a KV head's query rows, against the oracle."""
import math

import numpy as np
import pytest

import oracle
from workloads import normal_bf16

pytestmark = pytest.mark.gpu
D = 128
SCALE = float(np.float32(1.0 / math.sqrt(D)))


@pytest.fixture(autouse=True)
def small_pieces():
    import paper_2510_14686_amd as xa
    xa.xattn_configure(xa.XATTN_CFG_PIECES, 0)
    xa.xattn_configure(xa.XATTN_CFG_MIN_PIECE_TOKENS, 16)
    yield
    xa.xattn_configure(xa.XATTN_CFG_PIECES, 0)
    xa.xattn_configure(xa.XATTN_CFG_MIN_PIECE_TOKENS, 0)


def _case(lens, T, Hq, Hkv):
    q = normal_bf16(41, 0, len(lens) * T * Hq * D).reshape(len(lens), T, Hq, D)
    ks = [normal_bf16(41, 1 + 2 * b, L * Hkv * D).reshape(L, Hkv, D) for b, L in enumerate(lens)]
    vs = [normal_bf16(41, 2 + 2 * b, L * Hkv * D).reshape(L, Hkv, D) for b, L in enumerate(lens)]
    return q, ks, vs


# rows per KV head: 1 and 3 (vector path), 4, 16, 17, 32 (one and two tiles), 33 and 64 (two workgroups per piece)
@pytest.mark.parametrize("T,group", [(1, 1), (3, 1), (1, 4), (4, 4), (1, 17), (4, 8), (3, 11), (16, 4)])
@pytest.mark.parametrize("Hkv", [1, 2, 3, 8])
@pytest.mark.parametrize("lens", [(5000, 16, 37, 3333), (700, 16, 37, 300), (17,)])
def test_pieces_and_rows_per_workgroup(T, group, Hkv, lens):
    """More pieces than compute units, so that every wave of a workgroup has a piece of its own; and short
    streams in the default partition: pieces of 16 keys, a workgroup for every 16 query rows."""
    import paper_2510_14686_amd as xa
    from gpu_util import check_against_oracle
    if sum(lens) < 2000:
        xa.xattn_configure(xa.XATTN_CFG_MIN_PIECE_TOKENS, 0)
    q, ks, vs = _case(lens, T, group * Hkv, Hkv)
    check_against_oracle(q, ks, vs, lens, SCALE, what="T=%d group=%d Hkv=%d" % (T, group, Hkv))


def test_a_workspace_for_one_piece_per_compute_unit_is_enough():
    import torch

    import paper_2510_14686_amd as xa
    from gpu_util import check_against_oracle
    lens, Hq, Hkv = [5000, 1, 37, 3333], 8, 2
    xa.xattn_configure(xa.XATTN_CFG_PIECES, torch.cuda.get_device_properties(0).multi_processor_count)
    small = xa.xattn_workspace_bytes(len(lens), 1, Hq, Hkv, D)
    xa.xattn_configure(xa.XATTN_CFG_PIECES, 0)
    assert small < xa.xattn_workspace_bytes(len(lens), 1, Hq, Hkv, D)
    q, ks, vs = _case(lens, 1, Hq, Hkv)
    ws = torch.empty(small, dtype=torch.uint8, device="cuda")
    xa.xattn_set_workspace(ws, small)
    try:
        check_against_oracle(q, ks, vs, lens, SCALE, what="small workspace")
    finally:
        torch.cuda.synchronize()
        xa.xattn_set_workspace(None, 0)
