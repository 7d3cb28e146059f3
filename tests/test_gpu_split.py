"""Grouped-query decode where a workgroup holds several pieces (the vector path with few KV heads) or its waves share one, and
where a wave or several workgroups share a KV head's query rows, against the oracle."""
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
    xa.xattn_configure(xa.XATTN_CFG_PATH, 0)


def _case(lens, T, Hq, Hkv):
    q = normal_bf16(41, 0, len(lens) * T * Hq * D).reshape(len(lens), T, Hq, D)
    ks = [normal_bf16(41, 1 + 2 * b, L * Hkv * D).reshape(L, Hkv, D) for b, L in enumerate(lens)]
    vs = [normal_bf16(41, 2 + 2 * b, L * Hkv * D).reshape(L, Hkv, D) for b, L in enumerate(lens)]
    return q, ks, vs


# rows per KV head: 1, 3, 4 and 16 (one tile), 17 and 32 (two), 33 and 64 (two workgroups per piece); the vector path
# with 1 to 8 rows per wave and up to eight workgroups per piece
@pytest.mark.parametrize("path", [0, 1])
@pytest.mark.parametrize("T,group", [(1, 1), (3, 1), (1, 4), (4, 4), (1, 17), (4, 8), (3, 11), (16, 4)])
@pytest.mark.parametrize("Hkv", [1, 2, 3, 8])
@pytest.mark.parametrize("lens", [(5000, 16, 37, 3333), (700, 16, 37, 300), (17,)])
def test_pieces_and_rows_per_workgroup(T, group, Hkv, lens, path):
    """With few KV heads more pieces than workgroups on the vector path, so that several waves of one have a piece of their own,
    and several waves on a piece on the matrix path; and short streams in the default partition: pieces of 16 keys, a workgroup
    for every 16 query rows."""
    import paper_2510_14686_amd as xa
    from gpu_util import check_against_oracle
    xa.xattn_configure(xa.XATTN_CFG_PATH, path)
    if sum(lens) < 2000:
        xa.xattn_configure(xa.XATTN_CFG_MIN_PIECE_TOKENS, 0)
    q, ks, vs = _case(lens, T, group * Hkv, Hkv)
    check_against_oracle(q, ks, vs, lens, SCALE, what="T=%d group=%d Hkv=%d" % (T, group, Hkv))


@pytest.mark.parametrize("path", [0, 1])
@pytest.mark.parametrize("T,group", [(1, 3), (1, 8), (4, 8), (3, 11)])
@pytest.mark.parametrize("Hkv", [1, 2, 3])
def test_every_part_of_every_workgroup_has_a_piece(T, group, Hkv, path):
    """256 workgroups of 8, 4 and 2 parts, fewer where several share a piece.  Vector path: a piece each, 2048 of 16 keys at
    most, which the stream fills; matrix path: a run of a piece each."""
    import paper_2510_14686_amd as xa
    from gpu_util import check_against_oracle
    xa.xattn_configure(xa.XATTN_CFG_PATH, path)
    lens = (33000, 5, 1000)
    q, ks, vs = _case(lens, T, group * Hkv, Hkv)
    check_against_oracle(q, ks, vs, lens, SCALE, what="T=%d group=%d Hkv=%d" % (T, group, Hkv))


@pytest.mark.parametrize("path", [0, 1])
def test_a_workspace_for_one_piece_per_compute_unit_is_enough(path):
    """The vector path then takes fewer pieces per workgroup; the matrix path never takes more."""
    import torch

    import paper_2510_14686_amd as xa
    from gpu_util import check_against_oracle
    lens, Hq, Hkv = [5000, 1, 37, 3333], 8, 2
    xa.xattn_configure(xa.XATTN_CFG_PATH, path)
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
