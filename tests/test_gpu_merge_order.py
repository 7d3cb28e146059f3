"""The merge kernels on calls of very unequal sequences, whose rows they deal out round robin, against the oracle."""
import math

import numpy as np
import pytest

import oracle
from workloads import normal_bf16

pytestmark = pytest.mark.gpu

# one long sequence first, in the middle and last, several ahead of the rest, among a few keys; 65 and 130: the table
# in groups of 64, more sequences than lanes
# (no sequences of one or two keys, whose results are values themselves: bf16 rounds those from 4 on by up to 2^-6 = 1.6e-2, more than
# the 1e-2 that assert_parity allows for an average)
LENS = {"first": [3000] + [20] * 8, "middle": [20] * 9 + [2500] + [20] * 6, "last": [5] * 20 + [1800], "ahead": [700] * 4 + [9] * 28,
        "few": [12] * 5 + [2000] + [12] * 6 + [30] * 3, "65": [15] * 64 + [4000], "130": [1200] * 3 + [10] * 127}


# rows per call up to 512 (16 waves a row), up to 2048 (4) and more (1)
@pytest.mark.parametrize("T,group,Hkv", [(1, 2, 1), (1, 4, 4), (4, 8, 4)])
@pytest.mark.parametrize("lens", LENS)
def test_gqa(lens, T, group, Hkv):
    from gpu_util import check_against_oracle
    D, name = 128, lens
    lens = [L + T - 1 for L in LENS[lens]]
    q = normal_bf16(51, 0, len(lens) * T * group * Hkv * D).reshape(len(lens), T, group * Hkv, D)
    ks = [normal_bf16(51, 1 + 2 * b, L * Hkv * D).reshape(L, Hkv, D) for b, L in enumerate(lens)]
    vs = [normal_bf16(51, 2 + 2 * b, L * Hkv * D).reshape(L, Hkv, D) for b, L in enumerate(lens)]
    check_against_oracle(q, ks, vs, lens, float(np.float32(1.0 / math.sqrt(D))), what="%s T=%d" % (name, T))


@pytest.mark.parametrize("T,H", [(1, 8), (2, 24), (2, 72)])
@pytest.mark.parametrize("lens", LENS)
def test_latent_kv(lens, T, H):
    from gpu_util import assert_parity
    from test_gpu_mla import gpu_mla
    name, lens = lens, [L + T - 1 for L in LENS[lens]]
    q = normal_bf16(52, 0, len(lens) * T * H * 576).reshape(len(lens), T, H, 576)
    cs = [normal_bf16(52, 1 + b, L * 576).reshape(L, 576) for b, L in enumerate(lens)]
    scale = float(np.float32(1.0 / math.sqrt(576.0)))
    out_bits, lse = gpu_mla(q, cs, lens, scale)
    ref_out, ref_lse = oracle.mla(q, cs, lens, 512, scale)
    assert_parity(out_bits, lse, ref_out, ref_lse, what="%s T=%d" % (name, T))


@pytest.mark.parametrize("Hq,Hkv", [(8, 2), (32, 8)])
def test_a_replayed_graph_takes_the_order_of_its_lengths(Hq, Hkv):
    """Recorded with even lengths, replayed with very unequal ones and back: the bits of an eager call each time."""
    import torch

    import paper_2510_14686_amd as xa
    B, D, scale = 16, 128, float(np.float32(1.0 / math.sqrt(128)))
    kv = [torch.from_numpy(normal_bf16(53, s, B * 4000 * Hkv * D).view(np.int16)).cuda() for s in (1, 2)]
    q = torch.from_numpy(normal_bf16(53, 0, B * Hq * D).view(np.int16)).cuda()
    ptrs = [torch.tensor([t.data_ptr() + b * 4000 * Hkv * D * 2 for b in range(B)], dtype=torch.int64, device="cuda") for t in kv]
    lens = torch.full((B,), 500, dtype=torch.int32, device="cuda")
    outs = [torch.zeros((B, 1, Hq, D), dtype=torch.int16, device="cuda") for _ in range(2)]
    lses = [torch.zeros((B, 1, Hq), dtype=torch.float32, device="cuda") for _ in range(2)]
    side = torch.cuda.Stream()
    torch.cuda.synchronize()

    def call(i, stream):
        xa.xattn_decode(q, ptrs[0], ptrs[1], lens, B, 1, Hq, Hkv, D, scale, outs[i], lses[i], stream)
    call(0, side)
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        call(0, side)
    for given in ([500] * B, [4000] + [50] * (B - 1), [500] * B, [20] * (B - 1) + [3999]):
        lens.copy_(torch.tensor(given, dtype=torch.int32))
        outs[0].fill_(0x7FC0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        call(1, torch.cuda.current_stream())
        torch.cuda.synchronize()
        assert torch.equal(outs[0], outs[1]) and torch.equal(lses[0], lses[1]), given
