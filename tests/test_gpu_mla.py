"""Latent-KV (MLA-shaped) decode attention on the GPU against the fp64 oracle."""
import math

import numpy as np
import pytest

import oracle
import workloads as wl
from workloads import MLA_CONFIGS, bf16_to_f32, f32_to_bf16, normal_bf16

pytestmark = pytest.mark.gpu

DQK, DV = 576, 512
SCALE = float(np.float32(1.0 / math.sqrt(192.0)))


def gpu_mla(q, cs, lens, scale, xtensor=False, seed=0, want_lse=True):
    import torch

    import paper_2510_14686_amd as xa
    B, T, H, _ = q.shape
    with xa.KVStore(cs, cs, xtensor=xtensor, seed=seed) as store:
        qd = torch.from_numpy(np.ascontiguousarray(q).view(np.int16)).cuda()
        lens_d = torch.from_numpy(np.ascontiguousarray(lens, dtype=np.int32)).cuda()
        out = torch.full((B, T, H, DV), 0x7FC0, dtype=torch.int16, device="cuda")
        lse = torch.full((B, T, H), float("nan"), dtype=torch.float32, device="cuda") if want_lse else None
        xa.xattn_mla_decode(qd, store.k_ptrs, lens_d, B, T, H, 512, 64, scale, out, lse, torch.cuda.current_stream())
        torch.cuda.synchronize()
        return out.cpu().numpy().view(np.uint16), (lse.cpu().numpy() if want_lse else None)


def _case(seed, lens, T, H, extra=0):
    B = len(lens)
    q = f32_to_bf16(bf16_to_f32(normal_bf16(seed, 0, B * T * H * DQK)) * np.float32(math.sqrt(192.0 / DQK)))
    q = q.reshape(B, T, H, DQK)
    cs = [normal_bf16(seed, 1 + b, (L + extra) * DQK).reshape(L + extra, DQK) for b, L in enumerate(lens)]
    return q, cs


@pytest.fixture(autouse=True)
def _default_partition():
    import paper_2510_14686_amd as xa
    xa.xattn_configure(xa.XATTN_CFG_PIECES, 0)
    xa.xattn_configure(xa.XATTN_CFG_MIN_PIECE_TOKENS, 0)
    xa.xattn_configure(xa.XATTN_CFG_PV_MODE, 0)
    xa.xattn_configure(xa.XATTN_CFG_MLA_LAYOUT, 0)
    yield
    xa.xattn_configure(xa.XATTN_CFG_PIECES, 0)
    xa.xattn_configure(xa.XATTN_CFG_MIN_PIECE_TOKENS, 0)
    xa.xattn_configure(xa.XATTN_CFG_PV_MODE, 0)
    xa.xattn_configure(xa.XATTN_CFG_MLA_LAYOUT, 0)


@pytest.mark.parametrize("T,H", [(1, 128), (2, 128), (1, 16), (1, 32), (3, 64), (1, 8), (2, 24), (1, 144)])
def test_mla_shapes(T, H):
    """Head counts from 8 to 144 (four waves per 16-row tile, one or two waves per 32-row tile, partial tiles, more than
    128 rows: several row groups) and 1 to 3 query tokens, ragged lengths around multiples of 16 keys."""
    from gpu_util import assert_parity
    lens = [T, T + 1, 15 + T, 16 + T, 17 + T, 64, 65, 200, 333, 1500]
    q, cs = _case(200 + T, lens, T, H)
    out_bits, lse = gpu_mla(q, cs, lens, SCALE)
    ref_out, ref_lse = oracle.mla(q, cs, lens, DV, SCALE)
    assert_parity(out_bits, lse, ref_out, ref_lse, "mla T=%d H=%d" % (T, H))


@pytest.mark.parametrize("pieces,min_piece", [(8, 16), (256, 16), (1024, 16), (1, 0), (37, 48)])
def test_mla_result_does_not_depend_on_the_partition(pieces, min_piece):
    import paper_2510_14686_amd as xa
    from gpu_util import assert_parity
    lens = [700, 33, 2, 2049, 16, 512, 90]
    q, cs = _case(210, lens, 2, 32)
    ref_out, ref_lse = oracle.mla(q, cs, lens, DV, SCALE)
    xa.xattn_configure(xa.XATTN_CFG_PIECES, pieces)
    xa.xattn_configure(xa.XATTN_CFG_MIN_PIECE_TOKENS, min_piece)
    out_bits, lse = gpu_mla(q, cs, lens, SCALE)
    assert_parity(out_bits, lse, ref_out, ref_lse, "mla pieces=%d" % pieces)


def test_mla_xtensor_equals_plain_and_rows_past_kv_len_are_not_read():
    from gpu_util import assert_parity
    lens = [3000, 1025, 40, 1821]          # 1152 B per token: about 1820 tokens per 2 MiB chunk
    q, cs = _case(211, lens, 1, 64, extra=30)
    for b, L in enumerate(lens):
        cs[b][L:] = 0x7FC0                  # NaN past the end
    a_out, a_lse = gpu_mla(q, cs, lens, SCALE, xtensor=False)
    b_out, b_lse = gpu_mla(q, cs, lens, SCALE, xtensor=True, seed=4)
    np.testing.assert_array_equal(a_out, b_out)
    np.testing.assert_array_equal(a_lse, b_lse)
    ref_out, ref_lse = oracle.mla(q, [c[:L] for c, L in zip(cs, lens)], lens, DV, SCALE)
    assert_parity(a_out, a_lse, ref_out, ref_lse, "mla padded")


@pytest.mark.parametrize("pv_mode,layout", [(1, 0), (0, 1), (1, 1), (0, 2)])
def test_mla_weight_precision_modes_and_workgroup_shapes(pv_mode, layout):
    """hi + lo weights (PV mode 1) and the kernel of 16-row tiles (layout 1; layout 2 above 64 rows is the default one)
    against the oracle; 144 heads: several row groups, the last one partial."""
    import paper_2510_14686_amd as xa
    from gpu_util import assert_parity
    lens = [1, 3, 31, 32, 33, 100, 777, 2100]
    q, cs = _case(230 + pv_mode, lens, 1, 144)
    ref_out, ref_lse = oracle.mla(q, cs, lens, DV, SCALE)
    xa.xattn_configure(xa.XATTN_CFG_PV_MODE, pv_mode)
    xa.xattn_configure(xa.XATTN_CFG_MLA_LAYOUT, layout)
    out_bits, lse = gpu_mla(q, cs, lens, SCALE)
    assert_parity(out_bits, lse, ref_out, ref_lse, "mla pv_mode=%d layout=%d" % (pv_mode, layout))


@pytest.mark.parametrize("layout", [1, 2])
@pytest.mark.parametrize("T,H,pv_mode,pieces", [(1, 128, 0, 0), (2, 128, 0, 0), (3, 80, 0, 37), (2, 72, 1, 0), (1, 128, 2, 8),
                                               (4, 40, 0, 1024)])
def test_mla_chosen_layouts(T, H, pv_mode, pieces, layout):
    """The kernel of 16-row tiles (layout 1) and the one of 32-row tiles (layout 2, from 65 query rows per sequence on):
    whole and partial row groups, causal limits inside and across 32-key blocks, every weight mode, ragged lengths,
    several partitions."""
    import paper_2510_14686_amd as xa
    from gpu_util import assert_parity
    lens = [T, T + 1, 31 + T, 32 + T, 33 + T, 64, 129, 200, 640, 1500, 2100]
    q, cs = _case(270 + 10 * T + pv_mode, lens, T, H)
    ref_out, ref_lse = oracle.mla(q, cs, lens, DV, SCALE)
    # Rows of one to four keys put out single value elements: the seeds are chosen so that none reaches
    # 4, from where on rounding the reference itself to bf16 is off by more than the bar (checked here).
    ref = np.asarray(ref_out, dtype=np.float64)
    assert np.abs(bf16_to_f32(f32_to_bf16(ref.astype(np.float32))) - ref).max() < 8e-3
    xa.xattn_configure(xa.XATTN_CFG_MLA_LAYOUT, layout)
    xa.xattn_configure(xa.XATTN_CFG_PV_MODE, pv_mode)
    xa.xattn_configure(xa.XATTN_CFG_PIECES, pieces)
    if pieces:
        xa.xattn_configure(xa.XATTN_CFG_MIN_PIECE_TOKENS, 16)
    out_bits, lse = gpu_mla(q, cs, lens, SCALE)
    assert_parity(out_bits, lse, ref_out, ref_lse, "mla layout=%d T=%d H=%d pv_mode=%d pieces=%d" % (layout, T, H, pv_mode, pieces))


@pytest.mark.parametrize("scale_up", [4.0, 16.0])
def test_mla_peaked_softmax(scale_up):
    """Large scores: a few keys carry nearly all the weight, the case where rounding the weights to
    bf16 shows most (the output is normalised by the sum of the rounded weights)."""
    from gpu_util import assert_parity
    lens = [2, 5, 40, 300, 1500]
    q, cs = _case(240, lens, 2, 32)
    ref_out, ref_lse = oracle.mla(q, cs, lens, DV, SCALE * scale_up)
    out_bits, lse = gpu_mla(q, cs, lens, SCALE * scale_up)
    assert_parity(out_bits, lse, ref_out, ref_lse, "mla peaked x%g" % scale_up)


def test_mla_outlier_value_columns_cost_the_other_columns_nothing():
    """One latent column in eight 512 times larger than the rest (Q's same columns 512 times smaller, so the
    scores do not change): split sequences pass their partial rows in a 16-bit form, and every column,
    large or small, must still meet the bar at its own magnitude."""
    from gpu_util import assert_parity
    lens = [700, 3000, 9000]                       # split over many workgroups
    big = np.arange(5, DV, 8)                      # 64 of the 512 value columns
    q, cs = _case(245, lens, 1, 128)
    qf = bf16_to_f32(q).copy()
    qf[..., big] /= np.float32(512.0)               # powers of two: exact in bf16
    q2 = f32_to_bf16(qf).reshape(q.shape)
    cs2 = []
    for c in cs:
        cf = bf16_to_f32(c).copy()
        cf[:, big] *= np.float32(512.0)
        cs2.append(f32_to_bf16(cf).reshape(c.shape))
    ref_out, ref_lse = oracle.mla(q2, cs2, lens, DV, SCALE)
    out_bits, lse = gpu_mla(q2, cs2, lens, SCALE)
    small = np.setdiff1d(np.arange(DV), big)
    got = bf16_to_f32(out_bits).reshape(ref_out.shape)
    assert_parity(f32_to_bf16(got[..., small]), lse, ref_out[..., small], ref_lse, "mla outliers, ordinary columns")
    assert_parity(f32_to_bf16(got[..., big] / np.float32(512.0)), None, ref_out[..., big] / 512.0, ref_lse,
                  "mla outliers, large columns")


def test_mla_argument_checks():
    import paper_2510_14686_amd as xa
    for args in ((1, 1, 16, 512, 32), (1, 1, 16, 256, 64), (1, 17, 16, 512, 64), (1, 16, 512, 512, 64)):
        with pytest.raises(xa.XattnError) as e:
            xa.xattn_mla_decode(16, 16, 16, *args, 0.1, 16)
        assert e.value.status == xa.binding.XATTN_EUNSUPPORTED
    with pytest.raises(xa.XattnError) as e:
        xa.xattn_mla_decode(0, 16, 16, 1, 1, 16, 512, 64, 0.1, 16)
    assert e.value.status == xa.binding.XATTN_EINVAL
    for bad_scale in (0.0, -0.1, float("inf"), float("nan")):
        with pytest.raises(xa.XattnError) as e:
            xa.xattn_mla_decode(16, 16, 16, 1, 1, 16, 512, 64, bad_scale, 16)
        assert e.value.status == xa.binding.XATTN_EINVAL


@pytest.mark.parametrize("name", ["mla_decode", "mla_verify"])
def test_mla_scaled_down_workloads(name):
    from gpu_util import assert_parity
    w = MLA_CONFIGS[name].scaled(name + "_small", 6, 8)
    lens = w.kv_lens()
    q, cs = w.make_q(), w.make_cache(lens)
    out_bits, lse = gpu_mla(q, cs, lens, w.scale, xtensor=True, seed=w.seed)
    ref_out, ref_lse = oracle.mla(q, cs, lens, w.d_latent, w.scale)
    assert_parity(out_bits, lse, ref_out, ref_lse, w.name)


def test_mla_few_dominant_keys_need_the_exact_weights():
    """Rows that a few keys carry: 16 query tokens on a 16-token sequence (token t sees t + 1 keys) and a
    peaked softmax on longer ones.  Their outputs reach |o| in [2, 4), where rounding the result to bf16
    alone takes up to 7.8e-3 of the 1e-2 bar, so the weights must go into the value product with more
    than 8 bits: the default does that for the first 128 keys of a segment and wherever a key carries a
    quarter of its row.  With one bf16 per weight everywhere (XATTN_CFG_PV_MODE = 2) the same input is
    measurably further from the oracle on exactly those rows."""
    import paper_2510_14686_amd as xa
    from gpu_util import assert_parity, errors
    T, H = 16, 64
    lens = [16, 17, 40, 777, 3000]
    B = len(lens)
    q, cs = _case(260, lens, T, H)
    q = f32_to_bf16(bf16_to_f32(q) * np.float32(3.0))                 # peaked: a few keys per row
    ref_out, ref_lse = oracle.mla(q, cs, lens, DV, SCALE)
    assert np.max(np.abs(ref_out)) > 3.0                               # the case does reach large outputs
    out_bits, lse = gpu_mla(q, cs, lens, SCALE)
    assert_parity(out_bits, lse, ref_out, ref_lse, "mla dominant keys, default weights")
    e_default = errors(out_bits, lse, ref_out, ref_lse)
    xa.xattn_configure(xa.XATTN_CFG_PV_MODE, 2)
    out2, lse2 = gpu_mla(q, cs, lens, SCALE)
    e_single = errors(out2, lse2, ref_out, ref_lse)
    print("max_abs / row rel-L2: default %.2e / %.2e, one bf16 per weight %.2e / %.2e"
          % (e_default[0], e_default[1], e_single[0], e_single[1]), flush=True)
    assert e_default[1] < e_single[1]                                  # the row error shows the weights' precision
