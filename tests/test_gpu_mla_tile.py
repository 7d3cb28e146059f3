"""The latent-KV kernel for more than 32 query rows (a wave per 32 rows) against the oracle."""
import numpy as np
import pytest

import host_lib
import oracle
from workloads import bf16_to_f32
from test_gpu_mla import DV, SCALE, _case, _default_partition, gpu_mla      # noqa: F401  (the fixture resets the knobs)

pytestmark = pytest.mark.gpu

# rows 33 (second wave with one row), 64, 65, 97, 127, 128 (one workgroup), 129, 261 (a row group with 1 and 5 rows);
# lengths around the 32-key block, the four LDS buffers and the four blocks with lo parts of a segment, then long ones
# that are split; keys that carry a row in late blocks (scores times 16: the second pass with the lo parts)
LENS = (1, 31, 32, 33, 64, 65, 97, 127, 128, 129, 160, 161, 193, 700, 2049)


@pytest.mark.parametrize("T,H", [(3, 11), (1, 64), (5, 13), (1, 97), (1, 127), (16, 8), (3, 43), (9, 29)])
@pytest.mark.parametrize("pieces,pv_mode,scale_up", [(0, 0, 1.0), (8, 0, 16.0), (37, 2, 1.0), (1024, 1, 4.0)])
def test_tiles_of_32_rows(T, H, pieces, pv_mode, scale_up):
    import paper_2510_14686_amd as xa
    xa.xattn_configure(xa.XATTN_CFG_PIECES, pieces)
    xa.xattn_configure(xa.XATTN_CFG_PV_MODE, pv_mode)
    if pieces > 256:
        xa.xattn_configure(xa.XATTN_CFG_MIN_PIECE_TOKENS, 16)
    _check(400 + T, [max(T, n) for n in LENS], T, H, scale_up, "T=%d H=%d pieces=%d" % (T, H, pieces))


def _check(seed, lens, T, H, scale_up, what):
    from gpu_util import TOL_LSE, TOL_REL_L2, assert_parity, errors
    # One-key rows put out single value elements: halved values (exact in bf16) keep every output below 4, from
    # where on bf16 rounding of the result alone exceeds the absolute bar.
    q, cs = _case(seed, lens, T, H)
    cs = [(bf16_to_f32(c) * 0.5).astype(np.float32) for c in cs]
    cs = [(c.view(np.uint32) >> 16).astype(np.uint16) for c in cs]
    scale = float(np.float32(2.0 * SCALE * scale_up))
    out_bits, lse = gpu_mla(q, cs, lens, scale)
    ref_out, ref_lse = oracle.mla(q, cs, lens, DV, scale)
    if scale_up == 1.0:
        assert_parity(out_bits, lse, ref_out, ref_lse, what)
        return
    # As in test_few_rows: one key can carry a row, so element by element: rounding to bf16 (half an ulp is at
    # most 2^-8 of the value) and the fp16 partial rows (2^-11 of values up to 5, weights summing to 1).
    _, rel_rows, _, lse_err = errors(out_bits, lse, ref_out, ref_lse)
    diff = np.abs(bf16_to_f32(out_bits).astype(np.float64).reshape(ref_out.shape) - ref_out)
    assert np.all(diff <= 2.0 ** -8 * np.abs(ref_out) + 5 * 2.0 ** -11), what
    assert rel_rows <= TOL_REL_L2 and lse_err <= TOL_LSE, what


def _form(lens, rows, pieces, min_piece):
    """How the kernel runs this partition: waves per tile, blocks of its longest segment, and a segment's exact blocks."""
    least, cost, few, keys = host_lib.mla_cut(rows, len(lens))
    cut = (pieces, min_piece, cost, 0, (0, 1)) if min_piece else (pieces, least, cost, 0, few)
    total, used = host_lib.plan(lens, *cut)
    longest = max(j1 - j0 for p in range(used) for _, j0, j1, _, _ in host_lib.piece_segments(lens, *cut[:3], p, few=cut[4]))
    return host_lib.mla_tile_split(total, used, pieces, rows), -(-int(longest) // keys), host_lib.mla_exact_blocks(used, rows, pieces)


# Up to 64 rows the partition alone decides: two waves per tile in pieces of up to 8 and up to 13 blocks (four exact ones,
# then the pairs of blocks that add the lo parts only where a key dominates), a wave per tile in the longest pieces
@pytest.mark.parametrize("T,H", [(3, 11), (1, 64)])
@pytest.mark.parametrize("pieces,pv_mode,scale_up,waves", [(18, 0, 1.0, 2), (18, 0, 16.0, 2), (30, 0, 16.0, 2), (18, 1, 16.0, 2), (18, 2, 1.0, 2),
                                                           (8, 0, 1.0, 1), (8, 1, 16.0, 1), (8, 2, 1.0, 1)])
def test_up_to_64_rows(T, H, pieces, pv_mode, scale_up, waves):
    import paper_2510_14686_amd as xa
    lens = [max(T, n) for n in LENS]
    split, blocks, exact = _form(lens, T * H, pieces, 0)
    assert split == waves and blocks >= exact + 4
    xa.xattn_configure(xa.XATTN_CFG_PIECES, pieces)
    xa.xattn_configure(xa.XATTN_CFG_PV_MODE, pv_mode)
    _check(460 + T, lens, T, H, scale_up, "T=%d H=%d pieces=%d pv_mode=%d" % (T, H, pieces, pv_mode))


# rows 65 and 97 (the last tile of one row), 128, 129 and 261 (two and three more row groups than without the split);
# pieces of 1 to 5 blocks, all exact, and of up to 14, half of which add the lo parts only where a key dominates
@pytest.mark.parametrize("T,H", [(5, 13), (1, 97), (16, 8), (3, 43), (9, 29)])
@pytest.mark.parametrize("min_piece,pv_mode,scale_up", [(0, 0, 1.0), (0, 1, 1.0), (0, 2, 1.0), (448, 0, 1.0), (448, 0, 16.0), (448, 1, 16.0), (448, 2, 1.0)])
def test_two_waves_per_tile_above_64_rows(T, H, min_piece, pv_mode, scale_up):
    import paper_2510_14686_amd as xa
    lens = [max(T, n) for n in LENS]
    split, blocks, exact = _form(lens, T * H, 128, min_piece)
    assert split == 2 and (blocks > exact + 3 if min_piece else blocks <= exact)
    xa.xattn_configure(xa.XATTN_CFG_PIECES, 128)
    xa.xattn_configure(xa.XATTN_CFG_MIN_PIECE_TOKENS, min_piece)
    xa.xattn_configure(xa.XATTN_CFG_PV_MODE, pv_mode)
    _check(430 + T, lens, T, H, scale_up, "T=%d H=%d pv_mode=%d min_piece=%d" % (T, H, pv_mode, min_piece))


def _moves(q, cs, lens, scale, cut):
    """How often the reference maximum of a row moves behind the first block of a segment: it follows the row's maximum
    when a block of 32 keys exceeds it by more than 2^8."""
    total, used = host_lib.plan(lens, *cut)
    moves = 0
    for p in range(used):
        for b, j0, j1, _, _ in host_lib.piece_segments(lens, *cut[:3], p, few=cut[4]):
            s = bf16_to_f32(q[b, 0]) @ bf16_to_f32(cs[b][j0:j1]).T * (scale * 1.4426950408889634)       # [heads, keys]
            m = s[:, :32].max(axis=1)
            for k in range(32, j1 - j0, 32):
                mx = s[:, k:k + 32].max(axis=1)
                moves += int((mx > m + 8).sum())
                m = np.where(mx > m + 8, mx, m)
    return moves


# one piece (segments of 29 and 11 blocks) and 8 of up to 7 blocks, a wave per tile or, with 64 rows in 8 pieces and 96 in
# 7, two
@pytest.mark.parametrize("H,pieces,min_piece,waves", [(96, 1, 0, 1), (96, 8, 0, 1), (64, 1, 0, 1), (64, 8, 0, 2), (96, 64, 224, 2)])
def test_reference_maximum_that_moves_rescales_every_column(H, pieces, min_piece, waves):
    """Keys whose scores grow along the sequence move the reference maximum of a row inside a segment, in some rows of a
    tile and not in others."""
    import paper_2510_14686_amd as xa
    from gpu_util import TOL_LSE, TOL_REL_L2, errors
    from workloads import f32_to_bf16
    lens = [900, 330]
    q, cs = _case(410, lens, 1, H)
    qf = bf16_to_f32(q).copy()
    qf[..., 0] = np.where(np.arange(H) % 3 == 0, 6.0, 0.0)                  # every third head sees the ramp
    ramped = []
    for c in cs:
        cf = bf16_to_f32(c).copy()
        cf[:, 0] = np.arange(cf.shape[0]) * 0.125                           # up to 112: scores up to 670 * SCALE = 48
        ramped.append(f32_to_bf16(cf).reshape(c.shape))
    q2 = f32_to_bf16(qf).reshape(q.shape)
    least, cost, few, _ = host_lib.mla_cut(H, len(lens))
    cut = (pieces, min_piece, cost, 0, (0, 1)) if min_piece else (pieces, least, cost, 0, few)
    assert _form(lens, H, pieces, min_piece)[0] == waves
    assert _moves(q2, ramped, lens, SCALE, cut) >= 12
    xa.xattn_configure(xa.XATTN_CFG_PIECES, pieces)
    xa.xattn_configure(xa.XATTN_CFG_MIN_PIECE_TOKENS, min_piece)
    ref_out, ref_lse = oracle.mla(q2, ramped, lens, DV, SCALE)
    out_bits, lse = gpu_mla(q2, ramped, lens, SCALE)
    _, rel_rows, _, lse_err = errors(out_bits, lse, ref_out, ref_lse)
    # Element by element: bf16 rounding (half an ulp is at most 2^-8 of the value), the fp16 partial rows (2^-11 of values
    # up to 5, weights summing to 1), and weights of one bf16 (2^-9 each, of keys below a quarter of the row: 2^-11).
    diff = np.abs(bf16_to_f32(out_bits).astype(np.float64).reshape(ref_out.shape) - ref_out)
    assert np.all(diff <= 2.0 ** -8 * np.abs(ref_out) + 10 * 2.0 ** -11)
    assert rel_rows <= TOL_REL_L2 and lse_err <= TOL_LSE


def test_pieces_of_minimal_length_keep_lo_parts_in_all_blocks():
    """Above 64 rows the minimum of 192 positions cuts the number of pieces: the default mode then gives what lo parts
    everywhere give, but for the order of fp32 sums, which moves a rounding to 16 bits now and then."""
    import paper_2510_14686_amd as xa
    lens = [2000] * 8
    split, blocks, exact = _form(lens, 128, 256, 0)
    assert 4 < blocks <= exact
    q, cs = _case(470, lens, 1, 128)
    outs = []
    for pv_mode in (0, 1, 2):
        xa.xattn_configure(xa.XATTN_CFG_PV_MODE, pv_mode)
        outs.append(gpu_mla(q, cs, lens, SCALE)[0])
    differ = [float(np.mean(o != outs[1])) for o in outs]
    print("differ from lo parts everywhere: default %.4f, one bf16 per weight %.4f" % (differ[0], differ[2]), flush=True)
    assert differ[0] < 0.01 and differ[2] > 0.05
