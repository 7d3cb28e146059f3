// Host test library only: the partition of xattn_plan.h (the same code the kernels run) behind C entry
// points, with the wave-parallel steps of the device front end (total, locate) replaced by plain loops.
#include <cstddef>
#include <cstdint>

#include "../xattn_plan.h"

using namespace xattn;

namespace {

Plan plan_of(const int32_t* kv_lens, int batch, int n_pieces, int min_piece, int seg_cost, int xcd_skew, int few_pieces, int few_min) {
    int64_t total = 0;
    for (int b = 0; b < batch; ++b) total += stream_len(kv_lens[b], seg_cost);
    if (total > INT32_MAX) total = -1;          // outside the documented limit: reported, not wrapped
    return plan_for_total((int)total, n_pieces, min_piece, seg_cost, xcd_skew, FewPieces{few_pieces, few_min});
}

}  // namespace

extern "C" {

// total_out: stream positions N (-1 when N would exceed 2^31 - 1); returns the number of pieces in use.
int xattn_test_plan(const int32_t* kv_lens, int batch, int n_pieces, int min_piece, int seg_cost, int xcd_skew, int few_pieces, int few_min, int32_t* total_out) {
    const Plan pl = plan_of(kv_lens, batch, n_pieces, min_piece, seg_cost, xcd_skew, few_pieces, few_min);
    if (total_out) *total_out = pl.total;
    return pl.total < 0 ? -1 : pl.n_pieces;
}

// bounds_out[0 .. n_used]: piece_bound(p) for p = 0 .. n_used.
int xattn_test_piece_bounds(const int32_t* kv_lens, int batch, int n_pieces, int min_piece, int seg_cost, int xcd_skew, int few_pieces, int few_min,
                            int32_t* bounds_out) {
    const Plan pl = plan_of(kv_lens, batch, n_pieces, min_piece, seg_cost, xcd_skew, few_pieces, few_min);
    if (pl.total < 0) return -1;
    for (int p = 0; p <= pl.n_pieces; ++p) bounds_out[p] = piece_bound(pl, p);
    return pl.n_pieces;
}

int xattn_test_piece_of(const int32_t* kv_lens, int batch, int n_pieces, int min_piece, int seg_cost, int xcd_skew, int few_pieces, int few_min, int position) {
    const Plan pl = plan_of(kv_lens, batch, n_pieces, min_piece, seg_cost, xcd_skew, few_pieces, few_min);
    if (pl.total < 0 || position < 0 || position >= pl.total) return -1;
    return piece_of(pl, position);
}

// The segments of piece p as the kernels walk them: rows of (b, j0, j1, slot, whole) in segs_out
// (up to max_segs rows); returns their number.
int xattn_test_piece_segments(const int32_t* kv_lens, int batch, int n_pieces, int min_piece, int seg_cost, int xcd_skew, int few_pieces, int few_min, int p,
                              int32_t* segs_out, int max_segs) {
    const Plan pl = plan_of(kv_lens, batch, n_pieces, min_piece, seg_cost, xcd_skew, few_pieces, few_min);
    if (pl.total < 0 || p < 0 || p >= pl.n_pieces) return -1;
    const int s0 = piece_bound(pl, p), s1 = piece_bound(pl, p + 1);
    // locate: the sequence that holds position s0 and the offset within its positions
    Walk w = {0, 0, s1 - s0};
    int before = 0;
    for (w.b = 0; w.b < batch; ++w.b) {
        const int v = stream_len(kv_lens[w.b], seg_cost);
        if (s0 < before + v) break;
        before += v;
    }
    w.j = s0 - before;
    int n = 0;
    PieceSeg ps;
    while (next_segment(w, batch, seg_cost, [&](int b) { return clamp_len(kv_lens[b]); }, ps)) {
        if (n < max_segs) {
            int32_t* row = segs_out + 5 * n;
            row[0] = ps.b; row[1] = ps.j0; row[2] = ps.j1; row[3] = p + ps.b; row[4] = ps.whole ? 1 : 0;
        }
        ++n;
    }
    return n;
}

// The segments of all parts of all pieces as the matrix path walks them, with their joins: rows of (piece, part, b, j0, j1,
// prev, next, ends) in out (up to max_rows); returns their number.
int xattn_test_part_runs(const int32_t* kv_lens, int batch, int n_pieces, int min_piece, int seg_cost, int xcd_skew, int few_pieces, int few_min,
                         int parts, int32_t* out, int max_rows) {
    const Plan pl = plan_of(kv_lens, batch, n_pieces, min_piece, seg_cost, xcd_skew, few_pieces, few_min);
    if (pl.total < 0) return -1;
    int n = 0;
    for (int p = 0; p < pl.n_pieces; ++p) {
        const int piece0 = piece_bound(pl, p), piece1 = piece_bound(pl, p + 1), sub = part_positions(piece1 - piece0, parts);
        for (int part = 0; part < parts; ++part) {
            const int s0 = piece0 + part * sub, s1 = s0 + sub < piece1 ? s0 + sub : piece1;
            if (s0 >= s1) continue;
            Walk w = {0, 0, s1 - s0};
            int before = 0;
            for (w.b = 0; w.b < batch; ++w.b) {
                const int v = stream_len(kv_lens[w.b], seg_cost);
                if (s0 < before + v) break;
                before += v;
            }
            w.j = s0 - before;
            PieceSeg ps;
            while (next_segment(w, batch, seg_cost, [&](int b) { return clamp_len(kv_lens[b]); }, ps)) {
                const PartRun r = part_run(part, ps.j0, ps.j1, ps.L, piece1 - s1, sub);
                const int32_t row[8] = {p, part, ps.b, ps.j0, ps.j1, r.prev, r.next, r.ends};
                for (int i = 0; i < 8 && n < max_rows; ++i) out[8 * n + i] = row[i];
                ++n;
            }
        }
    }
    return n;
}

// Whether a merge kernel's rows, seq_rows per sequence, are dealt out round robin; the positions before a sequence as a wave's lanes
// of `chunk` sequences know them.
int xattn_test_spread_rows(const int32_t* kv_lens, int batch, int seg_cost, int chunk, int n_pieces, int seq_rows) {
    int total = 0;
    for (int b = 0; b < batch; ++b) total += stream_len(kv_lens[b], seg_cost);
    const Plan pl = plan_for_total(total, n_pieces, 16, seg_cost);
    int at = 0, found = 0;
    for (int x = 1; x <= 8; ++x) {
        const int until = x == 8 ? batch : batch_part(x, batch) / chunk * chunk;
        int next = 0;
        for (int b = 0; b < until; ++b) next += stream_len(kv_lens[b], seg_cost);
        found |= large_part(pl, next - at, seq_rows);
        at = next;
    }
    return found;
}

// KV heads per workgroup and waves per head of the matrix path: heads * 16 + waves.
int xattn_test_piece_share(int n_kv_heads, int max_waves) {
    const PieceShare s = piece_share(n_kv_heads, max_waves);
    return s.heads * 16 + s.parts;
}

// The same of a call on n_cu compute units, whose query rows make row_groups groups; runs_out: share_runs of it and, then, of
// 1 to max_waves heads.
int xattn_test_call_share(int n_cu, int row_groups, int n_kv_heads, int max_waves, int32_t* runs_out) {
    const PieceShare s = call_share(n_cu, row_groups, n_kv_heads, max_waves);
    runs_out[0] = share_runs(n_cu, row_groups, n_kv_heads, s);
    for (int h = 1; h <= max_waves; ++h) runs_out[h] = share_runs(n_cu, row_groups, n_kv_heads, share_of(h, max_waves));
    return s.heads * 16 + s.parts;
}

// How xattn_decode's workgroups share a plan of `total` positions out: count_out[piece in use * rows_total + row] =
// the number of workgroup parts that compute it.  Returns the rows a wave holds in this launch; -1 where a part
// works on a piece that is not in use, or on no row.
int xattn_test_decode_work(int total, int n_pieces, int min_piece, int seg_cost, int xcd_skew, int few_pieces, int few_min, int parts,
                           int rows_total, int rows_max, int32_t* count_out) {
    const Plan pl = plan_for_total(total, n_pieces, min_piece, seg_cost, xcd_skew, FewPieces{few_pieces, few_min});
    const int grid_x = decode_grid_x(n_pieces, parts, rows_total, rows_max);
    int rows = -1;
    for (int bid = 0; bid < grid_x; ++bid)
        for (int part = 0; part < parts; ++part) {
            const DecodeWork w = decode_work(pl, grid_x, parts, rows_total, rows_max, bid, part);
            if (!w.any) continue;
            if (w.piece < 0 || w.piece >= pl.n_pieces || w.row0 < 0 || w.row0 >= rows_total || (rows >= 0 && w.rows != rows)) return -1;
            rows = w.rows;
            for (int r = w.row0; r < rows_total && r < w.row0 + w.rows; ++r) ++count_out[(size_t)w.piece * rows_total + r];
        }
    return rows;
}

// How a latent-KV call above 32 query rows is cut: smallest piece, segment cost, few pieces and their smallest, keys per block.
int xattn_test_mla_cut(int rows_total, int batch, int32_t* out) {
    const int32_t cut[] = {mla_min_piece(rows_total, batch), kMlaSegCost, kMlaFew.pieces, kMlaFew.min_piece, kMlaKeys};
    for (int i = 0; i < 5; ++i) out[i] = cut[i];
    return 0;
}

// The blocks of a segment that run with hi + lo weights, in that call with `used` of n_pieces pieces in use.
int xattn_test_mla_exact_blocks(int used, int rows_total, int n_pieces) {
    return mla_exact_blocks(Plan{0, used, kMlaSegCost, 0}, rows_total, n_pieces);
}

// Waves per tile of mla_tile_kernel in that call, for a plan of `total` positions in `used` pieces.
int xattn_test_mla_tile_split(int total, int used, int n_pieces, int rows_total) {
    return mla_tile_split(Plan{total, used, kMlaSegCost, 0}, n_pieces, rows_total);
}

// How its workgroups share the pieces and tiles out: count_out[piece in use * tiles + tile of 32 rows] = the number of
// workgroups that compute it.  Returns the waves per tile; -1 where a workgroup works on a piece that is not in use, or
// on no row.
int xattn_test_mla_tile_work(int total, int used, int n_pieces, int rows_total, int32_t* count_out) {
    const Plan pl{total, used, kMlaSegCost, 0};
    const int split = mla_tile_split(pl, n_pieces, rows_total), tiles = (rows_total + kTileRows - 1) / kTileRows;
    for (int bid = 0; bid < mla_tile_grid(n_pieces, rows_total); ++bid) {
        const MlaTileWork w = mla_tile_work(pl, split, rows_total, bid);
        if (!w.any) continue;
        if (w.piece < 0 || w.piece >= used || w.row0 < 0 || w.row0 >= rows_total || w.row0 % kTileRows != 0) return -1;
        for (int t = w.row0 / kTileRows; t < tiles && t < w.row0 / kTileRows + kTileWaves / split; ++t) ++count_out[(size_t)w.piece * tiles + t];
    }
    return split;
}

// meta_out[2 b], meta_out[2 b + 1]: (first partial slot, number of segments) of sequence b.
int xattn_test_meta(const int32_t* kv_lens, int batch, int n_pieces, int min_piece, int seg_cost, int xcd_skew, int few_pieces, int few_min, int32_t* meta_out) {
    const Plan pl = plan_of(kv_lens, batch, n_pieces, min_piece, seg_cost, xcd_skew, few_pieces, few_min);
    if (pl.total < 0) return -1;
    int start = 0;
    for (int b = 0; b < batch; ++b) {
        const int len = clamp_len(kv_lens[b]);
        const SeqMeta m = seq_meta(pl, b, start, len);
        meta_out[2 * b] = m.first_slot;
        meta_out[2 * b + 1] = m.n_seg;
        start += stream_len(len, seg_cost);
    }
    return 0;
}

}  // extern "C"
