// The token-stream partition of the decode kernels (paper section 4.4.3, "Layer 3": balance compute
// units by token count, split long sequences, let short ones share a unit) as plain integer code that
// compiles for the device and for the host: the kernels use it through the wave-level front end in
// xattn_device.h, the CPU property tests through host_test/plan_shim.cpp.
//
// All keys of the batch form one stream that is cut into pieces of equal COST.  A sequence of L > 0
// tokens occupies L + seg_cost positions of the stream: its tokens, then seg_cost positions that stand
// for the fixed work every (piece, sequence) segment costs (first loads, Q, the stores of its result),
// so a workgroup whose piece spans a sequence boundary gets correspondingly fewer tokens.  A piece
// bound that falls into those extra positions means "the end of that sequence".  seg_cost = 0 gives
// pieces of equal token count.  Sequences without tokens occupy no positions.
//
// Limits: stream positions are 32-bit.  N = sum_b (L_b + seg_cost) must stay below 2^31, which the
// memory of one GPU guarantees for real caches (2^31 tokens of the smallest supported row, 256 bytes
// of K plus 256 of V, are 1 TiB); n_pieces <= 65536.
#ifndef XATTN_PLAN_H_
#define XATTN_PLAN_H_

#include <stdint.h>

#if defined(__HIPCC__)
#define XATTN_HD __host__ __device__ __forceinline__
#else
#define XATTN_HD inline
#endif

namespace xattn {

constexpr int kPlanRound = 16;        // piece bounds are multiples of the 16-key block (except the last)
constexpr int kMaxPieces = 65536;

struct Plan {
    int total;      // N: positions of the whole stream
    int n_pieces;   // pieces in use: see plan_for_total
    int seg_cost;
    int xcd_skew;   // per mille; see piece_bound
    double inv;     // 1 / (pieces that share a part of the stream: an XCD part with skew, else all of it)
};
constexpr int kMaxXcdSkew = 200;
constexpr int kMinSkewPiece = 32 * kPlanRound;      // positions per piece from which the XCD skew applies

XATTN_HD int clamp_len(int v) { return v > 0 ? v : 0; }
// Stream positions of a sequence of `len` tokens (any sign).
XATTN_HD int stream_len(int len, int seg_cost) { return len > 0 ? len + seg_cost : 0; }

// A short stream is cut finer than min_piece, down to few.min_piece positions, into up to few.pieces
// pieces: as long as that only spreads it over idle compute units, shorter pieces finish earlier.
struct FewPieces {
    int pieces, min_piece;
};
// Every wave works the plan out ahead of its first load, so its quotients are products with an inverse: an integer division
// is some forty dependent instructions, of which a start had a dozen in a row.  floor(a / m) = floor((a + 1/4) / m): the
// product is within 2^-51 of that, relative, and so closer than the 1 / (4 m) that lie between it and the next integer on
// either side, for a < 2^47, a / m < 2^31 and m <= kMaxPieces, or for a < 2^31 and any m.  (That, and less code ahead of the
// first loads: 12 sequences of 100 to 800 tokens, 24 rows of 2 KV heads 12.3 -> 11.8 us; 300 of 30 to 200, 8 rows of 2 17.2 ->
// 16.7; one of 30001 27.7 -> 27.5; 64 of 512 to 4096 level.)
XATTN_HD double plan_inverse(int m) {
#if defined(__HIP_DEVICE_COMPILE__)
    double r = __builtin_amdgcn_rcp((double)m);      // 1 / m to 2^-20 or better, twice as many bits with each step
    r = __builtin_fma(__builtin_fma(-(double)m, r, 1.0), r, r);
    return __builtin_fma(__builtin_fma(-(double)m, r, 1.0), r, r);
#else
    return 1.0 / (double)m;
#endif
}
XATTN_HD int plan_quotient(int a, double inv) { return (int)(((double)a + 0.25) * inv); }

// What the plan of a call follows from beside the lengths, and the inverses of the two minima.
struct PlanRule {
    int n_pieces, min_piece, seg_cost, xcd_skew;
    FewPieces few;
    int parts;
    double inv_min, inv_few;
};
XATTN_HD PlanRule plan_rule(int n_pieces, int min_piece, int seg_cost, int xcd_skew, FewPieces few, int parts) {
    const int least = min_piece > 0 ? min_piece : 1;
    return PlanRule{n_pieces, least, seg_cost, xcd_skew, few, parts, plan_inverse(least), plan_inverse(few.min_piece)};
}
XATTN_HD Plan plan_for_total(int total, const PlanRule& rule) {
    int n = plan_quotient(total, rule.inv_min);
    int n_few = plan_quotient(total, rule.inv_few);
    n_few = n_few < rule.few.pieces ? n_few : rule.few.pieces;
    n = n < n_few ? n_few : n;
    n = n < 1 ? 1 : n;
    Plan pl;
    pl.total = total;
    pl.n_pieces = n < rule.n_pieces ? n : rule.n_pieces;
    pl.seg_cost = rule.seg_cost;
    // the skew needs the eight XCD parts to hold the same number of pieces, and pieces long enough for a
    // few per cent of them to be a block or more (where the `parts` waves of a workgroup share a piece, a wave's share of it)
    const bool can_skew = rule.xcd_skew > 0 && pl.n_pieces % 8 == 0 && total >= (long long)kMinSkewPiece * rule.parts * pl.n_pieces;
    pl.xcd_skew = can_skew ? (rule.xcd_skew < kMaxXcdSkew ? rule.xcd_skew : kMaxXcdSkew) : 0;
    pl.inv = plan_inverse(can_skew ? pl.n_pieces >> 3 : pl.n_pieces);
    return pl;
}
XATTN_HD Plan plan_for_total(int total, int n_pieces, int min_piece, int seg_cost, int xcd_skew = 0, FewPieces few = {0, 1}, int parts = 1) {
    return plan_for_total(total, plan_rule(n_pieces, min_piece, seg_cost, xcd_skew, few, parts));
}

// floor(i * span / m), i <= m <= 65536 (see plan_inverse).
XATTN_HD uint32_t scaled_index(uint32_t i, uint32_t span, double inv_m) { return (uint32_t)(((double)i * (double)span + 0.25) * inv_m); }

// The chip's eight XCDs do not stream at the same rate: measured on MI355X, the odd-numbered ones
// take about 7 % longer than the even-numbered ones for the same bytes, whatever data they are given.
// The kernels hand XCD x the pieces x * n / 8 .. (x + 1) * n / 8 - 1 (consecutive workgroup ids go to
// consecutive XCDs), so the stream is first cut into eight XCD parts, part x starting at
// N * (x + (x odd ? skew : 0)) / 8 (skew = xcd_skew / 1000: even parts are longer by that fraction, odd
// parts shorter), and every part into n / 8 equal pieces.  xcd_skew = 0: eight equal parts.
XATTN_HD uint32_t xcd_part_start(const Plan& pl, int x) {
    // 32-bit arithmetic: N * x / 8 and N * skew / 8000, each as quotient part plus remainder part
    const uint32_t t = (uint32_t)pl.total, ux = (uint32_t)x, sk = (uint32_t)pl.xcd_skew;
    const uint32_t even = (t / 8u) * ux + (t % 8u) * ux / 8u;
    return (x & 1) ? even + (t / 8000u) * sk + (t % 8000u) * sk / 8000u : even;
}

// Piece p owns stream positions [piece_bound(p), piece_bound(p + 1)): floor(p * N / n_pieces) (or its
// skewed counterpart) rounded to the nearest multiple of the 16-key block, so every piece is within
// 16 positions of its exact share and all are used.
XATTN_HD int piece_bound(const Plan& pl, int p) {
    if (p >= pl.n_pieces) return pl.total;
    uint32_t x;
    if (pl.xcd_skew == 0) {
        x = scaled_index((uint32_t)p, (uint32_t)pl.total, pl.inv);
    } else {
        const uint32_t m = (uint32_t)pl.n_pieces / 8u, part = (uint32_t)plan_quotient(p, pl.inv);
        const uint32_t a = xcd_part_start(pl, (int)part), b = xcd_part_start(pl, (int)part + 1);
        x = a + scaled_index((uint32_t)p - part * m, b - a, pl.inv);
    }
    const uint32_t rounded = (x + kPlanRound / 2) / kPlanRound * kPlanRound;
    return rounded < (uint32_t)pl.total ? (int)rounded : pl.total;
}

// The piece that owns stream position x (0 <= x < N): an estimate, corrected against piece_bound.
XATTN_HD int piece_of(const Plan& pl, int x) {
    int p;
    if (pl.xcd_skew == 0) {
        p = (int)((float)x * (float)pl.n_pieces / (float)pl.total);
    } else {
        const int m = pl.n_pieces / 8;
        int part = 0;
        while (part < 7 && xcd_part_start(pl, part + 1) <= (uint32_t)x) ++part;
        const uint32_t a = xcd_part_start(pl, part), b = xcd_part_start(pl, part + 1);
        p = part * m + (int)((float)((uint32_t)x - a) * (float)m / (float)(b - a));
    }
    p = p < 0 ? 0 : (p > pl.n_pieces - 1 ? pl.n_pieces - 1 : p);
    while (p + 1 < pl.n_pieces && piece_bound(pl, p + 1) <= x) ++p;
    while (p > 0 && piece_bound(pl, p) > x) --p;
    return p;
}

// xattn_decode's workgroups.  grid.x = decode_grid_x(...) of them work on the pieces: a workgroup holds `parts`
// pieces, and the query rows of a KV head that a wave cannot hold (rows_max) go to further workgroups.
XATTN_HD int decode_grid_x(int n_pieces, int parts, int rows_total, int rows_max) {
    const int sets = (n_pieces + parts - 1) / parts;         // workgroups of different pieces
    return (sets + 7) / 8 * 8 * ((rows_total + rows_max - 1) / rows_max);
}
struct DecodeWork {
    int piece, row0;      // rows [row0, row0 + rows) of the rows_total
    int rows;             // per wave: rows_max or fewer, the same in the whole launch
    bool any;             // false: nothing to do
};
// What part `part` of workgroup `bid` works on.  Consecutive workgroups go to different XCDs, so each XCD gets
// one contiguous eighth of the token stream.  Of an XCD's workgroups, consecutive ones are the row groups of the
// same pieces: they run at the same time and share the pieces' K and V in that XCD's L2.  A workgroup's parts are
// far apart in the XCD's eighth, so that a short stream's few pieces spread over the compute units.
XATTN_HD DecodeWork decode_work(const Plan& pl, int grid_x, int parts, int rows_total, int rows_max, int bid, int part) {
    const int per_xcd = (pl.n_pieces + 7) >> 3, slots_per_xcd = grid_x >> 3;
    DecodeWork w;
    w.rows = rows_max;
    // When the pieces in use leave enough workgroups idle, every tile of 16 rows gets one of its own (35 rows, 53
    // sequences of 6 to 100 tokens: 17.5 us in pairs, 10.0 us apart).
    const int sets_needed = (per_xcd + parts - 1) / parts;
    if (rows_max == 32 && (rows_total + 15) / 16 * sets_needed <= slots_per_xcd) w.rows = 16;
    const int n_groups = w.rows == rows_max ? (rows_total + rows_max - 1) / rows_max : (rows_total + 15) / 16, slot = bid >> 3;
    const int set = n_groups == 1 ? slot : slot / n_groups;
    const int local = part == 0 ? set : part * (slots_per_xcd / n_groups) + set;
    w.row0 = (slot - set * n_groups) * w.rows;
    w.piece = (bid & 7) * per_xcd + local;
    w.any = (set + 1) * n_groups <= slots_per_xcd && local < per_xcd && w.piece < pl.n_pieces;
    return w;
}

// The matrix path's workgroups: `heads` KV heads, and `parts` waves per head that share a piece, a run of positions each.  A
// sequence that the waves cut among themselves is put together in LDS; only what the piece's own ends cut leaves a
// partial result.
struct PieceShare {
    int heads, parts;
    int inv_heads;      // wave w < 32 is of part w * inv_heads / 32
};
XATTN_HD PieceShare share_of(int heads, int max_waves) { return PieceShare{heads, max_waves / heads, (31 + heads) / heads}; }
// Whether groups of four heads, or else of three, come out even.
XATTN_HD bool even_shares(int n_kv_heads) { return n_kv_heads <= 4 || n_kv_heads % 4 == 0 || n_kv_heads % 3 == 0; }
// Four heads of 256 bytes side by side stream as fast as eight; two cost 2.7 % of a large call, one 6 to 9.
XATTN_HD PieceShare piece_share(int n_kv_heads, int max_waves) {
    return share_of(n_kv_heads < 4 ? n_kv_heads : n_kv_heads % 4 != 0 && n_kv_heads % 3 == 0 ? 3 : 4, max_waves);
}
// Pieces where `on_a_piece` workgroups, those of other KV heads and other query rows counted, work on each: one workgroup per
// compute unit.
XATTN_HD int pieces_of(int n_cu, int on_a_piece) {
    const int pieces = on_a_piece == 1 ? n_cu : n_cu / on_a_piece / 8 * 8;
    return pieces < 8 ? 8 : pieces;
}
// 64 times the number of runs that the waves of a call cut a head's keys into, per round of workgroups: what it has of the chip.  A
// wave per head and piece leaves more partial results and a second round starts anew: an eighth off for each.
XATTN_HD int share_runs(int n_cu, int row_groups, int n_kv_heads, PieceShare s) {
    const int on_a_piece = row_groups * ((n_kv_heads + s.heads - 1) / s.heads), pieces = pieces_of(n_cu, on_a_piece);
    const int rounds = (pieces * on_a_piece + n_cu - 1) / n_cu;
    return 64 * pieces * s.parts / rounds / 8 * (s.parts == 1 ? 7 : 8) / 8 * (rounds > 1 ? 7 : 8);
}
// The share of a call.  Piece counts are multiples of 8 and groups of heads may not come out even, which can leave much of the chip
// idle: then heads are grouped otherwise, where that gives more runs.  (Where up to 32 query rows let a call be bound by memory,
// even groups stay unless the gain is large.)  32 sequences of 512 to 4096 tokens, 40 query rows per KV head, us, with groups of
// four, three or eight heads and so: 5 KV heads 81.7 / 63.3, 10 159.6 / 114.8, 11 162.2 / 134.6, 17 250.5 / 213.5; 24 of them, 18
// 193.6 / 150.0, 27 359.3 / 222.0, 30 373.1 / 235.8, 36 398.9 / 322.2, 40 423.3 / 356.5, 44 410.3 / 381.4; 4 rows, 5 KV heads 39.0 / 37.0, 10
// 57.2 / 50.6, 22 102.6 / 101.6, 33 158.3 / 150.9.  (A wave per piece and KV head: 18, 27 and 36 KV heads 187.0, 272.9, 345.5.)
XATTN_HD PieceShare call_share(int n_cu, int row_groups, int n_kv_heads, int max_waves) {
    PieceShare best = piece_share(n_kv_heads, max_waves);
    int most = share_runs(n_cu, row_groups, n_kv_heads, best);
    const bool stays = row_groups == 1 && even_shares(n_kv_heads);
    // all of the chip, or so much that nothing will change it: no time is spent on a short call
    if (64LL * n_cu * max_waves * (stays ? 5 : 7) <= 7LL * most * row_groups * n_kv_heads) return best;
    const int first = row_groups == 1 ? 4 : 2;
    const int others[] = {first, 6 - first, max_waves, 1};
    for (int h : others) {
        if (h >= n_kv_heads) continue;
        const PieceShare s = share_of(h, max_waves);
        const int runs = share_runs(n_cu, row_groups, n_kv_heads, s);
        if (stays ? runs * 5 <= most * 7 : runs <= most) continue;
        best = s;
        most = runs;
    }
    return best;
}
// Positions per part of a piece of `len` positions, all but the last one's: whole 16-key blocks, so parts without any
// positions come last.  (parts: a power of two.)
XATTN_HD int part_positions(int len, int parts) {
    return ((int)((uint32_t)(len + parts - 1) >> __builtin_ctz((unsigned)parts)) + kPlanRound - 1) / kPlanRound * kPlanRound;
}
// How a part's segment [j0, j1) of a sequence of L tokens joins with its neighbours'.  `left`: positions of the piece behind
// this part's own, `sub`: part_positions.
struct PartRun {
    bool prev;     // its tokens join those of the part before
    int next;      // the parts behind that hold more of the sequence
    bool ends;     // the sequence's last token is in the piece
};
XATTN_HD PartRun part_run(int part, int j0, int j1, int L, int left, int sub) {
    const int rest = L - j1, held = rest < left ? rest : left;
    PartRun r;
    r.prev = part > 0 && j0 > 0;
    r.next = 0;
    while (r.next * sub < held) ++r.next;      // seven at most
    r.ends = rest <= left;
    return r;
}

// What the merge kernel needs to know of a sequence that starts at stream position `start` and has
// `len` tokens: its first partial-result slot and its number of (piece, sequence) segments, i.e. the
// pieces from the one with its first token to the one with its last.  Slot of a segment = piece +
// sequence index (unique: piece and sequence index never both stand still between two segments).
struct SeqMeta { int first_slot, n_seg; };
XATTN_HD SeqMeta seq_meta(const Plan& pl, int b, int start, int len) {
    SeqMeta m;
    if (len <= 0) { m.first_slot = b; m.n_seg = 0; return m; }
    const int first = piece_of(pl, start);
    m.first_slot = first + b;
    m.n_seg = piece_of(pl, start + len - 1) - first + 1;
    return m;
}

// Table entry of a sequence for the merge kernel: its first slot, and its segments (kMaxPieces at most) with, in all entries of
// a call alike, the bit kSpreadRows.  Set: of the eight parts of the batch, whose rows an XCD each would merge (kReadOwn), one holds
// so many of the keys that its XCD would be the last by far, half of them, or 7/32 where the partial rows are many; the rows are then
// dealt out round robin.  One sequence of 30000 tokens among 15 of 100: latent-KV 128 rows 54.6 us by parts, 41.4 round robin, GQA 32
// rows of 8 KV heads 50.8 / 46.5; 8 of 4000 ahead of 56 of 100: 51.0 / 38.7 and 55.1 / 46.5; 4000 among 15 of 20: 24.0 / 21.6 and
// 21.5 / 19.2; 32 of 4000 ahead of 32 of 100, a quarter of the keys in a part: 73.2 / 70.3 and 115.1 / 113.8.  The other way round,
// with less in the largest part or fewer partial rows, a row's second entry is what counts: 23 sequences around 1600, lognormal, 8 rows of
// one KV head 12.5 by parts, 12.9 round robin; 12 of 100 to 800, latent-KV 128 rows 20.4 / 21.0; 1000 among 31 of 50, 4 rows of 8 KV
// heads 10.5 / 10.8; 1000 among 15 of 20, latent-KV 16 rows 11.7 / 12.3.
constexpr int kSpreadRows = 1 << 20;
constexpr int kFewPartialRows = 2048, kManyPartialRows = 16384;
// First sequence of part x (0 to 8) of a batch; whether a part of `positions` calls for round robin.
XATTN_HD int batch_part(int x, int batch) { return x * batch >> 3; }
XATTN_HD bool large_part(const Plan& pl, int positions, int seq_rows) {
    const long long rows = (long long)pl.n_pieces * seq_rows;
    return positions > (pl.total >> 5) * (rows >= kManyPartialRows ? 7 : rows >= kFewPartialRows ? 16 : 32) + 31;
}

// A piece's walk over the sequences it intersects, in stream order.
struct Walk {
    int b;            // next sequence to look at
    int j;            // offset into that sequence's L + seg_cost positions
    int remaining;    // stream positions left in the piece
};
struct PieceSeg {
    int b, L;         // sequence and its length
    int j0, j1;       // tokens [j0, j1) of it
    bool whole;       // the segment is the whole sequence: no partial result, no merge
};
// len_of(b) returns clamp_len(kv_lens[b]).  Returns false when the piece is exhausted.
template <typename LenFn>
XATTN_HD bool next_segment(Walk& w, int batch, int seg_cost, LenFn len_of, PieceSeg& out) {
    while (w.remaining > 0 && w.b < batch) {
        const int L = len_of(w.b);
        if (L == 0) { ++w.b; continue; }
        // the piece's share of this sequence's L + seg_cost positions, and the tokens among them
        const int left = L + seg_cost - w.j;
        const int n_pos = left < w.remaining ? left : w.remaining;
        const int j0 = w.j < L ? w.j : L, j1 = w.j + n_pos < L ? w.j + n_pos : L;
        w.remaining -= n_pos;
        const int bb = w.b;
        ++w.b;
        w.j = 0;
        if (j1 <= j0) continue;                    // only the sequence's extra positions: no tokens
        out.b = bb;
        out.L = L;
        out.j0 = j0;
        out.j1 = j1;
        out.whole = (j0 == 0 && j1 == L);
        return true;
    }
    return false;
}

// ---------------------------------------------------------------- latent-KV calls above 32 query rows
// How their stream is cut, and which softmax weights go into the value product as hi + lo bf16 parts whatever their size
// (see xattn_mla.hip): those of a segment's first mla_exact_blocks() blocks.  The two belong together: a longer piece with
// the same number of such blocks rounds more weights to one bf16.
constexpr int kMlaKeys = 32;                     // keys per block
// A segment's fixed work (Q, the first block's latency and scores, the rounding and stores of the output) in units of
// one token's share of the block loop.  256 would take 2 % off long calls (64 sequences of 1024 to 8192 tokens, 128 rows
// 103.0 -> 100.7 us, 256 rows 173.8 -> 170.6), but makes every piece of an uncut plan longer: more keys behind the first
// kExactBlocks, error against 64 bits 1.69e-3 -> 1.72e-3 (30 sequences of 64 to 256 tokens, 384 rows) and 1.73e-3 ->
// 1.75e-3 (63 of 172 to 688, 48 rows).
constexpr int kMlaSegCost = 192;
constexpr int kExactBlocks = 4;
constexpr int kExactShortBlocks = 7;
constexpr FewPieces kMlaFew = {32, 32};
// Fewest positions per piece.  Above 64 rows a segment's fixed work is worth more tokens, and with few sequences every
// piece is one more partial row to merge.  At least 64 / 128 / 192 / 256 positions per piece, us: 30 sequences of 100 to
// 700 tokens, 72 rows 25.8 / 25.3 / 27.0 / 29.0; 12 of 60 to 900, 144 rows 27.7 / 25.9 / 27.0 / 29.3; 20 of 300 to 1200,
// 128 rows 30.3 / 29.6 / 30.8 / 31.9; 8 of 2000 to 9000 38.8 / 38.8 / 34.9 / 35.9; one of 30000 39.8 / 38.4 / 35.5 / 35.7.
XATTN_HD int mla_min_piece(int rows_total, int batch) { return rows_total <= 64 ? 64 : batch > 8 ? 128 : 192; }
// Where that minimum cuts the number of pieces below the n_pieces that the call may use, all blocks of a piece run with
// hi + lo weights, as they do in pieces of 64: with the minima above and kMlaFew such a piece holds at most 7 blocks.
// (A caller's own minimum, XATTN_CFG_MIN_PIECE_TOKENS, has no such bound.)
XATTN_HD int mla_exact_blocks(const Plan& pl, int rows_total, int n_pieces) {
    return rows_total > 64 && pl.n_pieces < n_pieces ? kExactShortBlocks : kExactBlocks;
}

// mla_tile_kernel's workgroups: four waves, one tile of 32 rows each, or, split, two waves per tile that accumulate half of
// the columns each.  A split block takes 52 MFMAs of a wave instead of 68 and the output's rounding half as long, but the
// chip does 1.5 times the MFMAs and twice the block loads: about 2 us less per segment against 0.15 us more per block,
// hence only where a piece has under 512 positions (segment cost included), and where workgroups would be idle otherwise:
// the rows of a piece take twice as many.  Four waves with a tile each / split, us: 64 rows, 29 sequences of 131 to 262
// tokens 20.5 / 19.3, 32 of 30 to 100 18.5 / 16.7, 4 of 500 to 3000 21.3 / 20.0, 64 of 1024 to 8192 73.8 / 78.8; 72 rows, 16 of
// 20 to 256 21.4 / 18.4; 128 rows, 40 of 64 to 256 28.1 / 24.8, 4 of 500 to 3000 28.9 / 24.5; 256 rows, 16 of 64 to 256 26.1 /
// 22.9.
constexpr int kTileRows = 32;
constexpr int kTileWaves = 4;
constexpr int kTileShortLog2 = 9;
XATTN_HD int mla_tile_grid(int n_pieces, int rows_total) {
    return (n_pieces + 7) / 8 * 8 * ((rows_total + kTileWaves * kTileRows - 1) / (kTileWaves * kTileRows));
}
// Waves per tile of 32 rows: the same in the whole launch.
XATTN_HD int mla_tile_split(const Plan& pl, int n_pieces, int rows_total) {
    const int groups = (rows_total + kTileWaves / 2 * kTileRows - 1) / (kTileWaves / 2 * kTileRows);
    return (pl.total >> kTileShortLog2) < pl.n_pieces && mla_tile_grid(n_pieces, rows_total) >> 3 >= ((pl.n_pieces + 7) >> 3) * groups ? 2 : 1;
}
struct MlaTileWork {
    int piece, row0;      // the workgroup's rows: row0 .. row0 + kTileWaves / split * kTileRows - 1, as far as there are so many
    bool any;             // false: nothing to do
};
// Workgroup ids go round-robin over the 8 XCDs.  Of an XCD's workgroups, consecutive ones are the row groups of one piece:
// they run at the same time on the same XCD and share its L2, so the piece's cache rows come from HBM once.
XATTN_HD MlaTileWork mla_tile_work(const Plan& pl, int split, int rows_total, int bid) {
    const int per_xcd = (pl.n_pieces + 7) >> 3, rows = kTileWaves / split * kTileRows;
    const int groups = (rows_total + rows - 1) / rows, slot = bid >> 3;
    const int local = groups == 1 ? slot : slot / groups;
    MlaTileWork w;
    w.row0 = (slot - local * groups) * rows;
    w.piece = (bid & 7) * per_xcd + local;
    w.any = local < per_xcd && w.piece < pl.n_pieces;
    return w;
}

}  // namespace xattn
#endif
