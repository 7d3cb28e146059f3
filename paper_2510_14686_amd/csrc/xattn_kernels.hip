// Split-KV decode attention and its log-sum-exp merge for gfx950 (MI355X).
//
// Work decomposition (paper section 4.4.3, "Layer 3": balance compute units by token count, split
// long sequences, let short ones share a unit).  The keys of the whole batch form one stream of
// N = sum_b kv_lens[b] tokens, cut into P pieces of N / P tokens (to within one 16-key block); a workgroup
// owns one piece of that stream, whatever sequences it falls in, for up to four KV heads, side by side in
// memory: a wave streams one head's K and V of a run of the piece's tokens (no block table: section 4.3,
// "Operator Adaptation").  Each (piece, sequence) intersection is a segment; the waves that hold runs of it put
// their sums together in LDS.  A segment that covers its whole sequence writes the final result; any other writes an
// un-normalised partial (o, m, l) to slot piece + sequence_index, and the merge kernel combines a sequence's
// slots (the aggregation step of section 4.4.3, "Layer 2").  (A wave per head with a piece and a partial result of
// its own, 8 heads of a piece in a workgroup, before: 64 sequences of 512 to 4096 tokens, 2 KV heads 30.4 us, now
// 29.5; 8 KV heads 92.5 / 91.9; 32 of 1024 to 8192, 32 rows per KV head 130.5 / 119.6, where the partial results were
// 38 MB; one of 30001 27.9 / 26.7.)  Combining inside the decode kernel by the last wave
// to finish a sequence was tried and is slower: that wave alone reads all of a long sequence's
// partials with dependent device-scope loads, while the merge kernel spreads them over the chip.
//
// Loads: 16 lanes hold one 256-byte K (or V) row, 8 bf16 each, one 128-bit non-temporal buffer load
// per lane, so a wave load covers four rows; the buffer descriptor's size is the sequence's byte
// length, so a ragged last block reads zeros instead of memory past the sequence (which an xTensor
// range may not have mapped).  All query rows that share the KV head (GQA group x new tokens:
// section 4.4.1, K is loaded once for all of them and Q stays in registers) use the row from
// registers.  Two inner loops:
//   * vector path (XATTN_CFG_PATH = 1): q.k by bf16 dot2 into fp32, reduced over the 16 lanes with DPP;
//     online softmax in fp32 (log2 domain); p.v by fp32 FMA.
//   * matrix path (one or two tiles of 16 rows per wave; beyond 32 rows several workgroups share a piece.
//     verify, 32 rows per KV head, 165109 tokens: one tile per wave, every piece read twice, 238.6 us; two
//     tiles 130.9 us, of which about 20 are fixed: 38 MB of partial results): the K block is transposed
//     through wave-private LDS into the MFMA operand layout, S^T = K Q^T by bf16 MFMA 16x16x32;
//     softmax on the accumulator layout (a lane holds 4 keys of one row); O^T += V^T P^T by bf16 MFMA
//     16x16x16 straight from the V registers (V never touches LDS), with p fed as three bf16 parts
//     so that it keeps its 24 significant bits.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "xattn_device.h"
#include "xattn_kernels.h"
#include "xattn_launch.h"

namespace xattn {
namespace {

// One (piece, sequence) intersection as seen by one wave.
struct Segment {
    int b, L;            // sequence and its length
    int j0, j1;          // keys [j0, j1) of the sequence
    const void* kp;      // the sequence's K and V ranges
    const void* vp;
    int slot;            // partial-result slot (piece + sequence index)
    bool whole;          // the segment is the whole sequence: write the final result
    int kvh;             // this wave's KV head
    int row0, n_rows;    // query rows [row0, row0 + n_rows) of the head's group * q_len rows
};

// Sequence length in bytes for the buffer descriptor (sequences of 4 GiB or more are not supported).
__device__ __forceinline__ uint32_t seq_bytes(const DecodeParams& prm, int L) {
    const unsigned long long b = (unsigned long long)L * (unsigned)prm.n_kv_heads * kRowBytes;
    return b > 0xffffffffull ? 0xffffffffu : (uint32_t)b;
}

// ---------------------------------------------------------------------------------- vector path
template <int R>
struct RowState {
    float m[R];        // running max of the scaled scores, log2 domain
    float l[R];        // running sum of exp2(s - m)
    float o[R][8];     // running sum of exp2(s - m) * v, this lane's 8 of the 128 columns
};

struct KvBlock {
    u32x4_t k[kU];
    u32x4_t v[kU];
};

// Key rows j_first + 4u + (lane / 16), u = 0..3; soffset carries the wave-uniform part.
__device__ __forceinline__ void load_block(KvBlock& blk, __amdgpu_buffer_rsrc_t rk, __amdgpu_buffer_rsrc_t rv,
                                           uint32_t voffset, uint32_t row_stride, int j_first) {
#pragma unroll
    for (int u = 0; u < kU; ++u) {
        const uint32_t so = (uint32_t)(j_first + 4 * u) * row_stride;
        blk.k[u] = load_b128_nt(rk, voffset, so);
        blk.v[u] = load_b128_nt(rv, voffset, so);
    }
}

// One block of kU key rows per 16-lane group against R query rows.
// j_sub: absolute key index of this lane's row for u = 0 (rows u are 4 apart).  lim_of(r): first key
// index row r may NOT see (segment end and causal limit); used only when kMasked.
template <int R, bool kMasked, typename LimFn>
__device__ __forceinline__ void compute_block(RowState<R>& st, const KvBlock& blk, const uint32_t (&q)[R][4],
                                              float scale_log2, int j_sub, LimFn lim_of) {
    float s[R][kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
        const uint32_t k0 = blk.k[u].x, k1 = blk.k[u].y, k2 = blk.k[u].z, k3 = blk.k[u].w;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            float acc = dot2_bf16(q[r][0], k0, 0.0f);
            acc = dot2_bf16(q[r][1], k1, acc);
            acc = dot2_bf16(q[r][2], k2, acc);
            acc = dot2_bf16(q[r][3], k3, acc);
            acc = row16_sum(acc) * scale_log2;
            if (kMasked) acc = (j_sub + 4 * u < lim_of(r)) ? acc : kNegInf;
            s[r][u] = acc;
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        float mb = s[r][0];
#pragma unroll
        for (int u = 1; u < kU; ++u) mb = fmaxf(mb, s[r][u]);
        const float m_new = fmaxf(st.m[r], mb);
        // While a row has seen no key yet its max is -inf: subtract 0 instead so that exp2 sees
        // -inf (-> 0), not -inf - -inf.
        const float m_use = (kMasked && m_new == kNegInf) ? 0.0f : m_new;
        const float alpha = fast_exp2(st.m[r] - m_use);
        float sum = 0.0f;
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            s[r][u] = fast_exp2(s[r][u] - m_use);
            sum += s[r][u];
        }
        st.l[r] = st.l[r] * alpha + sum;
        st.m[r] = m_new;
#pragma unroll
        for (int e = 0; e < 8; ++e) st.o[r][e] *= alpha;
    }
#pragma unroll
    for (int u = 0; u < kU; ++u) {
        float v[8];
        v[0] = bf16_lo(blk.v[u].x); v[1] = bf16_hi(blk.v[u].x);
        v[2] = bf16_lo(blk.v[u].y); v[3] = bf16_hi(blk.v[u].y);
        v[4] = bf16_lo(blk.v[u].z); v[5] = bf16_hi(blk.v[u].z);
        v[6] = bf16_lo(blk.v[u].w); v[7] = bf16_hi(blk.v[u].w);
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int e = 0; e < 8; ++e) st.o[r][e] = __builtin_fmaf(s[r][u], v[e], st.o[r][e]);
    }
}

// Rows r >= seg.n_rows are padding: they repeat the tile's first row and are never stored.
template <int R>
__device__ __forceinline__ void vector_segment(const DecodeParams& prm, const Segment& seg, int lane) {
    const int sub = lane >> 4, ds = lane & 15;
    const int G = prm.group, T = prm.q_len, Hq = prm.n_q_heads;
    const uint32_t row_stride = (uint32_t)prm.n_kv_heads * kRowBytes;
    const __amdgpu_buffer_rsrc_t rk = make_rsrc(seg.kp, seq_bytes(prm, seg.L));
    const __amdgpu_buffer_rsrc_t rv = make_rsrc(seg.vp, seq_bytes(prm, seg.L));
    const uint32_t voffset = (uint32_t)sub * row_stride + (uint32_t)seg.kvh * kRowBytes + ds * 16;

    // Q rows of this KV head: row r <-> (token t = r / G, head kvh*G + r % G); lane takes columns ds*8..+8.
    auto row_token = [&](int r) { return (seg.row0 + (r < seg.n_rows ? r : 0)) / G; };
    auto row_index = [&](int r) {      // row of [batch*T*Hq]
        const int rr = seg.row0 + (r < seg.n_rows ? r : 0);
        const int t = rr / G;
        return (seg.b * T + t) * Hq + seg.kvh * G + (rr - t * G);
    };
    auto lim_of = [&](int r) {
        const int causal = seg.L - T + row_token(r) + 1;
        return causal < seg.j1 ? causal : seg.j1;
    };
    uint32_t q[R][4];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint4 qv = *reinterpret_cast<const uint4*>(prm.q + (long)row_index(r) * kHeadDim + ds * 8);
        q[r][0] = qv.x; q[r][1] = qv.y; q[r][2] = qv.z; q[r][3] = qv.w;
    }
    // token 0 of the tile has the tightest causal limit
    const int causal0 = seg.L - T + seg.row0 / G + 1;
    const int min_lim = causal0 < seg.j1 ? causal0 : seg.j1;

    RowState<R> st;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        st.m[r] = kNegInf;
        st.l[r] = 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) st.o[r][e] = 0.0f;
    }

    // Full blocks: every key visible to every row.  Two register buffers, the next block's loads are
    // issued before the current block's arithmetic.
    const int n_full = min_lim > seg.j0 ? (min_lim - seg.j0) / kBlockKeys : 0;
    KvBlock A, Bk;
    int blk = 0;
    if (n_full > 0) {
        load_block(A, rk, rv, voffset, row_stride, seg.j0);
        for (; blk + 2 <= n_full; blk += 2) {
            load_block(Bk, rk, rv, voffset, row_stride, seg.j0 + (blk + 1) * kBlockKeys);
            compute_block<R, false>(st, A, q, prm.scale_log2, 0, lim_of);
            if (blk + 2 < n_full) load_block(A, rk, rv, voffset, row_stride, seg.j0 + (blk + 2) * kBlockKeys);
            compute_block<R, false>(st, Bk, q, prm.scale_log2, 0, lim_of);
        }
        if (blk < n_full) compute_block<R, false>(st, A, q, prm.scale_log2, 0, lim_of);
    }
    // Ragged tail and the causally masked last keys.
    for (int jt = seg.j0 + n_full * kBlockKeys; jt < seg.j1; jt += kBlockKeys) {
        load_block(A, rk, rv, voffset, row_stride, jt);
        compute_block<R, true>(st, A, q, prm.scale_log2, jt + sub, lim_of);
    }

    // Combine the four 16-lane groups (each saw every fourth key) into one state per row.
#pragma unroll
    for (int r = 0; r < R; ++r) {
        float m = st.m[r];
        m = fmaxf(m, __shfl_xor(m, 16, 64));
        m = fmaxf(m, __shfl_xor(m, 32, 64));
        const float m_use = (m == kNegInf) ? 0.0f : m;
        const float w = fast_exp2(st.m[r] - m_use);
        float l = st.l[r] * w;
        l += __shfl_xor(l, 16, 64);
        l += __shfl_xor(l, 32, 64);
        st.m[r] = m;
        st.l[r] = l;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            float o = st.o[r][e] * w;
            o += __shfl_xor(o, 16, 64);
            o += __shfl_xor(o, 32, 64);
            st.o[r][e] = o;
        }
    }

    // Store: group `sub` stores rows r with r % 4 == sub.
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (r >= seg.n_rows || (r & 3) != sub) continue;
        if (seg.whole) {
            const long orow = row_index(r);
            const float inv = st.l[r] > 0.0f ? 1.0f / st.l[r] : 0.0f;
            uint4 w;
            w.x = cvt_bf16(st.o[r][0] * inv, st.o[r][1] * inv);
            w.y = cvt_bf16(st.o[r][2] * inv, st.o[r][3] * inv);
            w.z = cvt_bf16(st.o[r][4] * inv, st.o[r][5] * inv);
            w.w = cvt_bf16(st.o[r][6] * inv, st.o[r][7] * inv);
            *reinterpret_cast<uint4*>(prm.out + orow * kHeadDim + ds * 8) = w;
            if (prm.lse && ds == 0)
                prm.lse[orow] = st.l[r] > 0.0f ? (st.m[r] + __log2f(st.l[r])) * kLn2 : kNegInf;
        } else {
            const int t = (seg.row0 + r) / G, g = (seg.row0 + r) - t * G;
            const long prow = (long)seg.slot * (T * Hq) + t * Hq + seg.kvh * G + g;
            float4* po = reinterpret_cast<float4*>(prm.part_o + prow * kHeadDim + ds * 8);
            po[0] = make_float4(st.o[r][0], st.o[r][1], st.o[r][2], st.o[r][3]);
            po[1] = make_float4(st.o[r][4], st.o[r][5], st.o[r][6], st.o[r][7]);
            if (ds == 0) reinterpret_cast<float2*>(prm.part_ml)[prow] = make_float2(st.m[r], st.l[r]);
        }
    }
}

// ---------------------------------------------------------------------------------- matrix path
// Lane (kb, n) = (lane / 16, lane % 16).  Loads: lane holds 16 bytes (chunk n of 16) of key rows
// 4*i + kb, i = 0..3, of the 16-key block, so that a load instruction reads four consecutive 256-byte rows.
// Below, "key 4*kb + i" of a block is the one that lane group kb holds in register i.  (K loaded as the MFMA
// takes it, 64 bytes of each of 16 rows per instruction, needs no LDS and costs 5 to 8 % of the large calls.)
// MFMA index maps (any consistent map of the 128 columns to the contraction index, and of output columns to
// physical columns, is allowed):
//   S^T[key][row] = sum_c K[key][c] Q[row][c]: 16x16x32 step s, lane (kb, x) contracts chunk 4*s + kb
//   O^T_e[x][row] += V[key][8*x + e] P[row][key]: 16x16x4 call (i, e) contracts keys 4*kb + i
// Pitch of a K row in LDS: 2 * odd chunks modulo 16, conflict-free for writes of whole rows and for the
// operand reads, and every access is one address plus a constant.
constexpr int kKPitch = kRowBytes + 32;
struct KvRegs {
    u32x4_t k[4];
    u32x4_t v[4];
};

// The loads of the next block, issued two at a time at four points of the block in hand: eight at once
// ahead of the block cost 2 % of the large calls (long_context 260.8 us all at once, 257.2 us K first and V
// behind the scores, 255.5 us in four pairs).
struct NextLoad {
    KvRegs& r;
    __amdgpu_buffer_rsrc_t rk, rv;
    uint32_t voffset, row_stride;
    int j_block;
    bool on;
    __device__ __forceinline__ void k(int i) const { r.k[i] = load_b128_nt(rk, voffset, (uint32_t)(j_block + 4 * i) * row_stride); }
    __device__ __forceinline__ void v(int i) const { r.v[i] = load_b128_nt(rv, voffset, (uint32_t)(j_block + 4 * i) * row_stride); }
    template <int kPoint>
    __device__ __forceinline__ void at() const {
        if (!on) return;
        if constexpr (kPoint < 2) {
            k(2 * kPoint);
            k(2 * kPoint + 1);
        } else {
            v(2 * kPoint - 4);
            v(2 * kPoint - 3);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    __device__ __forceinline__ void all() const {
#pragma unroll
        for (int i = 0; i < 4; ++i) k(i);
#pragma unroll
        for (int i = 0; i < 4; ++i) v(i);
    }
};
struct NoLoad {
    template <int kPoint>
    __device__ __forceinline__ void at() const {}
};

struct MatrixState {
    f32x4_t o[8];     // O^T tiles: o[e][j] = column 8*(4*kb + j) + e of row n
    float m, l;       // row n: running max (all kb groups agree), this lane's share of the running sum
};

// kPvBf16x3Apart sums the products of the weights' second and third parts apart from the first part's: a part that
// is zero or negative makes NaN of an infinite value, and is dropped at the segment's end where the first part's
// sum is not finite.  (The 32 registers and their rescaling cost 0.3 us of a call; running such a segment once more
// with fp32 products, in a branch that is not taken otherwise, costs 0.5.)
template <int kPv>
constexpr bool kLowApart = kPv == kPvBf16x3Apart;
template <int kPv>
struct LowSums {
    f32x4_t o[kLowApart<kPv> ? 8 : 1];
};

// One 16-key block against kTiles tiles of 16 rows: every K register and every V operand permuted from
// registers feeds the MFMAs of all tiles.
template <int kPv, int kTiles, typename Next>
__device__ __forceinline__ void matrix_block(MatrixState (&st)[kTiles], LowSums<kPv>& low, const KvRegs& r, const bf16x8_t (&qop)[kTiles][4],
                                             char* lds_wave, float scale_log2, int j_block, const int (&lim)[kTiles], int kb,
                                             int n, Next next) {
    next.template at<0>();
    // K block -> wave-private LDS, then back as the MFMA A operand.
#pragma unroll
    for (int i = 0; i < 4; ++i) *reinterpret_cast<u32x4_t*>(lds_wave + (4 * kb + i) * kKPitch + n * 16) = r.k[i];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    next.template at<1>();
    f32x4_t s[kTiles];
#pragma unroll
    for (int t = 0; t < kTiles; ++t) s[t] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int step = 0; step < 4; ++step) {
        const bf16x8_t a = *reinterpret_cast<const bf16x8_t*>(lds_wave + n * kKPitch + (4 * step + kb) * 16);
#pragma unroll
        for (int t = 0; t < kTiles; ++t) s[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, qop[t][step], s[t], 0, 0, 0);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

    next.template at<2>();
    // s[t][i] = score of the key in register i, row 4*i + kb of the block, for row n of tile t
    float p[kTiles][4];
#pragma unroll
    for (int t = 0; t < kTiles; ++t) {
#pragma unroll
        for (int i = 0; i < 4; ++i) p[t][i] = s[t][i] * scale_log2;
        if (__builtin_amdgcn_ballot_w64(j_block + kBlockKeys > lim[t]) != 0) {      // only blocks that reach a limit
#pragma unroll
            for (int i = 0; i < 4; ++i) p[t][i] = (j_block + 4 * i + kb < lim[t]) ? p[t][i] : kNegInf;
        }
        const float mx = kb_max(fmaxf(fmaxf(p[t][0], p[t][1]), fmaxf(p[t][2], p[t][3])));
        // The reference is the exact running maximum: no weight exceeds 1, so a sum stays as far inside the fp32
        // range as its values allow, and the largest key's weight is exactly 1 in any number of bf16 parts.
        const bool moves = mx > st[t].m;
        if (__builtin_amdgcn_ballot_w64(moves) != 0) {
            const float m_new = moves ? mx : st[t].m;
            const float alpha = moves ? fast_exp2(st[t].m - m_new) : 1.0f;
            const bool first = __builtin_amdgcn_ballot_w64(moves && st[t].m != kNegInf) == 0;      // all sums are still 0
            st[t].m = m_new;
            st[t].l *= alpha;
            if (!first) {
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    st[t].o[e] *= alpha;
                    if constexpr (kLowApart<kPv>) low.o[e] *= alpha;
                }
            }
        }
        const float m_use = (st[t].m == kNegInf) ? 0.0f : st[t].m;
#pragma unroll
        for (int i = 0; i < 4; ++i) p[t][i] = fast_exp2(p[t][i] - m_use);
        st[t].l += (p[t][0] + p[t][1]) + (p[t][2] + p[t][3]);
    }
    next.template at<3>();
    if (kPv == kPvFp32) {
        // O^T_e += V_i[e] (x) p_i over the 4 key groups: fp32 MFMA, p exact.
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float v[8];
            v[0] = bf16_lo(r.v[i].x); v[1] = bf16_hi(r.v[i].x);
            v[2] = bf16_lo(r.v[i].y); v[3] = bf16_hi(r.v[i].y);
            v[4] = bf16_lo(r.v[i].z); v[5] = bf16_hi(r.v[i].z);
            v[6] = bf16_lo(r.v[i].w); v[7] = bf16_hi(r.v[i].w);
#pragma unroll
            for (int t = 0; t < kTiles; ++t)
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    st[t].o[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[e], p[t][i], st[t].o[e], 0, 0, 0);
        }
    } else {
        // bf16 MFMA 16x16x16 contracts the block's 16 keys at once: lane (kb, x) supplies keys 4*kb + i,
        // i = 0..3, of column 8*x + e (the e-th bf16 of its four V registers) and of row n (its four p).
        // kPvBf16x3 feeds p as three bf16 parts in three MFMAs, which keeps all of its 24 significant bits.  (Two
        // parts keep 16 of them, and the 2^-17 of the largest weight is then the error of a row that one key
        // carries, ahead of the output's rounding.  The third costs 0 to 0.3 % of the large calls, 1 % with two
        // tiles, 2 % of 64 sequences of two KV heads.)
        constexpr bool kLo = kPv == kPvBf16x3 || kPv == kPvBf16x3Apart;
        u32x2_t ph[kTiles], pl[kTiles], pr[kTiles];
#pragma unroll
        for (int t = 0; t < kTiles; ++t) {
            const f32x2_t p01 = {p[t][0], p[t][1]}, p23 = {p[t][2], p[t][3]};
            const bf16x2_t h01 = __builtin_convertvector(p01, bf16x2_t), h23 = __builtin_convertvector(p23, bf16x2_t);
            ph[t] = u32x2_t{__builtin_bit_cast(uint32_t, h01), __builtin_bit_cast(uint32_t, h23)};
            pl[t] = pr[t] = u32x2_t{0u, 0u};
            if (kLo) {
                const f32x2_t r01 = p01 - __builtin_convertvector(h01, f32x2_t);
                const f32x2_t r23 = p23 - __builtin_convertvector(h23, f32x2_t);
                const bf16x2_t l01 = __builtin_convertvector(r01, bf16x2_t), l23 = __builtin_convertvector(r23, bf16x2_t);
                pl[t] = u32x2_t{__builtin_bit_cast(uint32_t, l01), __builtin_bit_cast(uint32_t, l23)};
                const f32x2_t q01 = r01 - __builtin_convertvector(l01, f32x2_t);
                const f32x2_t q23 = r23 - __builtin_convertvector(l23, f32x2_t);
                pr[t] = u32x2_t{cvt_bf16(q01[0], q01[1]), cvt_bf16(q23[0], q23[1])};
            }
        }
        const uint32_t vw[4][4] = {{r.v[0].x, r.v[0].y, r.v[0].z, r.v[0].w}, {r.v[1].x, r.v[1].y, r.v[1].z, r.v[1].w},
                                   {r.v[2].x, r.v[2].y, r.v[2].z, r.v[2].w}, {r.v[3].x, r.v[3].y, r.v[3].z, r.v[3].w}};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const uint32_t sel = (e & 1) ? 0x07060302u : 0x05040100u;      // high or low halves of both words
            const u32x2_t a = {__builtin_amdgcn_perm(vw[1][e >> 1], vw[0][e >> 1], sel),
                               __builtin_amdgcn_perm(vw[3][e >> 1], vw[2][e >> 1], sel)};
#pragma unroll
            for (int t = 0; t < kTiles; ++t) {
                st[t].o[e] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4_t, a),
                                                                       __builtin_bit_cast(s16x4_t, ph[t]), st[t].o[e], 0, 0, 0);
                if (kLo) {
                    f32x4_t& lo = kLowApart<kPv> ? low.o[kLowApart<kPv> ? e : 0] : st[t].o[e];
                    lo = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4_t, a),
                                                                   __builtin_bit_cast(s16x4_t, pr[t]), lo, 0, 0, 0);
                    lo = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4_t, a),
                                                                   __builtin_bit_cast(s16x4_t, pl[t]), lo, 0, 0, 0);
                }
            }
        }
    }
}

// A segment in flight on the matrix path: its per-lane constants, its Q operand and the loads of its
// first block.  matrix_begin issues the loads, matrix_run consumes the blocks, matrix_finish stores.
// The kernel begins the next segment before it finishes the current one, so that the new
// segment's first loads are not queued behind the old segment's stores (a wave's memory operations
// complete in order, and a store's completion takes several microseconds under a saturated read
// stream) and the read stream does not drain at a segment boundary.
template <int kTiles>
struct MatrixCtx {
    Segment seg;
    __amdgpu_buffer_rsrc_t rk, rv;
    uint32_t voffset;
    bf16x8_t qop[kTiles][4];
    int lim[kTiles];  // first key index row n of the tile may not see
    KvRegs first;     // block 0
};

// Row r of the segment's rows <-> (token t, head kvh*G + g).  r / G as a product with 1 / G: (r + 1/2) / G is
// at least 1 / (2 G) >= 2^-7 away from an integer (G <= 64), far more than the product's rounding.
__device__ __forceinline__ int row_token(const DecodeParams& prm, int r) { return (int)(((float)r + 0.5f) * prm.inv_group); }
__device__ __forceinline__ int seq_row(const DecodeParams& prm, const Segment& seg, int r) {      // row within the sequence
    const int rr = seg.row0 + r;
    const int t = row_token(prm, rr);
    return t * prm.n_q_heads + seg.kvh * prm.group + (rr - t * prm.group);
}

template <int kTiles>
__device__ __forceinline__ void matrix_begin(MatrixCtx<kTiles>& c, const DecodeParams& prm, const Segment& seg, int lane) {
    const int kb = lane >> 4, n = lane & 15;
    const uint32_t row_stride = (uint32_t)prm.n_kv_heads * kRowBytes;
    c.seg = seg;
    c.rk = make_rsrc(seg.kp, seq_bytes(prm, seg.L));
    c.rv = make_rsrc(seg.vp, seq_bytes(prm, seg.L));
    c.voffset = (uint32_t)kb * row_stride + (uint32_t)seg.kvh * kRowBytes + n * 16;
    NextLoad{c.first, c.rk, c.rv, c.voffset, row_stride, seg.j0, true}.all();
    // Q through a descriptor over the sequence's rows: rows past n_rows lie past its end and read as zero.
    const int seq_rows = prm.q_len * prm.n_q_heads;
    const __amdgpu_buffer_rsrc_t rq = make_rsrc(prm.q + (long)seg.b * seq_rows * kHeadDim, (uint32_t)(seq_rows * kRowBytes));
#pragma unroll
    for (int t = 0; t < kTiles; ++t) {
        const bool row_ok = 16 * t + n < seg.n_rows;
        const int r = row_ok ? 16 * t + n : 0;
        const int qoff = (row_ok ? seq_row(prm, seg, r) : seq_rows) * kRowBytes + kb * 16;
#pragma unroll
        for (int step = 0; step < 4; ++step)
            c.qop[t][step] = __builtin_bit_cast(bf16x8_t, __builtin_amdgcn_raw_buffer_load_b128(rq, qoff + 64 * step, 0, 0));
        const int causal = seg.L - prm.q_len + row_token(prm, seg.row0 + r) + 1;
        c.lim[t] = causal < seg.j1 ? causal : seg.j1;
    }
}

template <int kPv, int kTiles>
__device__ __forceinline__ void matrix_run(MatrixState (&st)[kTiles], MatrixCtx<kTiles>& c, const DecodeParams& prm, int lane,
                                           char* lds_wave) {
    const int kb = lane >> 4, n = lane & 15;
    const uint32_t row_stride = (uint32_t)prm.n_kv_heads * kRowBytes;
    const Segment& seg = c.seg;
#pragma unroll
    for (int t = 0; t < kTiles; ++t) {
#pragma unroll
        for (int e = 0; e < 8; ++e) st[t].o[e] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
        st[t].m = kNegInf;
        st[t].l = 0.0f;
    }
    static_assert(!kLowApart<kPv> || kTiles == 1, "one tile's registers");
    LowSums<kPv> low;
    if constexpr (kLowApart<kPv>)
#pragma unroll
        for (int e = 0; e < 8; ++e) low.o[e] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    // Two register buffers: the next block's 8 loads per lane go out during the current block's arithmetic.
    const int n_blocks = (seg.j1 - seg.j0 + kBlockKeys - 1) / kBlockKeys;
    auto key0 = [&](int blk) { return seg.j0 + blk * kBlockKeys; };
    KvRegs Bk;
    int blk = 0;
    for (; blk + 2 <= n_blocks; blk += 2) {
        matrix_block<kPv, kTiles>(st, low, c.first, c.qop, lds_wave, prm.scale_log2, key0(blk), c.lim, kb, n,
                                  NextLoad{Bk, c.rk, c.rv, c.voffset, row_stride, key0(blk + 1), true});
        matrix_block<kPv, kTiles>(st, low, Bk, c.qop, lds_wave, prm.scale_log2, key0(blk + 1), c.lim, kb, n,
                                  NextLoad{c.first, c.rk, c.rv, c.voffset, row_stride, key0(blk + 2), blk + 2 < n_blocks});
    }
    if (blk < n_blocks)
        matrix_block<kPv, kTiles>(st, low, c.first, c.qop, lds_wave, prm.scale_log2, key0(blk), c.lim, kb, n, NoLoad());
    if constexpr (kLowApart<kPv>) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float sum = st[0].o[e][j] + low.o[e][j];
                st[0].o[e][j] = __builtin_amdgcn_fmed3f(sum, sum, st[0].o[e][j]);      // of a NaN and o: o
            }
    }
}

// Stores the 16 rows of tile t of the segment; rows past the last get an offset past the descriptor's end,
// and their stores are dropped.
constexpr uint32_t kPastTheEnd = 0x40000000u;
template <bool kWriteThrough>
__device__ __forceinline__ void matrix_finish(const MatrixState& st, const Segment& seg, int tile, const DecodeParams& prm,
                                              int lane, char* lds_wave) {
    const int kb = lane >> 4, n = lane & 15;
    const int seq_rows = prm.q_len * prm.n_q_heads;
    const int n_rows = seg.n_rows - 16 * tile;
    const float l = kb_sum(st.l);
    // Store through LDS so that every store instruction writes whole contiguous rows (a lane's own
    // accumulators are 16-byte pieces of 16 different rows).
    auto fence = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    if (seg.whole) {
        constexpr int kPitch = kRowBytes + 16;                   // bf16 rows, padded against bank conflicts
        const float inv = l > 0.0f ? 1.0f / l : 0.0f;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            uint4 w;
            w.x = cvt_bf16(st.o[0][j] * inv, st.o[1][j] * inv);
            w.y = cvt_bf16(st.o[2][j] * inv, st.o[3][j] * inv);
            w.z = cvt_bf16(st.o[4][j] * inv, st.o[5][j] * inv);
            w.w = cvt_bf16(st.o[6][j] * inv, st.o[7][j] * inv);
            *reinterpret_cast<uint4*>(lds_wave + n * kPitch + (4 * kb + j) * 16) = w;
        }
        fence();
#pragma unroll
        for (int i = 0; i < 4; ++i) {                             // 4 rows of 256 bytes per store instruction
            if (4 * i >= n_rows) break;
            const int r = 4 * i + (lane >> 4);
            const uint32_t off = (uint32_t)seq_row(prm, seg, 16 * tile + r) * kRowBytes + (lane & 15) * 16;
            const u32x4_t w = *reinterpret_cast<const u32x4_t*>(lds_wave + r * kPitch + (lane & 15) * 16);
            store_b128<kWriteThrough>(prm.out + (long)seg.b * seq_rows * kHeadDim, (uint32_t)(seq_rows * kRowBytes),
                          off | (r < n_rows ? 0u : kPastTheEnd), w);
        }
        if (n < n_rows && prm.lse && kb == 0)
            prm.lse[(long)seg.b * seq_rows + seq_row(prm, seg, 16 * tile + n)] = l > 0.0f ? (st.m + __log2f(l)) * kLn2 : kNegInf;
    } else {
        constexpr int kPitch = kRowBytes + 16;                   // half a row in fp32, padded: lanes kb < 2 hold the first halves
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            if ((kb >> 1) == half) {
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    float4* w = reinterpret_cast<float4*>(lds_wave + n * kPitch + (4 * (kb & 1) + j) * 32);
                    w[0] = make_float4(st.o[0][j], st.o[1][j], st.o[2][j], st.o[3][j]);
                    w[1] = make_float4(st.o[4][j], st.o[5][j], st.o[6][j], st.o[7][j]);
                }
            }
            fence();
#pragma unroll
            for (int i = 0; i < 4; ++i) {                         // 256 bytes of 4 rows per store instruction
                if (4 * i >= n_rows) break;
                const int r = 4 * i + (lane >> 4);
                const uint32_t off = (uint32_t)seq_row(prm, seg, 16 * tile + r) * (kHeadDim * 4) + half * kRowBytes + (lane & 15) * 16;
                const u32x4_t w = *reinterpret_cast<const u32x4_t*>(lds_wave + r * kPitch + (lane & 15) * 16);
                store_b128<kWriteThrough>(prm.part_o + (long)seg.slot * seq_rows * kHeadDim, (uint32_t)(seq_rows * kHeadDim * 4),
                                          off | (r < n_rows ? 0u : kPastTheEnd), w);
            }
            if (half == 0) fence();
        }
        if (n < n_rows && kb == 0) {
            const long prow = (long)seg.slot * seq_rows + seq_row(prm, seg, 16 * tile + n);
            reinterpret_cast<float2*>(prm.part_ml)[prow] = make_float2(st.m, l);
        }
    }
    fence();      // the next tile, or the next segment's K blocks, reuse this LDS
}

// The state of a tile, left in LDS by the wave that holds a later run of the sequence's keys, and added to the own one by the
// wave that holds the first.
__device__ __forceinline__ void state_put(const MatrixState& st, char* area, int lane) {
#pragma unroll
    for (int e = 0; e < 8; ++e) *reinterpret_cast<f32x4_t*>(area + e * 1024 + lane * 16) = st.o[e];
    *reinterpret_cast<float2*>(area + 8192 + lane * 8) = make_float2(st.m, st.l);
}
__device__ __forceinline__ void state_add(MatrixState& st, const char* area, int lane) {
    const float2 ml = *reinterpret_cast<const float2*>(area + 8192 + lane * 8);
    const float m = fmaxf(st.m, ml.x), m_use = m == kNegInf ? 0.0f : m;
    const float mine = fast_exp2(st.m - m_use), other = fast_exp2(ml.x - m_use);
    st.m = m;
    st.l = st.l * mine + ml.y * other;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const f32x4_t o = *reinterpret_cast<const f32x4_t*>(area + e * 1024 + lane * 16);
#pragma unroll
        for (int j = 0; j < 4; ++j) st.o[e][j] = __builtin_fmaf(o[j], other, st.o[e][j] * mine);
    }
}

// ---------------------------------------------------------------------------------- decode kernel
// grid.x = workgroups of pieces times groups of R query rows, grid.z = groups of KV heads.  Matrix path: a workgroup works on
// one piece, share.heads KV heads in share.parts waves each (see piece_share).  Vector path: up to 8 KV heads and `parts`
// pieces, one wave per KV head and piece.
// kMatrix selects the matrix path (R must be 16 * kTiles then).
// Fixed work of a (piece, sequence) segment in token units for the partition (0 = pieces of equal token
// count; 16 measured best of 0 / 16 / 48: 0.2 to 1 % on the four large workloads).
constexpr int kGqaSegCost = 16;

// What the plan needs are arguments of their own, not members of prm: the first 14 words of scalar arguments are in registers
// when a wave starts (see build.py), so the loads of the lengths, or a merge kernel's of its table, do not wait for one of
// their addresses.  All kernels so, 0.4 to 0.5 us per launch: 695 tokens 9.5 -> 8.7 us, one sequence of 3000 12.4 -> 11.5, 300 of 30 to
// 200 16.5 -> 15.4, one of 30001 27.4 -> 26.6, 64 of 512 to 4096 92.5 -> 92.0, latent-KV 40 of 50 to 200, 16 rows 11.3 -> 10.5.
template <int R, bool kMatrix, int kPv>
__global__ __launch_bounds__(512) void split_decode_kernel(const int32_t* __restrict__ kv_lens, const void* const* k_ptrs, const void* const* v_ptrs,
                                                           int batch, int n_pieces, int min_piece, int few_pieces, int few_min,
                                                           int xcd_skew, uint32_t share, int grid_x, DecodeParams prm) {
    constexpr int kTiles = kMatrix ? R / 16 : 1;
    // Behind the waves' own parts: the states of all waves of a workgroup but the first of every KV head.
    constexpr int kStates = (kMaxWavesPerBlock - 1) * kTiles;
    __shared__ __attribute__((aligned(16))) char lds[kMatrix ? kMaxWavesPerBlock * kLdsPerWave + kStates * kLdsPerState : 16];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int heads = kMatrix ? (int)(share & 255u) : prm.n_kv_heads < kMaxWavesPerBlock ? prm.n_kv_heads : kMaxWavesPerBlock;
    const int parts = kMatrix ? (int)(share >> 8 & 255u) : prm.parts;
    const int part = parts == 1 ? 0 : kMatrix ? wave * (int)(share >> 16) >> 5 : wave / heads;
    const int kvh = blockIdx.z * heads + wave - part * heads;
    if (!kMatrix && kvh >= prm.n_kv_heads) return;
    // A piece's first segment takes its length and pointers from the plan's own round trips, which saves a start two
    // dependent loads (138468 tokens of 2 KV heads 31.7 -> 31.1 us, of 8 94.3 -> 93.2).  Only the first: kept longer the
    // window's registers cost the large calls up to 1.7 %.  Not with two tiles: that kernel's registers are full, and
    // those the window spills cost it 17 %.
    constexpr bool kWindow = kTiles == 1;
    SeqWindow win;
    SeqWindow* const window = kWindow ? &win : nullptr;
    const void* const* const win_k = kWindow ? k_ptrs : nullptr;
    const void* const* const win_v = kWindow ? v_ptrs : nullptr;
    const WavePlan wp = wave_plan(kv_lens, win_k, win_v, batch, n_pieces, min_piece, kGqaSegCost, xcd_skew, FewPieces{few_pieces, few_min},
                                  lane, window, kMatrix ? parts : 1);
    const Plan& pl = wp.pl;

    const int bid = blockIdx.x;
    const int rows_total = prm.group * prm.q_len;
    const DecodeWork work = decode_work(pl, grid_x, kMatrix ? 1 : parts, rows_total, R, bid, kMatrix ? 0 : part);
    const int p = work.piece, rows = work.rows;
    const int piece0 = piece_bound(pl, p), piece1 = piece_bound(pl, p + 1);
    const int sub = kMatrix ? part_positions(piece1 - piece0, parts) : piece1 - piece0;
    const int s0 = kMatrix ? piece0 + part * sub : piece0, s1 = s0 + sub < piece1 ? s0 + sub : piece1;

    // Unlikely, so that this code stands behind the rest and not between the plan and the first loads, and the likely answer needs
    // no load (the workgroup's size is one): 0.5 and 0.3 us of a short call, 695 tokens 8.6 -> 7.9, 300 sequences of 30 to 200 15.5 ->
    // 14.7, 64 of 512 to 4096 91.7 -> 91.3.
    if (__builtin_expect(64 * (grid_x - 1 - bid) < batch && blockIdx.z == 0 && wave == heads * parts - 1, 0)) {
        // For the merge kernel: first partial slot and number of segments of every sequence, 64
        // sequences per wave, the groups of 64 dealt out over the workgroups from the last one, which
        // has no piece of its own when the stream is short.  Of such a workgroup the last wave, which a short piece leaves
        // without keys (30 sequences of 100 to 900 tokens of one KV head by the first wave 11.4 us, by the last 10.9).
        for (int g = grid_x - 1 - bid; 64 * g < batch; g += grid_x) wave_write_meta(wp, kv_lens, batch, prm.q_len * prm.n_q_heads, g, lane, prm.meta);
    }
    if (!work.any || piece0 >= piece1) return;      // the whole workgroup on the matrix path
    if (!kMatrix && s0 >= s1) return;
    const bool active = s0 < s1 && kvh < prm.n_kv_heads;

    Walk walk;
    if (active) wave_locate(wp, kv_lens, win_k, win_v, batch, s0, lane, window, walk.b, walk.j);
    walk.remaining = uniform(s1 - s0);

    Segment seg;
    seg.kvh = kvh;
    seg.row0 = work.row0;
    seg.n_rows = rows_total - seg.row0 < rows ? rows_total - seg.row0 : rows;
    // Next (piece, sequence) intersection of this piece, in stream order; false when the piece is done.
    auto next_seg = [&](Segment& out, auto first) {
        constexpr bool kFirst = kWindow && decltype(first)::value;
        PieceSeg ps;
        auto len_of = [&](int b) {
            if constexpr (kFirst) return window_len(win, kv_lens, b);
            else return __builtin_amdgcn_readfirstlane(clamp_len(kv_lens[b]));
        };
        if (!next_segment(walk, batch, pl.seg_cost, len_of, ps)) return false;
        // Everything about a segment is wave-uniform; said so, it lives in scalar registers, and the loads
        // through its descriptors need no loop over the lanes' values.
        out = seg;
        out.b = uniform(ps.b);
        out.kp = kFirst ? window_ptr(win, win.k, k_ptrs, out.b) : uniform(k_ptrs[out.b]);
        out.vp = kFirst ? window_ptr(win, win.v, v_ptrs, out.b) : uniform(v_ptrs[out.b]);
        out.L = uniform(ps.L);
        out.j0 = uniform(ps.j0);
        out.j1 = uniform(ps.j1);
        out.slot = uniform(p) + out.b;
        out.whole = uniform(ps.whole);
        return true;
    };
    if constexpr (kMatrix) {
        char* lds_wave = lds + wave * kLdsPerWave;
        auto run_piece = [&](auto tiles) {
            constexpr int kT = decltype(tiles)::value;
            char* const lds_head = lds + kMaxWavesPerBlock * kLdsPerWave + (wave - part * heads) * (kT * kLdsPerState);
            auto state_of = [&](int of_part, int t) { return lds_head + (of_part - 1) * heads * (kT * kLdsPerState) + t * kLdsPerState; };
            MatrixState st[kT];
            MatrixCtx<kT> cur;
            auto put = [&] {
#pragma unroll
                for (int t = 0; t < kT; ++t) state_put(st[t], state_of(part, t), lane);
            };
            bool have = false;
            if (active) {
                Segment first;
                have = uniform(next_seg(first, std::true_type())) != 0;
                if (have) matrix_begin(cur, prm, first, lane);
            }
            if (have) {
                for (;;) {
                    matrix_run<kPv, kT>(st, cur, prm, lane, lds_wave);
                    Segment nxt_seg;
                    if (uniform(next_seg(nxt_seg, std::false_type())) == 0) break;
                    MatrixCtx<kT> nxt;
                    matrix_begin(nxt, prm, nxt_seg, lane);     // its loads go out before cur's stores
                    if (part > 0 && cur.seg.j0 > 0) {
                        put();
                    } else {
#pragma unroll
                        for (int t = 0; t < kT; ++t) matrix_finish<true>(st[t], cur.seg, t, prm, lane, lds_wave);
                    }
                    cur = nxt;
                }
            }
            // The last segment: what the wave before began goes to LDS, what this wave begins is put together there.
            PartRun run = {false, 0, false};
            if (have) run = part_run(part, cur.seg.j0, cur.seg.j1, cur.seg.L, piece1 - s1, sub);
            if (have && run.prev) put();
            if (parts > 1) __syncthreads();
            if (!have || run.prev) return;
            for (int q = part + 1; q <= part + run.next; ++q)
#pragma unroll
                for (int t = 0; t < kT; ++t) state_add(st[t], state_of(q, t), lane);
            cur.seg.whole = cur.seg.j0 == 0 && run.ends;
#pragma unroll
            for (int t = 0; t < kT; ++t) matrix_finish<false>(st[t], cur.seg, t, prm, lane, lds_wave);
        };
        if (kTiles == 2 && rows == 16) run_piece(std::integral_constant<int, 1>());
        else run_piece(std::integral_constant<int, kTiles>());
    } else {
        Segment s2;
        for (bool more = next_seg(s2, std::true_type()); more; more = next_seg(s2, std::false_type())) vector_segment<R>(prm, s2, lane);
    }
}

// ---------------------------------------------------------------------------------- merge kernel
// Aggregation of the partial results of split sequences (section 4.4.3, "Layer 2"):
//   M = max_s m_s;  l = sum_s l_s 2^(m_s - M);  out = sum_s o_s 2^(m_s - M) / l;  lse = (M + log2 l) ln 2
// kWaves waves per output row (b, t, h); lane holds columns 2*lane, 2*lane+1.  Sequences with a single
// segment were finished by the decode kernel and are skipped; sequences without keys get out = 0 and
// lse = -inf here.
// Bound by its dependent steps (table; records and partial rows; every further 8 partial rows), not by bytes: one wave
// per row took 21.4 us for one sequence of 30001 tokens (32 rows of 256 slots); sixteen waves that each sum a share of
// the slots and meet once in LDS take 5.2 us.  For the same reason a lane fetches one slot's record and takes its
// weight while the first 8 partial rows are on their way, weights pass by lane reads, and the row's sequence comes
// from a 32-bit division (the whole call, with a shuffle per weight and a 64-bit division before: 138468 tokens of 2 KV
// heads 32.3 -> 31.8 us; 695 tokens level, 8.9).
// kRead = kReadFarOnce: one of 30000 tokens, 32 rows of 8 KV heads 39.3 -> 37.0 us; 4 of 2000 to 16000, 16 rows 28.3 -> 27.3.
template <int kWaves, int kRead>
__global__ __launch_bounds__(kWaves == 1 ? 256 : 64 * kWaves) void merge_kernel(const int32_t* __restrict__ meta, const float* __restrict__ part_ml,
                                                                                const float* __restrict__ part_o, uint16_t* __restrict__ out,
                                                                                float* __restrict__ lse, int batch, uint32_t seq_rows, uint32_t per_xcd) {
    const int lane = threadIdx.x & 63;
    const int wave = uniform(threadIdx.x >> 6);
    const MergeRow mr = merge_row<kWaves, kRead>(meta, (uint32_t)batch, seq_rows, per_xcd, wave);
    const uint32_t row = mr.row, b = mr.b;
    const int n = mr.n;
    if (n == 1) return;
    const MergeShare sh = merge_share<kWaves>(n, wave);
    if (sh.alone && kWaves > 1 && wave > 0) return;       // few slots: the first wave does the row
    uint32_t* outp = reinterpret_cast<uint32_t*>(out + (long)row * kHeadDim) + lane;
    if (n == 0) {
        *outp = 0u;
        if (lse && lane == 0) lse[row] = kNegInf;
        return;
    }
    const long stride_rows = seq_rows, first_row = (long)mr.first_slot * stride_rows + (row - b * seq_rows);
    const float2* ml = reinterpret_cast<const float2*>(part_ml) + first_row;
    const f32x2_t* po = reinterpret_cast<const f32x2_t*>(part_o + first_row * kHeadDim) + lane;
    // Lane i holds (m, l) of slot first + i of the current group of 64 slots; the first 8 slots' partial
    // rows are requested in the same breath, so a typical row (up to 8 segments) costs one round trip.
    float M = kNegInf, l = 0.0f, o0 = 0.0f, o1 = 0.0f;
    if (sh.first < sh.end) {
        float2 mine = make_float2(kNegInf, 0.0f);
        if (sh.first + lane < sh.end) mine = ml[(sh.first + lane) * stride_rows];
        f32x2_t o[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {                     // (the last row again past the end: 2 to 5 % of short calls)
            o[u] = f32x2_t{0.0f, 0.0f};
            if (sh.first + u < sh.end) o[u] = load_partial<kRead>(&po[(sh.first + u) * stride_rows * (kHeadDim / 2)]);
        }
        M = mine.x;
        for (int base = sh.first + 64; base < sh.end; base += 64)
            if (base + lane < sh.end) M = fmaxf(M, ml[(base + lane) * stride_rows].x);
        M = wave_max(M);
        const float m_use = (M == kNegInf) ? 0.0f : M;
        float w = fast_exp2(mine.x - m_use);               // lanes past the end: 0
        l = mine.y * w;
        for (int i0 = 0; sh.first + i0 < sh.end; i0 += 8) {
            const int s0 = sh.first + i0;
            if (i0 > 0) {
                if ((i0 & 63) == 0) {
                    mine = (s0 + lane < sh.end) ? ml[(s0 + lane) * stride_rows] : make_float2(kNegInf, 0.0f);
                    w = fast_exp2(mine.x - m_use);
                    l = __builtin_fmaf(mine.y, w, l);
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) o[u] = load_partial<kRead>(&po[(s0 + u < sh.end ? s0 + u : sh.end - 1) * stride_rows * (kHeadDim / 2)]);
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const float w_s = lane_value(w, (i0 + u) & 63);
                const bool in = s0 + u < sh.end;          // past the end: nothing, also where the row read is infinite
                o0 = __builtin_fmaf(in ? o[u].x : 0.0f, w_s, o0);
                o1 = __builtin_fmaf(in ? o[u].y : 0.0f, w_s, o1);
            }
        }
        l = wave_sum(l);
    }
    if constexpr (kWaves > 1) {
        if (!sh.alone) {                                  // the waves' sums, each against its own maximum, meet in LDS
            __shared__ float2 part[kWaves][64], wave_ml[kWaves];
            part[wave][lane] = make_float2(o0, o1);
            if (lane == 0) wave_ml[wave] = make_float2(M, l);
            __syncthreads();
            if (wave > 0) return;
#pragma unroll
            for (int w = 1; w < kWaves; ++w) M = fmaxf(M, wave_ml[w].x);
            const float m_use = (M == kNegInf) ? 0.0f : M;
            l = o0 = o1 = 0.0f;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                const float f = fast_exp2(wave_ml[w].x - m_use);
                l = __builtin_fmaf(wave_ml[w].y, f, l);
                o0 = __builtin_fmaf(part[w][lane].x, f, o0);
                o1 = __builtin_fmaf(part[w][lane].y, f, o1);
            }
        }
    }
    const float inv = l > 0.0f ? 1.0f / l : 0.0f;
    *outp = cvt_bf16(o0 * inv, o1 * inv);
    if (lse && lane == 0) lse[row] = l > 0.0f ? (M + __log2f(l)) * kLn2 : kNegInf;
}

// ---------------------------------------------------------------------------------- write_kvcache
// One workgroup per (sequence, new token): copies the token's K row and V row (n_kv_heads * 256 bytes
// each) to row kv_len - q_len + t of the sequence's ranges, 16 bytes per lane, one half of the workgroup the
// K row and the other the V row.  Bound by its round trips: the rows are read while the length and the
// addresses are fetched (256 sequences of 2 KB rows, the call behind an append: 57.9 -> 57.3 us).
__global__ __launch_bounds__(256) void write_kvcache_kernel(const uint16_t* __restrict__ k_new, const uint16_t* __restrict__ v_new, void* const* k_ptrs,
                                                            void* const* v_ptrs, const int32_t* __restrict__ kv_lens, int q_len, int row_bytes) {
    const int b = blockIdx.x / q_len, t = blockIdx.x - b * q_len;
    const bool is_v = threadIdx.x >= 128;
    const char* src = reinterpret_cast<const char*>(is_v ? v_new : k_new) + (long)blockIdx.x * row_bytes;
    const int first = (threadIdx.x & 127) * 16;
    uint4 x = make_uint4(0u, 0u, 0u, 0u);
    if (first < row_bytes) x = *reinterpret_cast<const uint4*>(src + first);
    const long pos = (long)kv_lens[b] - q_len + t;
    char* dst = static_cast<char*>(is_v ? v_ptrs[b] : k_ptrs[b]) + pos * row_bytes;
    if (pos < 0) return;
    for (int i = first; i < row_bytes; i += 128 * 16) {
        if (i != first) x = *reinterpret_cast<const uint4*>(src + i);
        *reinterpret_cast<uint4*>(dst + i) = x;
    }
}

template <int R, bool kMatrix, int kPv = kPvBf16x3>
hipError_t launch_decode_r(const DecodeParams& prm, dim3 grid, dim3 block, hipStream_t stream) {
    const uint32_t share = (uint32_t)prm.share.heads | (uint32_t)prm.share.parts << 8 | (uint32_t)prm.share.inv_heads << 16;
    return launch(split_decode_kernel<R, kMatrix, kPv>, grid, (int)block.x, stream, prm.kv_lens, prm.k_ptrs, prm.v_ptrs, prm.batch,
                  kMatrix ? prm.shared_pieces : prm.n_pieces, prm.min_piece_tokens, prm.few.pieces, prm.few.min_piece, prm.xcd_skew,
                  share, (int)grid.x, prm);
}

}  // namespace

hipError_t launch_write_kvcache(const WriteParams& prm, hipStream_t stream) {
    return launch(write_kvcache_kernel, dim3((unsigned)(prm.batch * prm.q_len)), 256, stream, prm.k_new, prm.v_new, prm.k_ptrs, prm.v_ptrs,
                  prm.kv_lens, prm.q_len, prm.row_bytes);
}

// Measured on MI355X, the matrix path is the faster one from a single query row per KV head up, although most
// of a tile is then padding: it keeps the next segment's loads ahead of the stores, and the calls are bound by
// HBM.  138468 tokens of 8 KV heads, 1 / 2 / 3 rows: vector path 95.4 / 97.2 / 99.0 us, matrix path 92.8 /
// 93.0 / 93.2; 80 to 700 tokens 9.1 -> 8.7 and 11.0 -> 10.5; no shape tried was slower by more than 1 %.  The
// weights keep 24 bits there: the error against 64 bits is the vector path's to seven digits on eight shapes
// (1.656835e-3, which is the output's own rounding).  The vector path stays as a second computation of the same
// function that shares none of the matrix path's layouts, for cross-checks.
bool use_matrix_path(int path) { return path != kPathVector; }

int rows_per_wave(int rows_total, int path) {
    if (use_matrix_path(path)) return rows_total <= 16 ? 16 : 32;
    static const int kSizes[] = {1, 2, 3, 4, 5, 6, 8};
    for (int s : kSizes)
        if (rows_total <= s) return s;
    return 8;
}

hipError_t launch_decode(const DecodeParams& prm, hipStream_t stream, hipEvent_t* events) {
    const int rows_total = prm.group * prm.q_len;
    const bool matrix = use_matrix_path(prm.path);
    const int R = rows_per_wave(rows_total, prm.path);
    const int heads = matrix ? prm.share.heads : prm.n_kv_heads < kMaxWavesPerBlock ? prm.n_kv_heads : kMaxWavesPerBlock;
    const int grid_x = matrix ? decode_grid_x(prm.shared_pieces, 1, rows_total, R) : decode_grid_x(prm.n_pieces, prm.parts, rows_total, R);
    const dim3 grid(grid_x, 1, (prm.n_kv_heads + heads - 1) / heads), block(64 * heads * (matrix ? prm.share.parts : prm.parts));
    hipError_t e;
    if (events && (e = hipEventRecord(events[0], stream)) != hipSuccess) return e;
    if (matrix && R == 32) {
        switch (prm.pv_mode) {
            case kPvBf16: e = launch_decode_r<32, true, kPvBf16>(prm, grid, block, stream); break;
            case kPvFp32: e = launch_decode_r<32, true, kPvFp32>(prm, grid, block, stream); break;
            default: e = launch_decode_r<32, true, kPvBf16x3>(prm, grid, block, stream); break;
        }
    } else if (matrix) {
        // The weight modes are the matrix path's from 4 rows per KV head on; below, where a call comes here by
        // default, its weights have 24 bits in every mode and its sums take infinite values, as on the vector path.
        switch (rows_total < 4 && (prm.path != kPathMatrix || prm.pv_mode == kPvBf16x3) ? kPvBf16x3Apart : prm.pv_mode) {
            case kPvBf16x3Apart: e = launch_decode_r<16, true, kPvBf16x3Apart>(prm, grid, block, stream); break;
            case kPvBf16: e = launch_decode_r<16, true, kPvBf16>(prm, grid, block, stream); break;
            case kPvFp32: e = launch_decode_r<16, true, kPvFp32>(prm, grid, block, stream); break;
            default: e = launch_decode_r<16, true, kPvBf16x3>(prm, grid, block, stream); break;
        }
    } else {
        switch (R) {
            case 1: e = launch_decode_r<1, false>(prm, grid, block, stream); break;
            case 2: e = launch_decode_r<2, false>(prm, grid, block, stream); break;
            case 3: e = launch_decode_r<3, false>(prm, grid, block, stream); break;
            case 4: e = launch_decode_r<4, false>(prm, grid, block, stream); break;
            case 5: e = launch_decode_r<5, false>(prm, grid, block, stream); break;
            case 6: e = launch_decode_r<6, false>(prm, grid, block, stream); break;
            default: e = launch_decode_r<8, false>(prm, grid, block, stream); break;
        }
    }
    if (e != hipSuccess) return e;
    if (events && (e = hipEventRecord(events[1], stream)) != hipSuccess) return e;
    const long rows = (long)prm.batch * prm.q_len * prm.n_q_heads;
    // Fewer than 256 rows are read as fast either way, or 0.2 us faster through the L2s.
    e = launch_merge<256>(rows, prm.batch, [&](auto waves, auto read, unsigned grid) {
        constexpr int kWaves = decltype(waves)::value;
        return launch(merge_kernel<kWaves, decltype(read)::value>, dim3(grid), kWaves == 1 ? 256 : 64 * kWaves, stream, prm.meta, prm.part_ml,
                      prm.part_o, prm.out, prm.lse, prm.batch, (uint32_t)(prm.q_len * prm.n_q_heads), grid >> 3);
    });
    if (e != hipSuccess) return e;
    if (events && (e = hipEventRecord(events[2], stream)) != hipSuccess) return e;
    return hipSuccess;
}

}  // namespace xattn
