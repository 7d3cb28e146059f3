// Device-side helpers shared by the kernels of libxattn.so: vector types, lane operations, buffer
// loads and stores, and the token-stream partition (paper section 4.4.3, "Layer 3").
#ifndef XATTN_DEVICE_H_
#define XATTN_DEVICE_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "xattn_kernels.h"
#include "xattn_plan.h"

namespace xattn {
namespace {

constexpr int kU = 4;                 // key rows per 16-lane group per block
constexpr int kBlockKeys = 4 * kU;    // key rows per wave per block
constexpr int kRowBytes = kHeadDim * 2;
// Wave-private LDS of the matrix path: a 16-key K block (rows padded to 288 bytes) during the key loop, 256 bytes of 16 output
// rows when a segment is stored.
constexpr int kLdsPerWave = 16 * (kRowBytes + 32);
// A tile's running state in LDS as the lanes hold it: 8 x 16 bytes of sums, (m, l).
constexpr int kLdsPerState = 64 * (8 * 16 + 8);
constexpr float kNegInf = -__builtin_inff();
constexpr float kLn2 = 0.6931471805599453f;

typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_t;
typedef __attribute__((ext_vector_type(4))) float f32x4_t;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4_t;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2_t;
typedef __attribute__((ext_vector_type(2))) float f32x2_t;
typedef __attribute__((ext_vector_type(4))) short s16x4_t;

// ---------------------------------------------------------------------------------- lane helpers
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ const void* uniform(const void* ptr) {
    const uint64_t a = (uint64_t)(uintptr_t)ptr;
    return reinterpret_cast<const void*>((uintptr_t)((uint32_t)uniform((int)(uint32_t)a) | ((uint64_t)(uint32_t)uniform((int)(uint32_t)(a >> 32)) << 32)));
}
__device__ __forceinline__ void* uniform(void* ptr) { return const_cast<void*>(uniform(static_cast<const void*>(ptr))); }
template <int kCtrl>
__device__ __forceinline__ float dpp_f(float x) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), kCtrl, 0xf, 0xf, true));
}
// Sum over the 16 lanes of a DPP row; every lane of the row receives the total.
__device__ __forceinline__ float row16_sum(float x) {
    x += dpp_f<0xB1>(x);    // quad_perm [1,0,3,2]
    x += dpp_f<0x4E>(x);    // quad_perm [2,3,0,1]
    x += dpp_f<0x141>(x);   // row_half_mirror
    x += dpp_f<0x140>(x);   // row_mirror
    return x;
}
// Inclusive sum over the lanes: within rows of 16 by row shifts (lanes shifted in from outside read 0), then
// the rows' totals by the row broadcasts.  No LDS round trips, of which six would be in every prologue.
template <int kCtrl, int kRows>
__device__ __forceinline__ int dpp_add_i(int v) {
    return v + __builtin_amdgcn_update_dpp(0, v, kCtrl, kRows, 0xf, true);
}
__device__ __forceinline__ int wave_incl_scan_i(int v) {
    v = dpp_add_i<0x111, 0xf>(v);   // row_shr:1
    v = dpp_add_i<0x112, 0xf>(v);   // row_shr:2
    v = dpp_add_i<0x114, 0xf>(v);   // row_shr:4
    v = dpp_add_i<0x118, 0xf>(v);   // row_shr:8
    v = dpp_add_i<0x142, 0xa>(v);   // row_bcast:15 into rows 1 and 3
    v = dpp_add_i<0x143, 0xc>(v);   // row_bcast:31 into rows 2 and 3
    return v;
}
__device__ __forceinline__ float dot2_bf16(uint32_t a, uint32_t b, float c) {
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, a), __builtin_bit_cast(bf16x2_t, b), c,
                                           false);
}
__device__ __forceinline__ float bf16_lo(uint32_t x) { return __uint_as_float(x << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t x) { return __uint_as_float(x & 0xffff0000u); }
// Two values rounded to bf16 (nearest even) and packed: the conversion instruction.
__device__ __forceinline__ uint32_t cvt_bf16(float a, float b) {
    const f32x2_t v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// max / sum over the four lanes (kb = 0..3) that hold the same row: lane-swap instructions, no LDS.
// The swap exchanges, between its two register operands, lane group 1 (3) of the first with lane
// group 0 (2) of the second (16-lane form), or the upper half of the first with the lower half of
// the second (32-lane form): called on (x, x), the two results together hold both partners' values.
// (The results are copied to scalars before the bit cast: a bit cast applied directly to an element
// of the result vector read element 0 for both.)
__device__ __forceinline__ void swap16(float x, float& r0, float& r1) {
    const uint32_t a = __builtin_bit_cast(uint32_t, x);
    const u32x2_t t = __builtin_amdgcn_permlane16_swap(a, a, false, false);
    const uint32_t t0 = t.x, t1 = t.y;
    r0 = __builtin_bit_cast(float, t0);
    r1 = __builtin_bit_cast(float, t1);
}
__device__ __forceinline__ void swap32(float x, float& r0, float& r1) {
    const uint32_t a = __builtin_bit_cast(uint32_t, x);
    const u32x2_t t = __builtin_amdgcn_permlane32_swap(a, a, false, false);
    const uint32_t t0 = t.x, t1 = t.y;
    r0 = __builtin_bit_cast(float, t0);
    r1 = __builtin_bit_cast(float, t1);
}
__device__ __forceinline__ float kb_max(float x) {
    float a, b;
    swap16(x, a, b);
    x = fmaxf(a, b);
    swap32(x, a, b);
    return fmaxf(a, b);
}
__device__ __forceinline__ float kb_sum(float x) {
    float a, b;
    swap16(x, a, b);
    x = a + b;
    swap32(x, a, b);
    return a + b;
}
// The same over all lanes; no LDS round trips either.
__device__ __forceinline__ float wave_max(float x) {
    x = fmaxf(x, dpp_f<0xB1>(x));
    x = fmaxf(x, dpp_f<0x4E>(x));
    x = fmaxf(x, dpp_f<0x141>(x));
    return kb_max(fmaxf(x, dpp_f<0x140>(x)));
}
__device__ __forceinline__ float wave_sum(float x) { return kb_sum(row16_sum(x)); }
__device__ __forceinline__ float lane_value(float x, int lane) {      // lane: wave-uniform
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane));
}

// Raw buffer descriptor over [base, base + bytes): loads past the end return 0.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}
// 128-bit non-temporal load at base + voffset (per lane) + soffset (wave-uniform).
__device__ __forceinline__ u32x4_t load_b128_nt(__amdgpu_buffer_rsrc_t rsrc, uint32_t voffset, uint32_t soffset) {
    return __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)voffset, (int)soffset, 2 /* nt */);
}

// Stores of results and partial results: whole rows per instruction (see matrix_finish).  A segment
// that is followed by another one in the same workgroup is written through (sc1): left to the L2's
// write-back policy, its dirty lines are evicted one by one into the saturated read stream later
// (measured on the 16-row workload: 25 MB of partial results cost 37 us of a 400 us kernel, written
// through as full lines 14 us).  A workgroup's last segment keeps the write-back policy: its stores
// complete at the L2 and are flushed in bulk when the kernel ends, which is faster than waiting for
// a write-through at the kernel's tail.
template <bool kWriteThrough>
__device__ __forceinline__ void store_b128(void* base, uint32_t bytes, uint32_t off, u32x4_t v) {
    __builtin_amdgcn_raw_buffer_store_b128(v, make_rsrc(base, bytes), (int)off, 0, kWriteThrough ? 16 /* sc1 */ : 0);
}

// ---------------------------------------------------------------------------------- the plan
// Wave-level front end of the partition in xattn_plan.h.  Every wave computes the plan itself from
// kv_lens (the host never reads the lengths: section 4.2, "Integrating Custom Operators"), in two
// memory round trips (one up to 64 sequences, up to five above 1024) and two wave scans: lane l owns the `chunk` consecutive
// sequences l * chunk .. l * chunk + chunk - 1 (chunk = the power of two >= batch / 64, so at most 64
// for the largest batch) and adds up their stream positions from 128-bit loads, up to 20 lengths of them in
// flight together (above 1024 sequences another round trip for 16 more, see wave_plan); one scan over the 64 lane sums gives the total and every chunk's first position;
// a stream position is then located by one ballot (its chunk) and one scan over that chunk's
// sequences.  The loads go through a buffer descriptor over kv_lens, so indices past the batch read 0.
struct WavePlan {
    Plan pl;
    int chunk, chunk_log2;   // sequences per lane
    int mine;                // stream positions of this lane's sequences
    int excl;                // stream positions before this lane's first sequence
};
// Lengths and base addresses of up to 64 consecutive sequences, one per lane: those around the
// position a wave starts at, fetched in the same round trips as the plan, so that a segment's first
// K/V loads do not wait for another two dependent loads (its length, then its pointers).
struct SeqWindow {
    int base, count;         // sequences base .. base + count - 1 are held
    int len;                 // lane l: clamp_len(kv_lens[base + l])
    u32x2_t k, v;            // lane l: k_ptrs[base + l], v_ptrs[base + l] (v unused by kernels with one pointer array)
};

__device__ __forceinline__ u32x2_t load_ptr_entry(const void* const* ptrs, int batch, int idx) {
    const __amdgpu_buffer_rsrc_t r = make_rsrc(ptrs, (uint32_t)batch * 8u);
    return __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(r, idx * 8, 0, 0));
}
__device__ __forceinline__ void window_load(SeqWindow& win, const int32_t* __restrict__ kv_lens, const void* const* k_ptrs,
                                            const void* const* v_ptrs, int batch, int base, int count, int lane,
                                            int seg_cost, int& positions) {
    const __amdgpu_buffer_rsrc_t rl = make_rsrc(kv_lens, (uint32_t)batch * 4u);
    const int idx = lane < count ? base + lane : batch;            // past the batch: reads 0
    const int raw = (int)__builtin_amdgcn_raw_buffer_load_b32(rl, idx * 4, 0, 0);
    win.k = load_ptr_entry(k_ptrs, batch, idx);
    win.v = v_ptrs ? load_ptr_entry(v_ptrs, batch, idx) : u32x2_t{0u, 0u};
    win.base = base;
    win.count = count;
    win.len = clamp_len(raw);
    positions = stream_len(raw, seg_cost);
}
// Length and pointers of sequence b: from the window when it holds b, else from memory.  Wave-uniform.
__device__ __forceinline__ int window_len(const SeqWindow& win, const int32_t* __restrict__ kv_lens, int b) {
    const unsigned i = (unsigned)(b - win.base);
    if (i < (unsigned)win.count) return __builtin_amdgcn_readlane(win.len, __builtin_amdgcn_readfirstlane((int)i));
    return __builtin_amdgcn_readfirstlane(clamp_len(kv_lens[b]));
}
__device__ __forceinline__ const void* window_ptr(const SeqWindow& win, const u32x2_t& held, const void* const* ptrs, int b) {
    const unsigned i = (unsigned)(b - win.base);
    uint64_t a;
    if (i < (unsigned)win.count) {
        const int li = __builtin_amdgcn_readfirstlane((int)i);
        a = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)held.x, li) |
            ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)held.y, li) << 32);
    } else {
        const uint64_t m = (uint64_t)(uintptr_t)ptrs[b];
        a = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)m) |
            ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(m >> 32)) << 32);
    }
    return reinterpret_cast<const void*>((uintptr_t)a);
}

// Stream positions of up to 16 sequences, `count` of them (a multiple of four) from `first` on.
__device__ __forceinline__ int chunk_positions(__amdgpu_buffer_rsrc_t rl, int first, int count, int seg_cost) {
    u32x4_t v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = __builtin_amdgcn_raw_buffer_load_b128(rl, 4 * k < count ? (first + 4 * k) * 4 : 0x7ffffff0, 0, 0);
    int sum = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        sum += stream_len((int)v[k].x, seg_cost) + stream_len((int)v[k].y, seg_cost) +
               stream_len((int)v[k].z, seg_cost) + stream_len((int)v[k].w, seg_cost);
    return sum;
}

// win (optional): with at most 64 sequences (one per lane) the window is filled here, in the plan's own
// round trip.
__device__ __forceinline__ WavePlan wave_plan(const int32_t* __restrict__ kv_lens, const void* const* k_ptrs,
                                              const void* const* v_ptrs, int batch, int n_pieces, int min_piece,
                                              int seg_cost, int xcd_skew, FewPieces few, int lane, SeqWindow* win, int parts = 1) {
    WavePlan wp;
    const int lg = batch <= 64 ? 0 : 26 - __builtin_clz((unsigned)(batch - 1));      // least with 64 << lg >= batch
    wp.chunk_log2 = lg;
    wp.chunk = 1 << lg;
    const __amdgpu_buffer_rsrc_t rl = make_rsrc(kv_lens, (uint32_t)batch * 4u);
    const int first = lane << lg;
    const PlanRule rule = plan_rule(n_pieces, min_piece, seg_cost, xcd_skew, few, parts);
    int mine;
    if (win) {
        win->base = 0;
        win->count = 0;
    }
    if (lg == 0) {
        if (win) window_load(*win, kv_lens, k_ptrs, v_ptrs, batch, 0, batch, lane, seg_cost, mine);
        else mine = stream_len(__builtin_amdgcn_raw_buffer_load_b32(rl, first * 4, 0, 0), seg_cost);
    } else {
        // Four lengths, at chunk 2 the last two are the next lane's; of longer chunks sixteen more at a time, the first of
        // them in the same round trip.  (A form for every chunk size is code that all calls jump across: of 16 to 100 tokens and 2
        // KV heads, 1500 sequences 30.6 us, 2048 36.9, 4096 63.2, so 27.5, 34.4, 60.8; all 60 at once in a form of their own
        // for the longest chunks 28.7, 35.3, 60.8.)
        const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(rl, first * 4, 0, 0);
        mine = 0;
        for (int k = 4; k < wp.chunk; k += 16) mine += chunk_positions(rl, first + k, wp.chunk - k, seg_cost);
        mine += stream_len((int)v.x, seg_cost) + stream_len((int)v.y, seg_cost);
        if (lg > 1) mine += stream_len((int)v.z, seg_cost) + stream_len((int)v.w, seg_cost);
    }
    const int incl = wave_incl_scan_i(mine);
    wp.mine = mine;
    wp.excl = incl - mine;
    wp.pl = plan_for_total(__builtin_amdgcn_readlane(incl, 63), rule);
    return wp;
}

// The sequence b that holds stream position s (0 <= s < N) and the offset j of s within that
// sequence's L + seg_cost positions.  Both wave-uniform.  With more than 64 sequences the window is
// filled here with the located chunk.
__device__ __forceinline__ void wave_locate(const WavePlan& wp, const int32_t* __restrict__ kv_lens, const void* const* k_ptrs,
                                            const void* const* v_ptrs, int batch, int s, int lane, SeqWindow* win, int& b,
                                            int& j) {
    const unsigned long long hit = __ballot(s >= wp.excl && s < wp.excl + wp.mine);
    const int ln = hit ? __builtin_ctzll(hit) : 0;
    const int off = s - __shfl(wp.excl, ln, 64);
    if (wp.chunk_log2 == 0) {
        b = __builtin_amdgcn_readfirstlane(ln);
        j = __builtin_amdgcn_readfirstlane(off);
        return;
    }
    const int base = ln << wp.chunk_log2;
    int v;
    if (win) {
        window_load(*win, kv_lens, k_ptrs, v_ptrs, batch, base, wp.chunk, lane, wp.pl.seg_cost, v);
    } else {
        const __amdgpu_buffer_rsrc_t rl = make_rsrc(kv_lens, (uint32_t)batch * 4u);
        v = lane < wp.chunk ? stream_len(__builtin_amdgcn_raw_buffer_load_b32(rl, (base + lane) * 4, 0, 0), wp.pl.seg_cost) : 0;
    }
    const int incl = wave_incl_scan_i(v);
    const unsigned long long hit2 = __ballot(off >= incl - v && off < incl);
    const int ln2 = hit2 ? __builtin_ctzll(hit2) : 0;
    b = __builtin_amdgcn_readfirstlane(base + ln2);
    j = __builtin_amdgcn_readfirstlane(off - __shfl(incl - v, ln2, 64));
}

// For the merge kernel: (first partial slot, number of segments) of sequences 64 g .. 64 g + 63, one
// per lane.  A group of 64 sequences holds 64 / chunk whole chunks; a sequence's first position is its
// chunk's first position plus the positions of the chunk's earlier sequences.
__device__ __forceinline__ void wave_write_meta(const WavePlan& wp, const int32_t* __restrict__ kv_lens, int batch, int seq_rows, int g,
                                                int lane, int32_t* __restrict__ meta) {
    const int seq = 64 * g + lane;
    const __amdgpu_buffer_rsrc_t rl = make_rsrc(kv_lens, (uint32_t)batch * 4u);
    const int raw = __builtin_amdgcn_raw_buffer_load_b32(rl, seq * 4, 0, 0);
    __builtin_amdgcn_sched_barrier(0);      // until the next: while the lengths are on their way
    int x = lane, n = batch, rows = seq_rows;
    Plan pl = wp.pl;
    asm volatile("" : "+v"(x), "+s"(n), "+s"(rows), "+s"(pl.total));      // nothing of it ahead of the loop over g, or kept across it
    // lane x: what part x of the batch holds, cut at a lane's first sequence
    const int first = __shfl(wp.excl, batch_part(x & 7, n) >> wp.chunk_log2, 64), from = x < 8 ? first : pl.total;
    const int until = __builtin_amdgcn_update_dpp(0, from, 0x101, 0xf, 0xf, false);      // lane x + 1's
    const bool spread = n >= 8 && __ballot(x < 8 && large_part(pl, until - from, rows)) != 0;
    __builtin_amdgcn_sched_barrier(0);
    const int len = clamp_len(raw);
    const int v = stream_len(len, wp.pl.seg_cost);
    const int before = wave_incl_scan_i(v) - v;                       // within the group
    const int chunk_first = __shfl(wp.excl, (seq >> wp.chunk_log2) & 63, 64);
    const int start = chunk_first + before - __shfl(before, lane & ~(wp.chunk - 1), 64);
    if (seq < batch) {
        const SeqMeta m = seq_meta(wp.pl, seq, start, len);
        reinterpret_cast<int2*>(meta)[seq] = make_int2(m.first_slot, m.n_seg | (spread ? kSpreadRows : 0));
    }
}

// The output row of a merge kernel's workgroup or (kWaves == 1) wave, its sequence and that one's table entry.
struct MergeRow {
    uint32_t row, b;
    int first_slot, n;
};
template <int kWaves, int kRead>
__device__ __forceinline__ MergeRow merge_row(const int32_t* __restrict__ meta, uint32_t batch, uint32_t seq_rows, uint32_t per_xcd, int wave) {
    auto row_of = [&](uint32_t workgroup) { return kWaves == 1 ? workgroup * 4 + wave : workgroup; };
    auto entry = [&](uint32_t b) { return reinterpret_cast<const int2*>(meta)[b]; };
    MergeRow r;
    r.row = row_of(kRead == kReadOwn ? (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3) : blockIdx.x);
    r.b = r.row / seq_rows;
    if constexpr (kRead == kReadOwn) {
        constexpr int kPast = 2 * kSpreadRows;
        const int past = r.b < batch ? 0 : kPast;
        const int2 e = entry(past ? 0 : r.b);
        int slot = e.x, n = e.y | past;
        asm("" : "+s"(slot), "+s"(n));      // both words in one load: the compiler would fetch the slot behind the test
        if (__builtin_expect(n >= kSpreadRows, 0)) {
            r.n = 1;                        // no such row: nothing to do, as for a finished one
            if ((n & kSpreadRows) == 0) return r;
            r.row = row_of(blockIdx.x);
            r.b = r.row / seq_rows;
            if (r.b >= batch) return r;
            const int2 mine = entry(r.b);
            slot = mine.x;
            n = mine.y & (kSpreadRows - 1);
        }
        r.first_slot = slot;
        r.n = n;
    } else {
        r.n = 1;
        if (r.b >= batch) return r;
        const int2 e = entry(r.b);
        r.first_slot = e.x;
        r.n = e.y;
    }
    return r;
}
// A lane's share of a partial row.  (Which form as a branch of one kernel costs 2 % of the short calls.)
template <int kRead, typename T>
__device__ __forceinline__ T load_partial(const T* p) { return kRead == kReadFarOnce ? __builtin_nontemporal_load(p) : *p; }

// The share of a row's n partial results that one of the kWaves waves of a merge workgroup sums.  With few
// of them (`alone`) the first wave takes all: a second round trip costs less than meeting in LDS.
struct MergeShare {
    int first, end;
    bool alone;
};
template <int kWaves>
__device__ __forceinline__ MergeShare merge_share(int n, int wave) {
    MergeShare s;
    s.alone = kWaves == 1 || n <= kMergeAlone;
    const int per = s.alone ? n : (n + kWaves - 1) / kWaves;
    s.first = s.alone ? 0 : wave * per;
    s.end = s.first + per < n ? s.first + per : n;
    return s;
}

}  // namespace
}  // namespace xattn
#endif
