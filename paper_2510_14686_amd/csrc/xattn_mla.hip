// Latent-KV (MLA-shaped) split-KV decode attention for gfx950 (MI355X).
//
// The operator the paper itself adapts (section 4.3 "Operator Adaptation": attention on a contiguous
// virtual range, no block table; section 4.4.1 "MLA Optimization": the m+1 query tokens and all
// heads are multiplied with the same cached rows, K is loaded once for all of them and Q stays
// resident).  Per token the cache holds one row of 576 bf16 (512 latent + 64 rope) that is the key of
// every head, and whose first 512 values are every head's value.  With 128 heads that is 242 flop per
// cached byte: the path is bound by the matrix cores and what feeds them, with 16 rows by HBM.
//
// Partition: the same token-stream pieces as the GQA kernel (section 4.4.3, "Layer 3").  A workgroup owns one piece and
// up to 128 query rows (row = token * n_heads + head), and walks the piece in 32-key blocks that all its waves share
// through LDS.  Three kernels by the number of rows per sequence:
//   * up to 32: mla_rows_kernel, four waves per tile of 16 rows;
//   * more: mla_tile_kernel, one wave per tile of 32 rows, in short pieces two;
//   * mla_decode_kernel, one wave per tile of 16 rows, four tiles at most (XATTN_CFG_MLA_LAYOUT = 1): a second computation
//     of the same function that shares neither the layouts nor the MFMA shape of the others, for cross-checks.
// Common to them (the figures are mla_decode_kernel's):
//   * a block (32 x 1152 bytes, contiguous in memory) goes from HBM straight into LDS (buffer loads
//     with the LDS destination, 1 KiB per wave instruction, no staging registers), once per
//     workgroup, two blocks in flight during the arithmetic.  In LDS the latent and the rope part of the rows sit in two
//     areas laid out against bank conflicts (the LDS side of such a load is fixed to lane order, so
//     the layout is made through the global address each lane fetches);
//   * S^T = C Q^T: per 16-key tile 18 bf16 MFMA 16x16x32, the A operand (keys) read from LDS;
//   * softmax on the accumulator layout: lane (kb, n) holds, of row n, the keys 4 kb + i of both key
//     tiles, which is exactly the B operand (8 keys per lane) of the next product, so the weights
//     never leave the lane; row maxima cross the lane groups with lane-swap instructions; the
//     reference maximum of a row moves only when a block exceeds it by more than 2^8, so the
//     accumulators are rescaled about once per segment instead of in most blocks;
//   * O^T += C[:, 0:512]^T P^T: bf16 MFMA over the 32 keys, the A operand (value columns x
//     8 keys per lane) fetched with LDS transposing reads.  A weight enters the product as one bf16
//     where it is small against the row's sum, and as hi + lo bf16 parts (two MFMAs, 16 significant
//     bits) where it is not: in the first mla_exact_blocks() blocks of every segment, whose keys' share of
//     the final sum is not yet known, and in any later block that holds a key with at least 1/4 of
//     the row's running sum (of any row of the tile).  The output is normalised by the sum of the weights as they
//     entered the product.  (Rounding every weight to one bf16 costs nothing on diffuse rows, where the
//     errors average out; where a few keys carry the row, outputs are large enough for bf16 output
//     rounding to use up most of the tolerance, and the weights' own 2^-9 no longer fits beside it.)
// A segment that is not a whole sequence leaves its rows in the workspace as fp16, scaled by the
// row's largest magnitude, with (m, l, lq, 1 / scale) in fp32; the merge kernel combines them.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "xattn_device.h"
#include "xattn_kernels.h"
#include "xattn_launch.h"

namespace xattn {
namespace {

constexpr int kDqk = 576;                        // key width: latent + rope
constexpr int kDv = 512;                         // value width: the latent part
constexpr int kRowB = kDqk * 2;                  // 1152 bytes per cached token
// LDS image of a block: the first 1024 bytes of each row (the latent part, 64 chunks of 16 bytes) at
// pitch kPitch, the last 128 bytes (the rope part) in a tail area at pitch kTailPitch.  Both pitches are
// 2 * odd chunks modulo 16: measured, that serves the operand reads below without bank conflicts (an
// odd pitch halves their rate).
constexpr int kPitch = 1024 + 32;                // 1056
constexpr int kTailPitch = 128 + 32;             // 160
constexpr int kTailRowsPerLoad = 6;              // one wave-wide load fills the tails of 6 rows (60 lanes)
constexpr int kTailLoads = (kMlaKeys + kTailRowsPerLoad - 1) / kTailRowsPerLoad;          // 6
constexpr int kTailOff = kMlaKeys * kPitch;      // 33792: start of the tail area
constexpr int kLdsBlock = kTailOff + (kTailLoads - 1) * kTailRowsPerLoad * kTailPitch + 1024;   // 39616
constexpr int kDmaPerBlock = kMlaKeys + kTailLoads;   // 38 wave-wide loads of 64 x 16 bytes
constexpr int kTileB = 16 * kPitch;              // from key tile 0 to key tile 1 of a block
constexpr int kTailTileB = 16 * kTailPitch;
constexpr int kMainSteps = 1024 / 64;            // MFMA steps 0..15 read the latent part, 16..17 the tail
constexpr int kQSteps = kDqk / 32;               // 18 MFMA steps of 32 columns
constexpr int kQRegSteps = 13;                   // Q columns 0 .. 32 * 13 - 1 stay in registers, the rest of Q in LDS
constexpr int kQLdsWave = (kQSteps - kQRegSteps) * 1024;   // per 16-row tile: one 16-byte chunk per lane and step
constexpr int kQAhead = 2;                       // key fragments in flight ahead of the MFMAs, in steps
constexpr int kVAhead = 2;                       // value fragments in flight ahead of the MFMAs, in tile pairs
constexpr int kColTiles = kDv / 16;              // 32 tiles of 16 value columns
constexpr int kStagePitch = (kDv / 2) * 2 + 16;  // epilogue: 16 rows x 256 16-bit columns at a time per wave, padded rows
constexpr int kStageWave = 16 * kStagePitch;     // 8448 bytes
constexpr float kLazyLog2 = 8.0f;                // slack of the softmax reference maximum, in powers of two
// Precision of the softmax weights in the value product (see the header comment).
constexpr int kLoNever = 0;                      // one bf16 per weight everywhere
constexpr int kLoAlways = 1;                     // hi + lo bf16 parts everywhere
constexpr int kLoDynamic = 2;                    // default mode: hi + lo parts in a segment's first blocks (mla_exact_blocks),
                                                 // then only in blocks with a dominant key
constexpr float kDominantShare = 4.0f;           // a key is dominant from 1 / 4 of the row's running sum
constexpr int kStages = 3;                       // LDS block buffers: two blocks in flight behind the one in use

typedef short s16x4v_t __attribute__((ext_vector_type(4)));

// Running state of one 16-row tile.  Lane (kb, n) holds row n.
struct MlaTile {
    f32x4_t o[kColTiles];      // o[ct][i]: column 16 ct + 4 kb + i
    float m, l;                // reference maximum (log2 domain) and the running sum over all keys of the row
    float lq;                  // this lane's share of the sum over the weights as they entered the value product
};

template <typename F, int... I>
__device__ __forceinline__ void static_for(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>()), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) { static_for(f, std::make_integer_sequence<int, N>()); }

// The loads are written as assembly so that the compiler does not order them against LDS reads: it
// cannot tell the two halves of the double buffer apart and would wait for every outstanding load
// before each read.  dma_wait() before the workgroup barrier is what makes a block visible.
__device__ __forceinline__ void dma16(u32x4_t rsrc, uint32_t lds_addr, uint32_t voff, uint32_t soff) {
    // m0 carries the LDS address of the load.  As an operand of the statement it is written by the compiler, which
    // so knows of it (and often makes the address in it).  The load needs a wait state behind that write.
    asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds"
                 : : "{m0}"(lds_addr), "v"(voff), "s"(rsrc), "s"(soff) : "memory");
}
// Waits until at most n of this wave's loads are outstanding (they complete in order): n = the number
// of loads of the newest block leaves the block before it complete.
__device__ __forceinline__ void dma_wait(int n) {
    switch (n) {           // n is wave-uniform; the instruction takes an immediate
        case 0: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
        case 4: asm volatile("s_waitcnt vmcnt(4)" ::: "memory"); break;
        case 5: asm volatile("s_waitcnt vmcnt(5)" ::: "memory"); break;
        case 9: asm volatile("s_waitcnt vmcnt(9)" ::: "memory"); break;
        case 10: asm volatile("s_waitcnt vmcnt(10)" ::: "memory"); break;
        case 19: asm volatile("s_waitcnt vmcnt(19)" ::: "memory"); break;
        case 38: asm volatile("s_waitcnt vmcnt(38)" ::: "memory"); break;
        default: asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); break;
    }
}

// This wave's share of the loads of one 32-key block into LDS.  A load fills 1024 consecutive LDS
// bytes in lane order.  Load r < 32: the latent part of row r, lane l fetching chunk l.  Load 32 + p:
// the tails of rows 6 p .. 6 p + 5, lane l = 10 i + c fetching chunk 64 + c of row 6 p + i (c < 8;
// lanes with c >= 8, l >= 60 or a row past the block fetch nothing).  Bytes past the sequence's end
// read as zero.  The per-lane parts of the addresses (dma.main_off, dma.tail_off) do not depend on
// the load, the rest is scalar.
struct DmaLane {
    uint32_t main_off, tail_off;
    int tail_row;                // 6 p + tail_row is the lane's row in a tail load; 64 for lanes that fetch nothing
};
__device__ __forceinline__ DmaLane dma_lane(int lane) {
    DmaLane d;
    const int i = lane / 10, c = lane - 10 * i;
    d.main_off = (uint32_t)lane * 16;
    d.tail_off = (uint32_t)(i * kRowB + 1024 + c * 16);
    d.tail_row = (c < 8 && i < kTailRowsPerLoad) ? i : 64;
    return d;
}
// Load q (of this wave's (kDmaPerBlock + NW - 1) / NW) of a block.
template <int NW>
__device__ __forceinline__ void block_load(char* lds_block, u32x4_t rc, int j_block, int wave, const DmaLane& dma, int q) {
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds_block;
    const int g = wave + q * NW;             // wave-uniform
    if (g < kMlaKeys) {
        dma16(rc, lds0 + g * kPitch, dma.main_off, (uint32_t)(j_block + g) * kRowB);
    } else if (g < kDmaPerBlock) {
        const int p = g - kMlaKeys;
        if (p * kTailRowsPerLoad + dma.tail_row < kMlaKeys)
            dma16(rc, lds0 + kTailOff + p * (kTailRowsPerLoad * kTailPitch), dma.tail_off,
                  (uint32_t)(j_block + p * kTailRowsPerLoad) * kRowB);
    }
}
// The same for workgroups of four or eight waves (mla_rows_kernel) with as few scalar instructions as possible: which
// loads fill the tail area is then known from q alone, and the tail loads run with all lanes.  The
// lanes that "fetch nothing" above then fetch bytes that do no harm: chunks 72 and 73 of a row (the
// start of the next row) land in the padding of the tail pitch, lanes 60-63 fetch what the next tail
// load puts in the same place, and rows past the block land behind the tail area, inside the buffer
// (kLdsBlock counts the last load in full).  Bytes past the sequence read as zero.
struct DmaWave {
    uint32_t lds_main, lds_tail;       // LDS address of this wave's first main / tail load
    uint32_t mem_main, mem_tail;       // byte offsets of the same in the sequence's cache
};
__device__ __forceinline__ DmaWave dma_wave_for(char* lds_block, int j_block, int wave) {
    DmaWave d;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)lds_block;
    d.lds_main = lds0 + wave * kPitch;
    d.lds_tail = lds0 + kTailOff + wave * (kTailRowsPerLoad * kTailPitch);
    d.mem_main = (uint32_t)(j_block + wave) * kRowB;
    d.mem_tail = (uint32_t)(j_block + wave * kTailRowsPerLoad) * kRowB;
    return d;
}
template <int NW, int Q>
__device__ __forceinline__ void block_load_static(const DmaWave& d, u32x4_t rc, const DmaLane& dma, int wave) {
    static_assert(NW == 4 || NW == 8, "the main rows must divide among the waves");
    constexpr int kMainLoads = kMlaKeys / NW;        // loads 0 .. kMainLoads - 1 of a wave are rows wave + NW q
    if constexpr (Q < kMainLoads) {
        dma16(rc, d.lds_main + Q * NW * kPitch, dma.main_off, d.mem_main + Q * NW * kRowB);
    } else if constexpr (NW * (Q - kMainLoads + 1) <= kTailLoads) {    // tail loads wave + NW (Q - kMainLoads), all waves
        dma16(rc, d.lds_tail + (Q - kMainLoads) * NW * (kTailRowsPerLoad * kTailPitch), dma.tail_off,
              d.mem_tail + (Q - kMainLoads) * NW * kTailRowsPerLoad * kRowB);
    } else if constexpr (NW * (Q - kMainLoads) < kTailLoads) {         // the last ones: the first waves only
        if (wave + NW * (Q - kMainLoads) < kTailLoads)
            dma16(rc, d.lds_tail + (Q - kMainLoads) * NW * (kTailRowsPerLoad * kTailPitch), dma.tail_off,
                  d.mem_tail + (Q - kMainLoads) * NW * kTailRowsPerLoad * kRowB);
    }
}
template <int NW>
__device__ __forceinline__ void block_to_lds(char* lds_block, u32x4_t rc, int j_block, int wave, const DmaLane& dma) {
    if constexpr (NW == 4 || NW == 8) {
        const DmaWave d = dma_wave_for(lds_block, j_block, wave);
        static_for<(kDmaPerBlock + NW - 1) / NW>([&](auto q_c) { block_load_static<NW, decltype(q_c)::value>(d, rc, dma, wave); });
    } else {
#pragma unroll
        for (int q = 0; q < (kDmaPerBlock + NW - 1) / NW; ++q) block_load<NW>(lds_block, rc, j_block, wave, dma, q);
    }
}

// Two values rounded to fp16 (nearest even) and packed.
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_f16(float a, float b) {
    const f32x2_t v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2_t));
}

// Scheduling groups (the group sizes must be compile-time constants, hence the templates).
template <int N> __device__ __forceinline__ void sched_ds() { __builtin_amdgcn_sched_group_barrier(0x100, N, 0); }
template <int N> __device__ __forceinline__ void sched_mfma() { __builtin_amdgcn_sched_group_barrier(0x008, N, 0); }
constexpr int qk_reads_of(int step) { return 2 + (step >= kQRegSteps ? 1 : 0); }
constexpr int qk_reads_before(int steps) {
    int n = 0;
    for (int i = 0; i < steps; ++i) n += qk_reads_of(i);
    return n;
}
template <int STEP>
struct QkSched {
    static __device__ __forceinline__ void run() {
        sched_mfma<2>();
        if constexpr (STEP + kQAhead < kQSteps) sched_ds<qk_reads_of(STEP + kQAhead)>();
        if constexpr (STEP + 1 < kQSteps) QkSched<STEP + 1>::run();
    }
};

// One 32-key block from LDS against this wave's tile of 16 rows.  kLo: how the softmax weights go into the value
// product (kLoNever, kLoAlways, kLoDynamic).
//   qk_base = block + n * kPitch + kb * 16                     (key row n of a tile, chunk kb)
//   qt_base = block + kTailOff + n * kTailPitch + kb * 16      (the same for the rope part)
//   pv_base = block + (4 kb + n / 4) * kPitch + (n % 4) * 8    (transposing read, see below)
template <int kLo>
__device__ __forceinline__ void mla_block(MlaTile& st, const char* qk_base, const char* qt_base, const char* pv_base,
                                          const bf16x8_t (&qop)[kQRegSteps], const char* q_lds, float scale_log2,
                                          int j_block, int lim, int kb) {
    // S^T tile kt: A = keys 16 kt .. 16 kt + 15 of the block (lane (kb, n): key n, columns 32 step +
    // 8 kb .. + 7), B = Q; the result at lane (kb, n) is key 16 kt + 4 kb + i against row n.
    f32x4_t s[2];
    s[0] = s[1] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    // The key fragments (and, from step kQRegSteps on, the lane's Q chunks, which it parked in LDS at
    // q_lds + (step - kQRegSteps) * 1024) are fetched kQAhead steps before the MFMAs
    // that use them.
    bf16x8_t ka[kQSteps][2], ql[kQSteps - kQRegSteps];
    auto load_step = [&](int step) {
        if (step < kMainSteps) {
            ka[step][0] = *reinterpret_cast<const bf16x8_t*>(qk_base + step * 64);
            ka[step][1] = *reinterpret_cast<const bf16x8_t*>(qk_base + kTileB + step * 64);
        } else {
            ka[step][0] = *reinterpret_cast<const bf16x8_t*>(qt_base + (step - kMainSteps) * 64);
            ka[step][1] = *reinterpret_cast<const bf16x8_t*>(qt_base + kTailTileB + (step - kMainSteps) * 64);
        }
        if (step >= kQRegSteps) ql[step - kQRegSteps] = *reinterpret_cast<const bf16x8_t*>(q_lds + (step - kQRegSteps) * 1024);
    };
#pragma unroll
    for (int step = 0; step < kQAhead; ++step) load_step(step);
#pragma unroll
    for (int step = 0; step < kQSteps; ++step) {
        if (step + kQAhead < kQSteps) load_step(step + kQAhead);
        const bf16x8_t qv = step < kQRegSteps ? qop[step < kQRegSteps ? step : 0] : ql[step < kQRegSteps ? 0 : step - kQRegSteps];
        s[0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[step][0], qv, s[0], 0, 0, 0);
        s[1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[step][1], qv, s[1], 0, 0, 0);
    }
    // Pin that order for the instruction scheduler: the first reads, then MFMAs and reads in turn.
    sched_ds<qk_reads_before(kQAhead)>();
    QkSched<0>::run();
    // O^T tile ct: A = value columns 16 ct .. + 15 (lane (kb, n): column n, keys as in the softmax
    // below), B = P^T.  A transposing read hands lane n of a 16-lane group, from the 64 values that
    // the group's lanes point at taken in lane order, the values n, n + 16, n + 32, n + 48: lanes 4 j ..
    // 4 j + 3 point at 16 consecutive columns of key 4 kb + j, so lane n receives column n of keys
    // 4 kb .. 4 kb + 3.  The first value fragments are fetched here, ahead of the softmax.
    bf16x8_t va[kColTiles];
    auto load_v = [&](int ct) {
        const s16x4v_t v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (__attribute__((address_space(3))) s16x4v_t*)(pv_base + ct * 32));
        const s16x4v_t v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (__attribute__((address_space(3))) s16x4v_t*)(pv_base + kTileB + ct * 32));
        const u32x2_t w0 = __builtin_bit_cast(u32x2_t, v0), w1 = __builtin_bit_cast(u32x2_t, v1);
        return __builtin_bit_cast(bf16x8_t, u32x4_t{w0.x, w0.y, w1.x, w1.y});
    };
#pragma unroll
    for (int ct = 0; ct < 2 * kVAhead; ++ct) va[ct] = load_v(ct);
    // Softmax.  The lane's 8 weights of a row, ordered (kt, i), are the B operand of the value product
    // when contraction index 8 kb + 4 kt + i stands for key 16 kt + 4 kb + i.
    // Keys at or past lim (the end of the segment, or the causal limit of the row) count as
    // -inf; only the blocks that reach that far pay for the comparison.  scale_log2 > 0, so the
    // maximum is taken before scaling, and one fused multiply-add scales and shifts.
    float p[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) p[t] = s[t >> 2][t & 3];
    if (__builtin_amdgcn_ballot_w64(j_block + kMlaKeys > lim) != 0) {
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            const int key = j_block + 16 * (t >> 2) + 4 * kb + (t & 3);
            p[t] = key < lim ? p[t] : kNegInf;
        }
    }
    float mx = fmaxf(fmaxf(fmaxf(p[0], p[1]), fmaxf(p[2], p[3])), fmaxf(fmaxf(p[4], p[5]), fmaxf(p[6], p[7])));
    mx = kb_max(mx) * scale_log2;
    // The reference maximum follows the row's maximum lazily: it moves only when a block exceeds
    // it by more than kLazyLog2, so weights reach 2^kLazyLog2 at most (harmless in fp32 sums and in
    // bf16's relative precision) and the rescaling of the 128 accumulators below, which would
    // otherwise run in most blocks (some row of the tile sees a new maximum), runs about once.
    const float m_new = mx > st.m + kLazyLog2 ? mx : st.m;
    const float m_use = (m_new == kNegInf) ? 0.0f : m_new;
    const float alpha = fast_exp2(st.m - m_use);
    float sum = 0.0f;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        p[t] = fast_exp2(__builtin_fmaf(p[t], scale_log2, -m_use));
        sum += p[t];
    }
    st.l = st.l * alpha + kb_sum(sum);
    st.m = m_new;
    if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
        for (int ct = 0; ct < kColTiles; ++ct) st.o[ct] *= alpha;
    }
    // Dominant key: the block's largest weight of a row against the row's sum so far (this block
    // included), which is at most the sum the output is divided by in the end.  The tile adds the
    // lo parts if any of its rows has one.
    const bool with_lo = kLo == kLoAlways ||
                         (kLo == kLoDynamic && __builtin_amdgcn_ballot_w64(fast_exp2(mx - m_use) * kDominantShare >= st.l) != 0);
    // Where a weight goes in as one bf16 the output is normalised by the sum of the ROUNDED weights:
    // a softmax over slightly perturbed scores (relative weight error 2^-9, the same for equal
    // weights, none for a lone key) instead of rounded weights over an exact sum.
    uint32_t h[4], lo[4] = {0u, 0u, 0u, 0u};
    float sum_q = 0.0f;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const f32x2_t pp = {p[2 * u], p[2 * u + 1]};
        const bf16x2_t hh = __builtin_convertvector(pp, bf16x2_t);
        const f32x2_t back = __builtin_convertvector(hh, f32x2_t);
        h[u] = __builtin_bit_cast(uint32_t, hh);
        sum_q += back[0] + back[1];
        p[2 * u] -= back[0];
        p[2 * u + 1] -= back[1];
    }
    if (with_lo) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const f32x2_t rest = {p[2 * u], p[2 * u + 1]};
            lo[u] = __builtin_bit_cast(uint32_t, __builtin_convertvector(rest, bf16x2_t));
        }
    }
    st.lq = st.lq * alpha + (with_lo ? sum : sum_q);
    const bf16x8_t ph = __builtin_bit_cast(bf16x8_t, u32x4_t{h[0], h[1], h[2], h[3]});
    const bf16x8_t pl = __builtin_bit_cast(bf16x8_t, u32x4_t{lo[0], lo[1], lo[2], lo[3]});
    // Value product, fragments kVAhead tile pairs ahead; per pair the hi parts of both tiles
    // first, then the lo parts, so that no MFMA waits for the one just before it.
#pragma unroll
    for (int c2 = 0; c2 < kColTiles; c2 += 2) {
        if (c2 + 2 * kVAhead < kColTiles) {
            va[c2 + 2 * kVAhead] = load_v(c2 + 2 * kVAhead);
            va[c2 + 2 * kVAhead + 1] = load_v(c2 + 2 * kVAhead + 1);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) st.o[c2 + u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[c2 + u], ph, st.o[c2 + u], 0, 0, 0);
        if (kLo == kLoAlways) {
#pragma unroll
            for (int u = 0; u < 2; ++u) st.o[c2 + u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[c2 + u], pl, st.o[c2 + u], 0, 0, 0);
        }
    }
#pragma unroll
    for (int c2 = 0; c2 < kColTiles; c2 += 2) {
        __builtin_amdgcn_sched_group_barrier(0x008, 2 * (kLo == kLoAlways ? 2 : 1), 0);
        if (c2 + 2 * kVAhead < kColTiles) __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
    }
    if (kLo == kLoDynamic && with_lo) {
        // The rare block with a dominant key: a second pass over the value fragments with the lo parts.
#pragma unroll
        for (int ct = 0; ct < kColTiles; ++ct)          // fully unrolled: the accumulators are registers
            st.o[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(load_v(ct), pl, st.o[ct], 0, 0, 0);
    }
}

// kMode: 0 = default (hi + lo weights in the first mla_exact_blocks() blocks of a segment and wherever a key
// dominates its row), 1 = hi + lo weights everywhere, 2 = one bf16 per weight everywhere.
template <int NW, int kMode>
__global__ __launch_bounds__(64 * NW) void mla_decode_kernel(
        const int32_t* __restrict__ kv_lens, const void* const* c_ptrs, int batch, int n_pieces, int min_piece,
        int few_pieces, int few_min, int xcd_skew, int q_len, int n_heads, MlaParams prm) {
    __shared__ __attribute__((aligned(16))) char lds_c[kStages * kLdsBlock];
    // Per wave: the Q chunks of steps kQRegSteps.. (each lane reads back what it wrote).
    __shared__ __attribute__((aligned(16))) char lds_q[NW * kQLdsWave];
    static_assert(NW * kStageWave <= kStages * kLdsBlock, "output staging must fit the block buffers");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kb = lane >> 4, n = lane & 15;
    const int T = q_len, H = n_heads, rows_total = T * H;
    SeqWindow win;
    const WavePlan wp = wave_plan(kv_lens, c_ptrs, nullptr, batch, n_pieces, min_piece, kMlaSegCost,
                                  xcd_skew, FewPieces{few_pieces, few_min}, lane, &win);
    const Plan& pl = wp.pl;
    const int per_xcd = (pl.n_pieces + 7) >> 3;
    // Workgroup ids go round-robin over the 8 XCDs.  Of an XCD's workgroups, consecutive ones are the
    // row groups of one piece: they run at the same time on the same XCD and share its L2, so the
    // piece's cache rows come from HBM once.
    const int bid = blockIdx.x;
    const int n_groups = (rows_total + 16 * NW - 1) / (16 * NW);
    const int slot_in_xcd = bid >> 3;
    const int row_group = slot_in_xcd % n_groups;
    const int p = (bid & 7) * per_xcd + slot_in_xcd / n_groups;
    const int s0 = piece_bound(pl, p), s1 = piece_bound(pl, p + 1);
    const bool active = slot_in_xcd / n_groups < per_xcd && p < pl.n_pieces && s0 < s1;

    if (tid < 64) {
        // For the merge kernel: first partial slot and number of segments of every sequence, 64
        // sequences per wave, the groups of 64 dealt out over the workgroups.
        for (int g = bid; 64 * g < batch; g += gridDim.x) wave_write_meta(wp, kv_lens, batch, rows_total, g, lane, prm.meta);
    }
    if (!active) return;       // the whole workgroup: every wave computed the same plan

    Walk walk;
    wave_locate(wp, kv_lens, c_ptrs, nullptr, batch, s0, lane, &win, walk.b, walk.j);
    walk.remaining = uniform(s1 - s0);

    // Lane n's row: index within the sequence's T * H rows.
    const int wave_row0 = (row_group * NW + wave) * 16, row = wave_row0 + n;
    char* q_lds = lds_q + wave * kQLdsWave + lane * 16;
    char* stage = lds_c + wave * kStageWave;
    const int exact_blocks = mla_exact_blocks(pl, rows_total, n_pieces);
    const DmaLane dma = dma_lane(lane);
    const int my_loads = (kDmaPerBlock - wave + NW - 1) / NW;      // block loads this wave issues per block
    const int qk_off = n * kPitch + kb * 16;
    const int qt_off = kTailOff + n * kTailPitch + kb * 16;
    const int pv_off = (4 * kb + (n >> 2)) * kPitch + (n & 3) * 8;
    auto fence = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };

    PieceSeg ps;
    while (uniform(next_segment(walk, batch, pl.seg_cost,
                                [&](int bb) { return window_len(win, kv_lens, bb); }, ps))) {
        const int b = uniform(ps.b), L = uniform(ps.L), j0 = uniform(ps.j0), j1 = uniform(ps.j1);
        const bool whole = uniform(ps.whole) != 0;
        const long slot = (long)uniform(p) + b;
        const unsigned long long cbytes = (unsigned long long)L * kRowB;
        const uint64_t caddr = (uint64_t)(uintptr_t)window_ptr(win, win.k, c_ptrs, b);
        // raw buffer descriptor: base, no stride, bytes, 32-bit raw format
        const u32x4_t rc = {(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)caddr),
                            (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(caddr >> 32) & 0xffffu)),
                            cbytes > 0xffffffffull ? 0xffffffffu : (uint32_t)cbytes, 0x00020000u};

        // Q operand: lane (kb, n) holds columns 32 step + 8 kb .. + 7 of row n; rows past the last
        // lie past the end of the descriptor and read as zero.
        const __amdgpu_buffer_rsrc_t rq = make_rsrc(prm.q + (long)b * rows_total * kDqk, (uint32_t)rows_total * kRowB);
        bf16x8_t qop[kQRegSteps];
        MlaTile st;
#pragma unroll
        for (int step = 0; step < kQSteps; ++step) {
            const u32x4_t qv = __builtin_amdgcn_raw_buffer_load_b128(rq, row * kRowB + kb * 16 + 64 * step, 0, 0);
            if (step < kQRegSteps) qop[step < kQRegSteps ? step : 0] = __builtin_bit_cast(bf16x8_t, qv);
            else *reinterpret_cast<u32x4_t*>(q_lds + (step - kQRegSteps) * 1024) = qv;
        }
        const int causal = L - T + (row < rows_total ? row : 0) / H + 1;
        const int lim = causal < j1 ? causal : j1;
#pragma unroll
        for (int ct = 0; ct < kColTiles; ++ct) st.o[ct] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
        st.m = kNegInf;
        st.l = 0.0f;
        st.lq = 0.0f;

        // Block 0 -> buffer 0, behind the Q loads: those do not need the sequence's base address, whose
        // own load they now cover.
        block_to_lds<NW>(lds_c, rc, j0, wave, dma);
        // Q is used here, before the loop, so that the wait for its loads sits here as well: a wait
        // inside the loop would also wait for the block loads that were just issued.
#pragma unroll
        for (int step = 0; step < kQRegSteps; ++step) asm volatile("" : "+v"(qop[step]));
        fence();                  // the Q chunks in LDS are read back by the lane that wrote them

        const int n_blocks = (j1 - j0 + kMlaKeys - 1) / kMlaKeys;
        if (n_blocks > 1) block_to_lds<NW>(lds_c + kLdsBlock, rc, j0 + kMlaKeys, wave, dma);   // block 1 -> buffer 1
        int cur_buf = 0, next_buf = 2;         // block blk sits in buffer blk % 3, block blk + 2 goes to next_buf
        // One block: every wave waits for its own loads of block blk (those of block blk + 1 may stay
        // in flight), then the barrier: block blk is in LDS and everyone is done reading block
        // blk - 1, whose buffer the loads of block blk + 2 may overwrite.
        auto step = [&](int blk, auto lo_mode) {
            const char* cur = lds_c + cur_buf * kLdsBlock;
            dma_wait(blk + 1 < n_blocks ? my_loads : 0);
            __syncthreads();
            if (blk + 2 < n_blocks) block_to_lds<NW>(lds_c + next_buf * kLdsBlock, rc, j0 + (blk + 2) * kMlaKeys, wave, dma);
            mla_block<decltype(lo_mode)::value>(st, cur + qk_off, cur + qt_off, cur + pv_off, qop, q_lds, prm.scale_log2,
                                                j0 + blk * kMlaKeys, lim, kb);
            cur_buf = cur_buf == kStages - 1 ? 0 : cur_buf + 1;
            next_buf = next_buf == kStages - 1 ? 0 : next_buf + 1;
        };
        // Default mode: the first blocks of a segment with hi + lo weights, the others with hi + lo
        // only where a key dominates.
        const int n_exact = kMode == 1 ? n_blocks : kMode == 2 ? 0 : (n_blocks < exact_blocks ? n_blocks : exact_blocks);
        int blk = 0;
        for (; blk < n_exact; ++blk) step(blk, std::integral_constant<int, kLoAlways>());
        for (; blk < n_blocks; ++blk)
            step(blk, std::integral_constant<int, kMode == 0 ? kLoDynamic : (kMode == 1 ? kLoAlways : kLoNever)>());
        __syncthreads();          // everyone is done with the block buffers: they stage the output now

        const float l = st.l;
        const float lq = kb_sum(st.lq);
        // A partial row goes out as fp16 after scaling its largest magnitude to 2^15 (the scale's
        // inverse is kept in fp32 beside the row's m and l): half the bytes of fp32 to write here
        // and to read back in the merge.  Every element keeps 11 significant bits of its own
        // (down to 2^-29 of the row's maximum), so a few large columns cost the others nothing.
        // The scale is capped so that rows of denormal size do not overflow it.
        float sc, inv_scale = 0.0f;
        if (whole) {
            sc = lq > 0.0f ? 1.0f / lq : 0.0f;
        } else {
            float amax = 0.0f;
#pragma unroll
            for (int ct = 0; ct < kColTiles; ++ct)
#pragma unroll
                for (int i = 0; i < 4; ++i) amax = fmaxf(amax, __builtin_fabsf(st.o[ct][i]));
            amax = kb_max(amax);
            sc = amax > 0.0f ? fminf(32768.0f / amax, 0x1.0p100f) : 0.0f;
            inv_scale = amax > 0.0f ? 1.0f / sc : 0.0f;
        }
        // Rounded to 16 bits (bf16 results, fp16 partial rows), half a row at a time through the
        // block buffers, which are free between the segment's last block and the next segment's
        // first: two rounds, each store instruction writing two whole 512-byte half rows.
        // The stores go through a buffer descriptor over the sequence's (or slot's) rows: 32-bit
        // offsets, and rows past rows_total fall outside and are dropped, so the loop has no branch.
        uint16_t* dst = whole ? prm.out + (long)b * rows_total * kDv : prm.part_o + slot * rows_total * kDv;
        const __amdgpu_buffer_rsrc_t rd = make_rsrc(uniform(static_cast<void*>(dst)), (uint32_t)rows_total * (kDv * 2));
        const uint32_t lane_dst = (uint32_t)((wave_row0 + (lane >> 5)) * (kDv * 2) + (lane & 31) * 16);
        const char* lane_stage = stage + (lane >> 5) * kStagePitch + (lane & 31) * 16;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int c = 0; c < kColTiles / 2; ++c) {
                const f32x4_t o = st.o[(kColTiles / 2) * h + c] * sc;
                uint2 w;
                w.x = whole ? cvt_bf16(o[0], o[1]) : pack_f16(o[0], o[1]);
                w.y = whole ? cvt_bf16(o[2], o[3]) : pack_f16(o[2], o[3]);
                *reinterpret_cast<uint2*>(stage + n * kStagePitch + (16 * c + 4 * kb) * 2) = w;
            }
            fence();
#pragma unroll
            for (int i = 0; i < 8; ++i) {          // rows 2 i and 2 i + 1, 256 columns each, per instruction
                const u32x4_t w = *reinterpret_cast<const u32x4_t*>(lane_stage + 2 * i * kStagePitch);
                __builtin_amdgcn_raw_buffer_store_b128(w, rd, (int)(lane_dst + 2 * i * (kDv * 2) + h * kDv), 0, 0);
            }
            fence();
        }
        if (row < rows_total && kb == 0) {
            if (whole) {
                if (prm.lse) prm.lse[(long)b * rows_total + row] = l > 0.0f ? (st.m + __log2f(l)) * kLn2 : kNegInf;
            } else {
                reinterpret_cast<float4*>(prm.part_ml)[slot * rows_total + row] = make_float4(st.m, l, lq, inv_scale);
            }
        }
        __syncthreads();          // the next segment's first block goes to buffer 0, which staged output until here
    }
}

// ----------------------------------------------------------------------- tiles of 32 query rows
// More than 32 query rows: a wave owns 32 rows, one wave per SIMD with 512 registers: the 32 x 512 fp32 output
// accumulators in the 256 accumulation registers, Q (33 of its 36 MFMA steps) and two blocks' scores in the
// ordinary ones.  With 32x32x16 MFMAs an operand fragment read from LDS (1 KiB) feeds 32 cycles of the matrix
// pipe; with 16x16x32 it is 16, as fast as the LDS delivers fragments, and a loop with a wave per 16 rows (eight of
// them) was bound by both in turn, 4600 cycles per block against 3100 here.
// A block's 32 keys run through two phases, the work of two blocks interleaved so that the matrix pipe has
// work while the vector unit does the softmax:
//   A: scores of block i + 1 (36 MFMAs), and between them the weights of block i from its scores;
//   B: values of block i (32 MFMAs), and between them the maximum of block i + 1's scores.
// What bounds it: a lone wave issues an instruction every four cycles or so, and the 68 MFMAs (2176 cycles) leave room for
// most of the others but not all: against MFMAs alone the loads into LDS cost 290 cycles of a block, the softmax 300, the
// operand reads 120.  And power: on random data the clock falls from 2.4 to 1.8 GHz (all-zero data: 256 rows 130 us
// instead of 164).  Whole calls, eight waves of 16 rows -> here, 64 sequences of 1024 to 8192 tokens: 128 rows
// 109.4 -> 100.3 us, 256 rows 184.4 -> 168.4, 72 rows 100.1 -> 84.3, 33 rows 77.7 -> 69.3 (four waves of 16 before); short
// ones (see mla_tile_split): 40 of 64 to 256, 128 rows 27.7 -> 24.5; 64 of 64 to 256, 256 rows level at 37.1.
// Tried without gain: operands 3, 5 or 6 fragments ahead; one wait for two fragments (2 % slower); a block's last
// MFMAs behind the next barrier; its first weights ahead of its first MFMA (1 % slower).
// Four LDS buffers: block i (values), i + 1 (scores), i + 2 and i + 3 on their way; one barrier per block.
// A block's image in LDS: row r's latent part at r * kPitch, 16 bytes further from row 16 on, and the rope parts
// as 128-byte rows whose 16-byte chunks are permuted by row (through the global address each lane fetches).
// Key row x of the score MFMA is row tile_key(x) of the block.  With that, the lanes that one pass of an
// LDS read serves (0-3, 12-15, 20-27 and so on for 128 bits; 0-31 for the transposing read) hit different banks; what
// conflicts remain take 3 to 4 % of the LDS-active cycles.
// The MFMAs are assembly statements: their accumulators can then be named (scores in ordinary registers, outputs
// in accumulation registers; through the builtin the compiler puts every MFMA result into the accumulation
// registers, which the outputs fill alone), and such statements keep their order among themselves and against
// memory operations, so LDS reads stay where they are written, a fixed number of MFMAs ahead of their use.  Vector
// instructions do move across them; the softmax is therefore cut into slices of a few instructions whose results
// pass through an empty statement of the same kind (pin): a slice cannot start before the pin its inputs came
// through nor end after its own.
// What the compiler cannot see of an MFMA inside a statement: a vector instruction may read a result register only
// once the MFMA has left the pipe (12 wait states), and an MFMA may read a register two instructions after a vector
// instruction wrote it (mfma_operands).  The compiler may copy scores from the end of the statement that made them on,
// not only where the source reads them, so the statement with a block's last score MFMA ends behind the wait
// (mfma_last_v) or behind two value MFMAs (mfma_last_acc).
constexpr int kTileSteps = kDqk / 16;            // 36 MFMA steps of 16 columns
constexpr int kTileQRegs = 33;                   // Q steps in registers, the rest parked in LDS
constexpr int kTileQLds = (kTileSteps - kTileQRegs) * 1024;      // per wave
constexpr int kTileCols = kDv / 32;              // 16 tiles of 32 value columns
constexpr int kTileStages = 4;
constexpr int kTileHalf = 16 * kPitch + 16;      // rows 16..31
constexpr int kTileTailOff = kTileHalf + 15 * kPitch + 1024;
constexpr int kTileBlock = kTileTailOff + kMlaKeys * 128;
constexpr int kTileLoads = kMlaKeys / kTileWaves + 1;            // loads per wave and block: 8 rows, and 8 rows' rope parts
constexpr int kTileKAhead = 4, kTileVAhead = 4;  // fragments in flight ahead of their MFMAs
constexpr int kTileStagePitch = kDv * 2 + 16;    // epilogue: whole rows, padded

typedef __attribute__((ext_vector_type(16))) float f32x16_t;

__device__ __forceinline__ void mfma_first_v(f32x16_t& acc, bf16x8_t a, bf16x8_t b) {      // acc = a b
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(acc) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_v(f32x16_t& acc, bf16x8_t a, bf16x8_t b) {            // acc += a b
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(acc) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_last_v(f32x16_t& acc, bf16x8_t a, bf16x8_t b) {       // acc += a b, done
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0\n\ts_nop 15\n\ts_nop 7" : "+v"(acc) : "v"(a), "v"(b));
}

// The output accumulators: column tile ct is a[16 ct : 16 ct + 15] wherever it is used, all 256 accumulation
// registers together.  Every access is a statement that names those registers: left to choose, the compiler moves
// tiles through ordinary registers, where it cannot know when an MFMA inside a statement has written its result.
struct TileAcc {
    f32x16_t t[kTileCols];
};
#define XATTN_ACC_EACH(X) X(0) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15)
#define XATTN_ACC_REG(ct, i) "a[16*" #ct "+" #i "]"
#define XATTN_ACC_TILE(ct) XATTN_ACC_TILE_##ct
#define XATTN_ACC_TILE_0 "{a[0:15]}"
#define XATTN_ACC_TILE_1 "{a[16:31]}"
#define XATTN_ACC_TILE_2 "{a[32:47]}"
#define XATTN_ACC_TILE_3 "{a[48:63]}"
#define XATTN_ACC_TILE_4 "{a[64:79]}"
#define XATTN_ACC_TILE_5 "{a[80:95]}"
#define XATTN_ACC_TILE_6 "{a[96:111]}"
#define XATTN_ACC_TILE_7 "{a[112:127]}"
#define XATTN_ACC_TILE_8 "{a[128:143]}"
#define XATTN_ACC_TILE_9 "{a[144:159]}"
#define XATTN_ACC_TILE_10 "{a[160:175]}"
#define XATTN_ACC_TILE_11 "{a[176:191]}"
#define XATTN_ACC_TILE_12 "{a[192:207]}"
#define XATTN_ACC_TILE_13 "{a[208:223]}"
#define XATTN_ACC_TILE_14 "{a[224:239]}"
#define XATTN_ACC_TILE_15 "{a[240:255]}"
template <int kCt>
__device__ __forceinline__ void acc_mfma(TileAcc& o, bf16x8_t a, bf16x8_t b) {            // tile kCt += a b
#define X(ct) if constexpr (kCt == ct) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+" XATTN_ACC_TILE(ct)(o.t[ct]) : "v"(a), "v"(b));
    XATTN_ACC_EACH(X)
#undef X
}
// s += a b, done; then tile 0 += a0 b0 + a1 b1, whose first MFMA waits for the one of s and takes 8 passes itself.
__device__ __forceinline__ void mfma_last_acc(f32x16_t& s, bf16x8_t a, bf16x8_t b, TileAcc& o, bf16x8_t a0, bf16x8_t b0, bf16x8_t a1, bf16x8_t b1) {
    asm volatile("v_mfma_f32_32x32x16_bf16 %0, %2, %3, %0\n\t"
                 "v_mfma_f32_32x32x16_bf16 %1, %4, %5, %1\n\t"
                 "v_mfma_f32_32x32x16_bf16 %1, %6, %7, %1"
                 : "+v"(s), "+" XATTN_ACC_TILE(0)(o.t[0]) : "v"(a), "v"(b), "v"(a0), "v"(b0), "v"(a1), "v"(b1));
}
// The first kN tiles.
template <int kN>
__device__ __forceinline__ void acc_zero(TileAcc& o) {
#define Z(ct, i) "v_accvgpr_write_b32 " XATTN_ACC_REG(ct, i) ", 0\n\t"
#define X(ct)                                                                                                              \
    if constexpr (ct < kN)                                                                                                 \
    asm volatile(Z(ct, 0) Z(ct, 1) Z(ct, 2) Z(ct, 3) Z(ct, 4) Z(ct, 5) Z(ct, 6) Z(ct, 7) Z(ct, 8) Z(ct, 9) Z(ct, 10)        \
                 Z(ct, 11) Z(ct, 12) Z(ct, 13) Z(ct, 14) Z(ct, 15) : "=" XATTN_ACC_TILE(ct)(o.t[ct]));
    XATTN_ACC_EACH(X)
#undef X
#undef Z
}
// Before the first vector instruction that reads the accumulators; all but the last two tiles were written long ago.
template <int kN>
__device__ __forceinline__ void acc_drain(TileAcc& o) {
    if constexpr (kN == 16) asm volatile("s_nop 15\n\ts_nop 7" : "+" XATTN_ACC_TILE(14)(o.t[14]), "+" XATTN_ACC_TILE(15)(o.t[15]));
    else asm volatile("s_nop 15\n\ts_nop 7" : "+" XATTN_ACC_TILE(6)(o.t[6]), "+" XATTN_ACC_TILE(7)(o.t[7]));
    static_assert(kN == 16 || kN == 8, "the last two tiles");
}
template <int kN>
__device__ __forceinline__ void acc_scale(TileAcc& o, float f) {                           // behind acc_drain
    float t0, t1, t2, t3;
#define R(ct, i, t) "v_accvgpr_read_b32 %" #t ", " XATTN_ACC_REG(ct, i) "\n\t"
#define M(t) "v_mul_f32 %" #t ", %" #t ", %5\n\t"
#define W(ct, i, t) "v_accvgpr_write_b32 " XATTN_ACC_REG(ct, i) ", %" #t "\n\t"
#define Q(ct, a, b, c, d) R(ct, a, 1) R(ct, b, 2) R(ct, c, 3) R(ct, d, 4) M(1) M(2) M(3) M(4) W(ct, a, 1) W(ct, b, 2) W(ct, c, 3) W(ct, d, 4)
#define X(ct)                                                                                          \
    if constexpr (ct < kN)                                                                             \
    asm volatile(Q(ct, 0, 1, 2, 3) Q(ct, 4, 5, 6, 7) Q(ct, 8, 9, 10, 11) Q(ct, 12, 13, 14, 15)         \
                 : "+" XATTN_ACC_TILE(ct)(o.t[ct]), "=&v"(t0), "=&v"(t1), "=&v"(t2), "=&v"(t3) : "v"(f));
    XATTN_ACC_EACH(X)
#undef X
#undef Q
#undef W
#undef M
#undef R
}
template <int kCt>
__device__ __forceinline__ void acc_read(const TileAcc& o, float (&v)[16]) {              // behind acc_drain
#define R(ct, i) "v_accvgpr_read_b32 %" #i ", " XATTN_ACC_REG(ct, i) "\n\t"
#define X(ct)                                                                                                              \
    if constexpr (kCt == ct)                                                                                               \
        asm volatile(R(ct, 0) R(ct, 1) R(ct, 2) R(ct, 3) R(ct, 4) R(ct, 5) R(ct, 6) R(ct, 7) R(ct, 8) R(ct, 9) R(ct, 10)   \
                     R(ct, 11) R(ct, 12) R(ct, 13) R(ct, 14) R(ct, 15)                                                     \
                     : "=v"(v[0]), "=v"(v[1]), "=v"(v[2]), "=v"(v[3]), "=v"(v[4]), "=v"(v[5]), "=v"(v[6]), "=v"(v[7]),     \
                       "=v"(v[8]), "=v"(v[9]), "=v"(v[10]), "=v"(v[11]), "=v"(v[12]), "=v"(v[13]), "=v"(v[14]), "=v"(v[15]) \
                     : XATTN_ACC_TILE(ct)(o.t[ct]));
    XATTN_ACC_EACH(X)
#undef X
#undef R
}
#undef XATTN_ACC_EACH
__device__ __forceinline__ void mfma_operands(bf16x8_t& a, bf16x8_t& b) { asm volatile("s_nop 1" : "+v"(a), "+v"(b)); }
template <typename A> __device__ __forceinline__ void pin(A& a) { asm volatile("" : "+v"(a)); }
template <typename A, typename B> __device__ __forceinline__ void pin(A& a, B& b) { asm volatile("" : "+v"(a), "+v"(b)); }
// max(a, b) of two scores (finite or -inf, no NaNs) as one instruction, the median of (a, b, largest
// finite float): fmaxf() first quiets each operand it cannot prove to be the result of arithmetic
// (matrix results, swapped lanes), an instruction apiece.
__device__ __forceinline__ float max_num(float a, float b) { return __builtin_amdgcn_fmed3f(a, b, 0x1.fffffep+127f); }
__device__ __forceinline__ float max3(float a, float b, float c) {
    float d;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}
__device__ __forceinline__ void max3_abs(float& m, float a, float b) {      // m = max(m, |a|, |b|)
    asm("v_max3_f32 %0, %0, |%1|, |%2|" : "+v"(m) : "v"(a), "v"(b));
}
template <int N>
__device__ __forceinline__ void dma_wait_for() { asm volatile("s_waitcnt vmcnt(%0)" : : "n"(N) : "memory"); }
// The same for all of them, in a form that the compiler reads: a load of its own that it still counts as outstanding
// would otherwise make it wait inside the block loop, and there for the blocks on their way as well.
__device__ __forceinline__ void dma_wait_all() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0f70);      // vmcnt(0)
    asm volatile("" ::: "memory");
}

// Row of the block that is key x of the score MFMAs; x = 8 g + 4 h + j gives 8 g + 2 j + h, so lane half h holds,
// as accumulator 4 g + j, key 8 g + 2 j + h.
__device__ __forceinline__ int tile_key(int x) { return (x & 24) + 2 * (x & 3) + ((x >> 2) & 1); }
// Chunk of a rope part as stored: chunk c of row r sits at c ^ tile_tail_swap(r).
__device__ __forceinline__ int tile_tail_swap(int row) { return ((row >> 1) & 3) | ((row >> 4) << 2); }

// This wave's loads of a block: rows wave + 4 q (q < 8), and the rope parts of rows 8 wave .. 8 wave + 7.  Rows past the
// end of the descriptor read as zero.
struct TileDma {
    uint32_t row_off, tail_off;      // per lane
};
__device__ __forceinline__ TileDma tile_dma(int wave, int lane) {
    const int i = lane >> 3;
    return TileDma{(uint32_t)lane * 16, (uint32_t)(i * kRowB + 1024 + ((lane & 7) ^ tile_tail_swap(8 * wave + i)) * 16)};
}
struct TileLoad {                    // a block's loads by this wave
    u32x4_t rc;
    uint32_t lds, mem;               // the wave's first row
    uint32_t lds_tail, mem_tail;
};
__device__ __forceinline__ TileLoad tile_load_for(const char* lds_block, u32x4_t rc, int j_block, int wave) {
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)lds_block;
    return TileLoad{rc, lds0 + (uint32_t)wave * kPitch, (uint32_t)(j_block + wave) * kRowB, lds0 + kTileTailOff + (uint32_t)wave * 1024,
                    (uint32_t)(j_block + 8 * wave) * kRowB};
}
template <int Q>
__device__ __forceinline__ void tile_load(const TileLoad& b, const TileDma& d) {
    if constexpr (Q < kTileLoads - 1)
        dma16(b.rc, b.lds + Q * kTileWaves * kPitch + (Q >= 4 ? 16 : 0), d.row_off, b.mem + Q * kTileWaves * kRowB);
    else
        dma16(b.rc, b.lds_tail, d.tail_off, b.mem_tail);
}

// A wave's Q on its way to the registers: whole rows by loads into LDS (a lane's own chunks straight from memory are 64
// separate lines per load: 5.7 us of a segment's start), in two rounds of half of the latent and half of the rope part,
// with chunks permuted by row so that the reads below meet different banks.  `first`: the workgroups of a sequence begin at
// different rows, or all of them ask for the same lines at the same time.
constexpr int kTileQStage = kTileRows * (512 + 64);
__device__ __forceinline__ void tile_q_load(char* stage, u32x4_t rq, int wave_row0, int lane, int round, int first) {
    uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)stage;
    asm volatile("" : "+s"(lds0), "+s"(wave_row0), "+s"(first));
    const int up = lane >> 5, c0 = (lane & 31) ^ up;
#pragma unroll
    for (int k = 0; k < kTileRows / 2; ++k) {
        const int i = (k + first) & (kTileRows / 2 - 1);         // rows 2 i and 2 i + 1
        dma16(rq, lds0 + i * 1024, (uint32_t)(up * kRowB + (c0 ^ (2 * i & 15)) * 16), (uint32_t)(wave_row0 + 2 * i) * kRowB + round * 512);
    }
#pragma unroll
    for (int i = 0; i < kTileRows / 16; ++i)     // half of the rope parts of rows 16 i .. 16 i + 15
        dma16(rq, lds0 + kTileRows * 512 + i * 1024, (uint32_t)((lane >> 2) * kRowB + 1024 + (((lane & 3) ^ (lane >> 4)) * 16)),
              (uint32_t)(wave_row0 + 16 * i) * kRowB + round * 64);
}
// Steps 16 round .. + 15 (latent part) and 32 + 2 round, + 1 (rope part) of the round in the stage.
__device__ __forceinline__ bf16x8_t tile_q_frag(const char* stage, int lane, int step) {
    const int n = lane & 31, h = lane >> 5;
    const char* p = step < 32 ? stage + n * 512 + ((2 * (step & 15) + h) ^ (n & 15)) * 16
                              : stage + kTileRows * 512 + n * 64 + ((2 * (step & 1) + h) ^ ((n >> 2) & 3)) * 16;
    return *reinterpret_cast<const bf16x8_t*>(p);
}

// What a lane keeps of its row (both halves of the wave hold the same rows).
struct TileRow {
    float m, l;          // reference maximum (log2 domain) and the running sum over the row's keys
    float lq;            // this lane's share of the sum over the weights as they entered the value product
    float mx;            // scaled maximum of the block whose weights come next
};
// Where a lane reads a block's operands: keys at k + 32 * step (steps 0..31) and, for the rope part, t ^ 32 * step, at tail.
struct TileReads {
    int key, tail, tail_chunk;       // offsets within a block; tail_chunk: byte offset within the 128-byte row
    int value;
};
__device__ __forceinline__ TileReads tile_reads(int lane) {
    const int h = lane >> 5, row = tile_key(lane & 31), m = lane & 15;
    TileReads r;
    r.key = row * kPitch + (row >= 16 ? 16 : 0) + h * 16;
    r.tail = kTileTailOff + row * 128;
    r.tail_chunk = (h ^ tile_tail_swap(row)) * 16;
    // value fragment (ct, s), read u: lanes of a 16-lane group point at 16 columns of keys 16 s + 8 u + 2 q + h, q = 0..3
    r.value = (2 * (m >> 2) + h) * kPitch + ((lane >> 4) & 1) * 32 + (m & 3) * 8;
    return r;
}
__device__ __forceinline__ bf16x8_t tile_key_frag(const char* block, const TileReads& rd, int step) {
    const char* p = step < 32 ? block + rd.key + step * 32 : block + rd.tail + (rd.tail_chunk ^ ((step - 32) * 32));
    return *reinterpret_cast<const bf16x8_t*>(p);
}
// Value fragment f = 2 * column tile + half of the keys: the transposing read gives lane n of a 16-lane group the n-th
// column of its group's four keys.
__device__ __forceinline__ bf16x8_t tile_value_frag(const char* block, const TileReads& rd, int f) {
    const char* p = block + rd.value + (f >> 1) * 64 + (f & 1) * kTileHalf;
    const s16x4v_t v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4v_t*)p);
    const s16x4v_t v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4v_t*)(p + 8 * kPitch));
    const u32x2_t w0 = __builtin_bit_cast(u32x2_t, v0), w1 = __builtin_bit_cast(u32x2_t, v1);
    return __builtin_bit_cast(bf16x8_t, u32x4_t{w0.x, w0.y, w1.x, w1.y});
}
// Keys at or past lim (the end of the segment, or the causal limit of the row) count as -inf.
__device__ __forceinline__ void tile_mask(f32x16_t& s, int j_block, int lim, int h) {
#pragma unroll
    for (int t = 0; t < 16; ++t) s[t] = j_block + 8 * (t >> 2) + 2 * (t & 3) + h < lim ? s[t] : kNegInf;
}
__device__ __forceinline__ float tile_max(float t) {
    float a, b;
    swap32(t, a, b);
    return fmaxf(a, b);
}

// Block i: its scores s become weights while the scores s_next of the block at `next` are computed (not in a
// segment's last block), then its values at `cur` are added to o.  issue(q): the caller's load q of a later block.
template <int kLo, bool kLast, int kN, typename Issue>
__device__ __forceinline__ void tile_block(TileAcc& o, TileRow& st, const f32x16_t& s, f32x16_t& s_next,
                                           const bf16x8_t (&qop)[kTileQRegs], const char* q_lds, const TileReads& rd,
                                           const char* cur, const char* next, float scale_log2, int j_next, int lim, int h,
                                           bool exact, Issue issue) {
    constexpr int kTileFrags = 2 * kN;               // value fragments (16 keys x 32 columns) of the wave's columns
    // A load every so many MFMAs, this many of them in phase A.
    constexpr int kTileLoadEvery = kN == 16 ? 7 : 5, kTileLoadsA = (kTileSteps + kTileLoadEvery - 4) / kTileLoadEvery;
    static_assert(kTileLoadsA + (kTileFrags + kTileLoadEvery - 4) / kTileLoadEvery >= kTileLoads, "a slot for every load");
    bf16x8_t ka[kTileSteps], ql[kTileSteps - kTileQRegs], va[kTileFrags];
    auto load_k = [&](auto f_c) {
        constexpr int F = decltype(f_c)::value;
        ka[F] = tile_key_frag(next, rd, F);
        if constexpr (F >= kTileQRegs) ql[F - kTileQRegs] = *reinterpret_cast<const bf16x8_t*>(q_lds + (F - kTileQRegs) * 1024);
    };
    if constexpr (!kLast) static_for<kTileKAhead>(load_k);
    // The reference maximum follows the row's maximum lazily, see mla_block.
    const bool moves = st.mx > st.m + kLazyLog2;
    if (__builtin_amdgcn_ballot_w64(moves) != 0) {
        const float m_new = moves ? st.mx : st.m;
        const float alpha = moves ? fast_exp2(st.m - m_new) : 1.0f;
        const bool first = __builtin_amdgcn_ballot_w64(moves && st.m != kNegInf) == 0;      // all sums are still 0
        st.m = m_new;
        st.l *= alpha;
        st.lq *= alpha;
        if (!first) {
            acc_drain<kN>(o);
            acc_scale<kN>(o, alpha);
        }
    }
    const float m_use = st.m == kNegInf ? 0.0f : st.m;
    // Phase A.
    float p[16], t4[4], sum = 0.0f, sum_q = 0.0f, dom = 0.0f;
    uint32_t hi[8], lo[8];
    auto weights = [&](auto f_c) {
        constexpr int F = decltype(f_c)::value;
        if constexpr (F < 16) {
            p[F] = fast_exp2(__builtin_fmaf(s[F], scale_log2, -m_use));
            pin(p[F]);
        } else if constexpr (F < 20) {
            constexpr int k = 4 * (F - 16);
            t4[F - 16] = (p[k] + p[k + 1]) + (p[k + 2] + p[k + 3]);
            pin(t4[F - 16]);
        } else if constexpr (F == 20) {
            sum = (t4[0] + t4[1]) + (t4[2] + t4[3]);
            pin(sum);
        } else if constexpr (F == 21) {
            float a, b;
            swap32(sum, a, b);
            st.l += a + b;
            pin(st.l);
        } else if constexpr (F == 22) {      // a key with at least 1 / kDominantShare of the row's sum so far
            if (kLo == kLoDynamic) {
                dom = fast_exp2(st.mx - m_use) * kDominantShare >= st.l ? 1.0f : 0.0f;
                pin(dom);
            }
        } else if constexpr (F < 27) {
            constexpr int u = 2 * (F - 23);
            hi[u] = cvt_bf16(p[2 * u], p[2 * u + 1]);
            hi[u + 1] = cvt_bf16(p[2 * u + 2], p[2 * u + 3]);
            pin(hi[u], hi[u + 1]);
        } else if constexpr (F < 31) {
            constexpr int u = 2 * (F - 27);
            if constexpr (kLo == kLoAlways) {
#pragma unroll
                for (int k = u; k < u + 2; ++k) lo[k] = cvt_bf16(p[2 * k] - bf16_lo(hi[k]), p[2 * k + 1] - bf16_hi(hi[k]));
                pin(lo[u], lo[u + 1]);
            } else {                         // the sum of the rounded weights: each pair times (1, 1), added in fp32
                sum_q = dot2_bf16(hi[u], 0x3f803f80u, sum_q);
                sum_q = dot2_bf16(hi[u + 1], 0x3f803f80u, sum_q);
                pin(sum_q);
            }
        }
    };
    static_for<kTileSteps>([&](auto f_c) {
        constexpr int F = decltype(f_c)::value;
        if constexpr (!kLast) {
            if constexpr (F + kTileKAhead < kTileSteps) load_k(std::integral_constant<int, F + kTileKAhead>());
        }
        if constexpr (F + kTileVAhead >= kTileSteps) va[F + kTileVAhead - kTileSteps] = tile_value_frag(cur, rd, F + kTileVAhead - kTileSteps);
        if constexpr (!kLast) {
            bf16x8_t qv;
            if constexpr (F < kTileQRegs) qv = qop[F];
            else qv = ql[F - kTileQRegs];
            if constexpr (F == 0) mfma_first_v(s_next, ka[F], qv);
            else if constexpr (F + 1 < kTileSteps) mfma_v(s_next, ka[F], qv);      // the last one below
            if constexpr (F % kTileLoadEvery == 3 && F / kTileLoadEvery < kTileLoadsA) issue(std::integral_constant<int, F / kTileLoadEvery>());
        }
        weights(f_c);
    });
    const bool with_lo = kLo == kLoAlways || (kLo == kLoDynamic && (exact || __builtin_amdgcn_ballot_w64(dom != 0.0f) != 0));
    st.lq += with_lo ? sum : sum_q;
    bf16x8_t ph[2], pl[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        ph[k] = __builtin_bit_cast(bf16x8_t, u32x4_t{hi[4 * k], hi[4 * k + 1], hi[4 * k + 2], hi[4 * k + 3]});
        if (kLo == kLoAlways) pl[k] = __builtin_bit_cast(bf16x8_t, u32x4_t{lo[4 * k], lo[4 * k + 1], lo[4 * k + 2], lo[4 * k + 3]});
    }
    mfma_operands(ph[0], ph[1]);
    if (kLo == kLoAlways) mfma_operands(pl[0], pl[1]);
    if constexpr (!kLast) {
        constexpr int kEnd = kTileSteps - 1;
        mfma_last_acc(s_next, ka[kEnd], ql[kEnd - kTileQRegs], o, va[0], ph[0], kLo == kLoAlways ? va[0] : va[1], kLo == kLoAlways ? pl[0] : ph[1]);
        if (__builtin_amdgcn_ballot_w64(j_next + kMlaKeys > lim) != 0) tile_mask(s_next, j_next, lim, h);   // blocks that reach a limit
    }
    // Phase B.
    constexpr int kDone = kLast ? 0 : kLo == kLoAlways ? 1 : 2;      // fragments whose MFMAs went with the last scores
    float t0, t1;
    static_for<kTileFrags>([&](auto c_c) {
        constexpr int C = decltype(c_c)::value;
        if constexpr (C + kTileVAhead < kTileFrags) va[C + kTileVAhead] = tile_value_frag(cur, rd, C + kTileVAhead);
        if constexpr (C >= kDone) {
            acc_mfma<(C >> 1)>(o, va[C], ph[C & 1]);
            if constexpr (kLo == kLoAlways) acc_mfma<(C >> 1)>(o, va[C], pl[C & 1]);
        }
        if constexpr (!kLast) {
            // The maximum of the next block's scores.
            if constexpr (C == 3) pin(s_next);
            if constexpr (C == 4) {
                t0 = max3(s_next[0], s_next[1], s_next[2]);
                t1 = max3(s_next[3], s_next[4], s_next[5]);
                pin(t0, t1);
            } else if constexpr (C >= 5 && C < 9) {
                t0 = max3(t0, s_next[2 * C - 4], s_next[2 * C - 3]);
                if constexpr (C == 8) t0 = max3(t0, s_next[14], s_next[15]);
                pin(t0);
            } else if constexpr (C == 9) {
                t0 = max3(t0, t1, t1);
                st.mx = tile_max(t0) * scale_log2;
                pin(st.mx);
            }
            if constexpr (C % kTileLoadEvery == 3 && C / kTileLoadEvery + kTileLoadsA < kTileLoads) issue(std::integral_constant<int, C / kTileLoadEvery + kTileLoadsA>());
        }
    });
    if (kLo == kLoDynamic && with_lo) {
        // The rare block with a dominant key: a second pass over the value fragments with the lo parts.
#pragma unroll
        for (int k = 0; k < 8; ++k) lo[k] = cvt_bf16(p[2 * k] - bf16_lo(hi[k]), p[2 * k + 1] - bf16_hi(hi[k]));
#pragma unroll
        for (int k = 0; k < 2; ++k) pl[k] = __builtin_bit_cast(bf16x8_t, u32x4_t{lo[4 * k], lo[4 * k + 1], lo[4 * k + 2], lo[4 * k + 3]});
        mfma_operands(pl[0], pl[1]);
        static_for<kTileFrags + kTileVAhead>([&](auto f_c) {
            constexpr int F = decltype(f_c)::value, C = F - kTileVAhead;
            if constexpr (F < kTileFrags) va[F] = tile_value_frag(cur, rd, F);
            if constexpr (C >= 0) acc_mfma<(C >> 1)>(o, va[C], pl[C & 1]);
        });
    }
}

// kMode: as mla_decode_kernel.  The form with two waves per tile: see mla_tile_split.  There each of the two computes the
// tile's scores and weights for itself and accumulates half of the columns.
template <int kMode>
__global__ __launch_bounds__(64 * kTileWaves) void mla_tile_kernel(
        const int32_t* __restrict__ kv_lens, const void* const* c_ptrs, int batch, int n_pieces, int min_piece,
        int few_pieces, int few_min, int xcd_skew, int q_len, int n_heads, MlaParams prm) {
    __shared__ __attribute__((aligned(16))) char lds_c[kTileStages * kTileBlock];
    __shared__ __attribute__((aligned(16))) char lds_q[kTileWaves * kTileQLds];      // each lane reads back what it wrote
    const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
    const int n = lane & 31, h = lane >> 5;
    const int T = q_len, H = n_heads, rows_total = T * H;
    SeqWindow win;
    const WavePlan wp = wave_plan(kv_lens, c_ptrs, nullptr, batch, n_pieces, min_piece, kMlaSegCost,
                                  xcd_skew, FewPieces{few_pieces, few_min}, lane, &win);
    const Plan& pl = wp.pl;
    auto work = [&](auto split_c) {
        constexpr int kSplit = decltype(split_c)::value;             // waves per tile
        constexpr int kN = kTileCols / kSplit, kTiles = kTileWaves / kSplit;     // column tiles per wave, row tiles per workgroup
        static_assert(kTiles * kTileRows * kTileStagePitch <= (kSplit == 1 ? 4 : 3) * kTileBlock, "output staging must fit the block buffers");
        const int bid = blockIdx.x;
        const MlaTileWork mine = mla_tile_work(pl, kSplit, rows_total, bid);
        const int p = mine.piece, s0 = piece_bound(pl, p), s1 = piece_bound(pl, p + 1);
        const bool active = mine.any && s0 < s1;
        if (tid < 64)
            for (int g = gridDim.x - 1 - bid; 64 * g < batch; g += gridDim.x) wave_write_meta(wp, kv_lens, batch, rows_total, g, lane, prm.meta);
        if (!active) return;       // the whole workgroup: every wave computed the same plan

        Walk walk;
        wave_locate(wp, kv_lens, c_ptrs, nullptr, batch, s0, lane, &win, walk.b, walk.j);
        walk.remaining = uniform(s1 - s0);
        dma_wait_all();

        const int tile = wave / kSplit, part = wave - tile * kSplit;
        const int wave_row0 = mine.row0 + tile * kTileRows;
        const bool busy = wave_row0 < rows_total;          // a wave without rows only loads
        const int row = wave_row0 + n;
        char* q_lds = lds_q + wave * kTileQLds + lane * 16;
        char* stage = lds_c + tile * (kTileRows * kTileStagePitch) + part * (kN * 64);
        const int exact_blocks = mla_exact_blocks(pl, rows_total, n_pieces);
        const TileDma dma = tile_dma(wave, lane);
        TileReads rd = tile_reads(lane);
        rd.value += part * (kN * 64);
        auto fence = [] {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        };

        PieceSeg ps;
        while (uniform(next_segment(walk, batch, pl.seg_cost,
                                    [&](int bb) { return window_len(win, kv_lens, bb); }, ps))) {
            const int b = uniform(ps.b), L = uniform(ps.L), j0 = uniform(ps.j0), j1 = uniform(ps.j1);
            const bool whole = uniform(ps.whole) != 0;
            const long slot = (long)uniform(p) + b;
            const unsigned long long cbytes = (unsigned long long)L * kRowB;
            const uint64_t caddr = (uint64_t)(uintptr_t)window_ptr(win, win.k, c_ptrs, b);
            const u32x4_t rc = {(uint32_t)uniform((int)(uint32_t)caddr), (uint32_t)uniform((int)((uint32_t)(caddr >> 32) & 0xffffu)),
                                cbytes > 0xffffffffull ? 0xffffffffu : (uint32_t)cbytes, 0x00020000u};
            const int n_blocks = (j1 - j0 + kMlaKeys - 1) / kMlaKeys;
            // The loads of block blk.  Past the segment's end they run against an empty descriptor (zeros land in a free
            // buffer), so that every block has its loads and the waits need no case.
            auto load_for = [&](int blk) {
                u32x4_t r = rc;
                if (blk >= n_blocks) r[2] = 0u;
                return tile_load_for(lds_c + (blk & 3) * kTileBlock, r, j0 + blk * kMlaKeys, wave);
            };
            auto load_block = [&](int blk) {
                const TileLoad b = load_for(blk);
                static_for<kTileLoads>([&](auto q_c) { tile_load<decltype(q_c)::value>(b, dma); });
            };

            // Q operand: lane (h, n) holds columns 16 step + 8 h .. + 7 of row n; rows past the last lie past the end of the
            // descriptor and read as zero.
            const uint64_t qaddr = (uint64_t)(uintptr_t)(prm.q + (long)b * rows_total * kDqk);
            const u32x4_t rq = {(uint32_t)uniform((int)(uint32_t)qaddr), (uint32_t)uniform((int)((uint32_t)(qaddr >> 32) & 0xffffu)),
                                (uint32_t)rows_total * kRowB, 0x00020000u};
            bf16x8_t qop[kTileQRegs];
            TileAcc o;
            f32x16_t s_even, s_odd;
            TileRow st{kNegInf, 0.0f, 0.0f, kNegInf};
            const int causal = L - T + (row < rows_total ? row : 0) / H + 1;
            const int lim = causal < j1 ? causal : j1;
            acc_zero<kN>(o);
            // Q goes through the buffers behind those of blocks 0 and 1, in the wave's own part of them.
            static_assert(kTileWaves * kTileQStage <= 2 * kTileBlock && kTileQRegs == 33, "Q's stage; the steps that are parked");
            char* q_stage = lds_c + 2 * kTileBlock + wave * kTileQStage;
            int q_lane = lane;
            pin(q_lane);              // the addresses are made here: kept from segment to segment they would be spilled
            auto park = [&](int step) { *reinterpret_cast<bf16x8_t*>(q_lds + (step - kTileQRegs) * 1024) = tile_q_frag(q_stage, q_lane, step); };
            if (busy) tile_q_load(q_stage, rq, wave_row0, q_lane, 0, bid >> 3);
            load_block(0);
            if (busy) {
                dma_wait_for<kTileLoads>();
#pragma unroll
                for (int step = 0; step < 16; ++step) qop[step] = tile_q_frag(q_stage, q_lane, step);
                qop[32] = tile_q_frag(q_stage, q_lane, 32);
                park(33);
#pragma unroll
                for (int step = 0; step < 16; ++step) pin(qop[step]);      // read before the second round overwrites them
                pin(qop[32]);
                fence();
                tile_q_load(q_stage, rq, wave_row0, q_lane, 1, bid >> 3);
            }
            load_block(1);
            dma_wait_for<kTileLoads>();
            if (busy) {
#pragma unroll
                for (int step = 16; step < 32; ++step) qop[step] = tile_q_frag(q_stage, q_lane, step);
                park(34);
                park(35);
#pragma unroll
                for (int step = 16; step < 32; ++step) pin(qop[step]);
                fence();
            }
            __syncthreads();
            load_block(2);
            if (busy) {
                // Scores of block 0.
                bf16x8_t ka[kTileSteps], ql[kTileSteps - kTileQRegs];
                auto load_k = [&](auto f_c) {
                    constexpr int F = decltype(f_c)::value;
                    ka[F] = tile_key_frag(lds_c, rd, F);
                    if constexpr (F >= kTileQRegs) ql[F - kTileQRegs] = *reinterpret_cast<const bf16x8_t*>(q_lds + (F - kTileQRegs) * 1024);
                };
                static_for<kTileKAhead>(load_k);
                static_for<kTileSteps>([&](auto f_c) {
                    constexpr int F = decltype(f_c)::value;
                    if constexpr (F + kTileKAhead < kTileSteps) load_k(std::integral_constant<int, F + kTileKAhead>());
                    bf16x8_t qv;
                    if constexpr (F < kTileQRegs) qv = qop[F];
                    else qv = ql[F - kTileQRegs];
                    if constexpr (F == 0) mfma_first_v(s_even, ka[F], qv);
                    else if constexpr (F + 1 < kTileSteps) mfma_v(s_even, ka[F], qv);
                    else mfma_last_v(s_even, ka[F], qv);
                });
                if (__builtin_amdgcn_ballot_w64(j0 + kMlaKeys > lim) != 0) tile_mask(s_even, j0, lim, h);
                float mx = max3(s_even[0], s_even[1], s_even[2]);
#pragma unroll
                for (int t = 3; t < 15; t += 2) mx = max3(mx, s_even[t], s_even[t + 1]);
                st.mx = tile_max(max3(mx, s_even[15], s_even[15])) * prm.scale_log2;
            }
            // Block blk while block blk + 1 is scored.  Every wave waits for its own loads of block blk + 1 (those of block
            // blk + 2 may stay in flight), then the barrier: block blk + 1 is in LDS and everyone is done with block blk - 1,
            // whose buffer the loads of block blk + 3 overwrite.
            auto step = [&](int blk, f32x16_t& s, f32x16_t& s_next, auto lo_mode) {
                dma_wait_for<kTileLoads>();
                __syncthreads();
                const TileLoad later = load_for(blk + 3);
                tile_block<decltype(lo_mode)::value, false, kN>(o, st, s, s_next, qop, q_lds, rd, lds_c + (blk & 3) * kTileBlock,
                                                            lds_c + ((blk + 1) & 3) * kTileBlock, prm.scale_log2, j0 + (blk + 1) * kMlaKeys,
                                                            lim, h, false, [&](auto q_c) { tile_load<decltype(q_c)::value>(later, dma); });
            };
            auto last = [&](f32x16_t& s, auto lo_mode) {
                tile_block<decltype(lo_mode)::value, true, kN>(o, st, s, s, qop, q_lds, rd, lds_c + ((n_blocks - 1) & 3) * kTileBlock, nullptr,
                                                           prm.scale_log2, 0, lim, h, n_blocks <= exact_blocks, [](auto) {});
            };
            // Default mode: the first blocks of a segment with hi + lo weights, the others with hi + lo only where a
            // key dominates.
            constexpr auto kFirstMode = std::integral_constant<int, kMode == 2 ? kLoNever : kLoAlways>();
            constexpr auto kThenMode = std::integral_constant<int, kMode == 0 ? kLoDynamic : kMode == 1 ? kLoAlways : kLoNever>();
            if (busy) {
                int blk = 0;
                for (; blk + 1 < n_blocks && blk < exact_blocks; ++blk) {
                    step(blk, s_even, s_odd, kFirstMode);
                    s_even = s_odd;
                }
                for (; blk + 2 < n_blocks; blk += 2) {
                    step(blk, s_even, s_odd, kThenMode);
                    step(blk + 1, s_odd, s_even, kThenMode);
                }
                if (blk + 1 < n_blocks) {
                    step(blk, s_even, s_odd, kThenMode);
                    s_even = s_odd;
                    ++blk;
                }
                last(s_even, kThenMode);
                acc_drain<kN>(o);
            } else {
                for (int blk = 0; blk + 1 < n_blocks; ++blk) {
                    dma_wait_for<kTileLoads>();
                    __syncthreads();
                    load_block(blk + 3);
                }
            }
            dma_wait_for<0>();        // the empty loads behind the last block: they write (zeros) to the buffers
            __syncthreads();          // everyone is done with the block buffers: they stage the output now
            // Rounded as in mla_decode_kernel: bf16 results; partial rows fp16, scaled to the row's largest magnitude, which
            // the waves of a tile agree on in LDS.
            float amax = 0.0f;
            float* amax_of = reinterpret_cast<float*>(lds_c + 3 * kTileBlock);
            if (!whole) {
                if (busy) {
                    float m4[4] = {0.0f, 0.0f, 0.0f, 0.0f};
                    static_for<kN>([&](auto ct_c) {
                        float v[16];
                        acc_read<decltype(ct_c)::value>(o, v);
#pragma unroll
                        for (int i = 0; i < 16; i += 2) max3_abs(m4[(i / 2) & 3], v[i], v[i + 1]);
                    });
                    amax = tile_max(fmaxf(fmaxf(m4[0], m4[1]), fmaxf(m4[2], m4[3])));
                    if (kSplit > 1 && h == 0) amax_of[wave * kTileRows + n] = amax;
                }
                if constexpr (kSplit > 1) __syncthreads();
            }
            if (busy) {
                const float l = st.l;
                float lq, lq_b;
                swap32(st.lq, lq, lq_b);
                lq += lq_b;
                float sc, inv_scale = 0.0f;
                if (whole) {
                    sc = lq > 0.0f ? 1.0f / lq : 0.0f;
                } else {
                    if constexpr (kSplit == 2) amax = fmaxf(amax, amax_of[(wave ^ 1) * kTileRows + n]);
                    sc = amax > 0.0f ? fminf(32768.0f / amax, 0x1.0p100f) : 0.0f;
                    inv_scale = amax > 0.0f ? 1.0f / sc : 0.0f;
                }
                uint16_t* dst = whole ? prm.out + (long)b * rows_total * kDv : prm.part_o + slot * rows_total * kDv;
                const __amdgpu_buffer_rsrc_t rd_out = make_rsrc(uniform(static_cast<void*>(dst)), (uint32_t)rows_total * (kDv * 2));
                // 128 columns at a time through the stage, their rows stored behind the rounding of the next 128; four rows of
                // 256 bytes per store, rows past the last are dropped.
                int lane_out = lane;
                pin(lane_out);        // as q_lane
                char* lane_stage = stage + (lane_out & 31) * kTileStagePitch + 8 * (lane_out >> 5);
                const char* lane_rows = stage + (lane_out >> 4) * kTileStagePitch + (lane_out & 15) * 16;
                const int lane_dst = (wave_row0 + (lane_out >> 4)) * (kDv * 2) + part * (kN * 64) + (lane_out & 15) * 16;
                auto round_quarter = [&](auto q_c, auto whole_c) {
                    static_for<4>([&](auto t_c) {
                        constexpr int ct = decltype(q_c)::value * 4 + decltype(t_c)::value;
                        float v[16];
                        acc_read<ct>(o, v);
#pragma unroll
                        for (int i = 0; i < 16; ++i) v[i] *= sc;
#pragma unroll
                        for (int g = 0; g < 4; ++g)      // columns 32 ct + 8 g + 4 h .. + 3 of row n
                            *reinterpret_cast<uint2*>(lane_stage + (32 * ct + 8 * g) * 2) =
                                decltype(whole_c)::value ? make_uint2(cvt_bf16(v[4 * g], v[4 * g + 1]), cvt_bf16(v[4 * g + 2], v[4 * g + 3]))
                                                         : make_uint2(pack_f16(v[4 * g], v[4 * g + 1]), pack_f16(v[4 * g + 2], v[4 * g + 3]));
                    });
                    fence();
                };
                auto store_quarter = [&](int q) {
#pragma unroll
                    for (int i = 0; i < kTileRows / 4; ++i) {
                        const u32x4_t w = *reinterpret_cast<const u32x4_t*>(lane_rows + 4 * i * kTileStagePitch + q * 256);
                        __builtin_amdgcn_raw_buffer_store_b128(w, rd_out, lane_dst + 4 * i * (kDv * 2) + q * 256, 0, 0);
                    }
                };
                auto store_rows = [&](auto whole_c) {
                    static_for<kN / 4>([&](auto q_c) {
                        round_quarter(q_c, whole_c);
                        if constexpr (decltype(q_c)::value > 0) store_quarter(decltype(q_c)::value - 1);
                    });
                    store_quarter(kN / 4 - 1);
                };
                if (whole) store_rows(std::true_type());
                else store_rows(std::false_type());
                if (row < rows_total && h == 0 && part == 0) {
                    if (whole) {
                        if (prm.lse) prm.lse[(long)b * rows_total + row] = l > 0.0f ? (st.m + __log2f(l)) * kLn2 : kNegInf;
                    } else {
                        reinterpret_cast<float4*>(prm.part_ml)[slot * rows_total + row] = make_float4(st.m, l, lq, inv_scale);
                    }
                }
            }
            __syncthreads();          // the next segment's first block goes to buffer 0, which staged output until here
        }
    };
    if (mla_tile_split(pl, n_pieces, rows_total) == 2) work(std::integral_constant<int, 2>());
    else work(std::integral_constant<int, 1>());
}


// ----------------------------------------------------------------------- few query rows: 32 at most
// With 16 rows (heads split over several GPUs) a cached byte meets 30 flop: bound by HBM, and what matters
// is that a compute unit keeps its loads in flight.  One wave per 16 rows does not: it issues 38 loads per
// block, then works through the block alone (2.4 TB/s at 16 rows).  Here four waves share a
// 16-row tile: of a block's scores wave q computes key tile q % 2 over half q / 2 of the key width (9 MFMAs,
// 36 registers of Q), the four partial tiles meet in LDS, every wave does the (small) softmax of the whole
// tile for itself, and accumulates 128 of the 512 value columns (8 MFMAs, 32 accumulators).  No operand
// is read from LDS twice per tile, and nothing has to be combined at the end of a segment but the rows'
// largest magnitudes.  Two barriers per block, two blocks in flight behind the one in use.
// The weights enter the value product as hi + lo bf16 parts throughout (the matrix cores are idle
// anyway), or as one bf16 where the caller asked for that.
// Measured, 64 sequences of 1024 to 8192 tokens, 16 heads: call 135.1 -> 61.3 us
// (5.4 TB/s); 32 sequences of 16384 tokens: 16 rows 221 -> 104 us, 32 rows 165 -> 107. At 64 rows this layout
// (two tiles per wave) takes 154 us where one wave per tile takes 134: the line lies at 32.
constexpr int kRowsSegCost = 96;                 // a segment's fixed work in tokens (48: +2 %, 160: +0.7 %)
constexpr int kRowsSteps = kQSteps / 2;          // score steps per wave
constexpr int kRowsCols = kColTiles / 4;         // value column tiles per wave
constexpr int kRowsStagePitch = kRowsCols * 32 + 16;

template <int RT, bool kLo>
__global__ __launch_bounds__(256 * RT) void mla_rows_kernel(
        const int32_t* __restrict__ kv_lens, const void* const* c_ptrs, int batch, int n_pieces, int min_piece,
        int few_pieces, int few_min, int xcd_skew, int q_len, int n_heads, MlaParams prm) {
    constexpr int NW = 4 * RT;
    __shared__ __attribute__((aligned(16))) char lds_c[kStages * kLdsBlock];
    __shared__ f32x4_t lds_x[RT][4][64];    // partial scores: [rt][key tile + 2 * half][lane]
    __shared__ float lds_amax[RT][4][16];
    static_assert(NW * 16 * kRowsStagePitch <= kStages * kLdsBlock, "output staging must fit the block buffers");
    const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
    const int kb = lane >> 4, n = lane & 15;
    const int rt = wave >> 2, quarter = wave & 3, kt = quarter & 1, half = quarter >> 1;
    const int T = q_len, H = n_heads, rows_total = T * H;
    SeqWindow win;
    const WavePlan wp = wave_plan(kv_lens, c_ptrs, nullptr, batch, n_pieces, min_piece, kRowsSegCost,
                                  xcd_skew, FewPieces{few_pieces, few_min}, lane, &win);
    const Plan& pl = wp.pl;
    const int per_xcd = (pl.n_pieces + 7) >> 3;
    const int bid = blockIdx.x;
    const int p = (bid & 7) * per_xcd + (bid >> 3);
    const int s0 = piece_bound(pl, p), s1 = piece_bound(pl, p + 1);
    const bool active = (bid >> 3) < per_xcd && p < pl.n_pieces && s0 < s1;
    if (tid < 64)
        for (int g = gridDim.x - 1 - bid; 64 * g < batch; g += gridDim.x) wave_write_meta(wp, kv_lens, batch, rows_total, g, lane, prm.meta);
    if (!active) return;       // the whole workgroup: every wave computed the same plan

    Walk walk;
    wave_locate(wp, kv_lens, c_ptrs, nullptr, batch, s0, lane, &win, walk.b, walk.j);
    walk.remaining = uniform(s1 - s0);

    const DmaLane dma = dma_lane(lane);
    const int my_loads = (kDmaPerBlock - wave + NW - 1) / NW;
    // Step t of the wave's half: MFMA step 9 * half + t; steps 16 and 17 lie in the tail area.
    const int qk_off = (16 * kt + n) * kPitch + kb * 16 + half * kRowsSteps * 64;
    const int qt_off = kTailOff + (16 * kt + n) * kTailPitch + kb * 16;
    const int pv_off = (4 * kb + (n >> 2)) * kPitch + (n & 3) * 8 + quarter * kRowsCols * 32;
    char* stage = lds_c + wave * (16 * kRowsStagePitch);
    auto fence = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };

    PieceSeg ps;
    while (uniform(next_segment(walk, batch, pl.seg_cost,
                                [&](int bb) { return window_len(win, kv_lens, bb); }, ps))) {
        const int b = uniform(ps.b), L = uniform(ps.L), j0 = uniform(ps.j0), j1 = uniform(ps.j1);
        const bool whole = uniform(ps.whole) != 0;
        const long slot = (long)uniform(p) + b;
        const unsigned long long cbytes = (unsigned long long)L * kRowB;
        const uint64_t caddr = (uint64_t)(uintptr_t)window_ptr(win, win.k, c_ptrs, b);
        const u32x4_t rc = {(uint32_t)uniform((int)(uint32_t)caddr), (uint32_t)uniform((int)((uint32_t)(caddr >> 32) & 0xffffu)),
                            cbytes > 0xffffffffull ? 0xffffffffu : (uint32_t)cbytes, 0x00020000u};
        const int n_blocks = (j1 - j0 + kMlaKeys - 1) / kMlaKeys;
        // Q operand: lane (kb, n) holds columns 32 step + 8 kb .. + 7 of row n; rows past the last read as zero.
        const __amdgpu_buffer_rsrc_t rq = make_rsrc(prm.q + (long)b * rows_total * kDqk, (uint32_t)rows_total * kRowB);
        const int row = 16 * rt + n;             // of the sequence's T * H rows
        bf16x8_t qop[kRowsSteps];
#pragma unroll
        for (int t = 0; t < kRowsSteps; ++t)
            qop[t] = __builtin_bit_cast(bf16x8_t, __builtin_amdgcn_raw_buffer_load_b128(
                                                      rq, row * kRowB + (half * kRowsSteps + t) * 64 + kb * 16, 0, 0));
        const int causal = L - T + (row < rows_total ? row : 0) / H + 1;
        const int lim = causal < j1 ? causal : j1;
        block_to_lds<NW>(lds_c, rc, j0, wave, dma);
        // Q is used here so that the wait for its loads sits outside the loop (see mla_decode_kernel).
#pragma unroll
        for (int t = 0; t < kRowsSteps; ++t) asm volatile("" : "+v"(qop[t]));
        if (n_blocks > 1) block_to_lds<NW>(lds_c + kLdsBlock, rc, j0 + kMlaKeys, wave, dma);

        f32x4_t o[kRowsCols];
        float m = kNegInf, l = 0.0f, lq = 0.0f;
#pragma unroll
        for (int c = 0; c < kRowsCols; ++c) o[c] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
        int cur_buf = 0, next_buf = 2;
        for (int blk = 0; blk < n_blocks; ++blk) {
            const char* cur = lds_c + cur_buf * kLdsBlock;
            // every wave waits for its own loads of block blk; behind the barrier the block is in LDS and
            // everyone is done with block blk - 1 and its partial scores
            dma_wait(blk + 1 < n_blocks ? my_loads : 0);
            __syncthreads();
            if (blk + 2 < n_blocks) block_to_lds<NW>(lds_c + next_buf * kLdsBlock, rc, j0 + (blk + 2) * kMlaKeys, wave, dma);
            f32x4_t s = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int t = 0; t < kRowsSteps; ++t) {
                // the wave's half decides (uniformly) whether its last two steps read the tail area
                const bool tail = t >= kMainSteps - kRowsSteps && half == 1;
                const bf16x8_t a = *reinterpret_cast<const bf16x8_t*>(
                    cur + (tail ? qt_off + (t - (kMainSteps - kRowsSteps)) * 64 : qk_off + t * 64));
                s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, qop[t], s, 0, 0, 0);
            }
            lds_x[rt][quarter][lane] = s;
            __syncthreads();
            float q[8];                          // scores, then weights: key 16 kt + 4 kb + i at index 4 kt + i
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const f32x4_t sum = lds_x[rt][k][lane] + lds_x[rt][k + 2][lane];
#pragma unroll
                for (int i = 0; i < 4; ++i) q[4 * k + i] = sum[i];
            }
            bf16x8_t va[kRowsCols];              // value fragments: see mla_block for the transposing read
#pragma unroll
            for (int c = 0; c < kRowsCols; ++c) {
                const s16x4v_t v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (__attribute__((address_space(3))) s16x4v_t*)(cur + pv_off + c * 32));
                const s16x4v_t v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                    (__attribute__((address_space(3))) s16x4v_t*)(cur + pv_off + kTileB + c * 32));
                const u32x2_t w0 = __builtin_bit_cast(u32x2_t, v0), w1 = __builtin_bit_cast(u32x2_t, v1);
                va[c] = __builtin_bit_cast(bf16x8_t, u32x4_t{w0.x, w0.y, w1.x, w1.y});
            }
            const int j_block = j0 + blk * kMlaKeys;
            if (__builtin_amdgcn_ballot_w64(j_block + kMlaKeys > lim) != 0) {
#pragma unroll
                for (int t = 0; t < 8; ++t) q[t] = j_block + 16 * (t >> 2) + 4 * kb + (t & 3) < lim ? q[t] : kNegInf;
            }
            float mx = max_num(max_num(max_num(q[0], q[1]), max_num(q[2], q[3])), max_num(max_num(q[4], q[5]), max_num(q[6], q[7])));
            mx = kb_max(mx) * prm.scale_log2;
            const bool moves = mx > m + kLazyLog2;          // the reference maximum follows lazily, see mla_block
            if (__builtin_amdgcn_ballot_w64(moves) != 0) {
                const float m_new = moves ? mx : m;
                const float alpha = moves ? fast_exp2(m - m_new) : 1.0f;
                m = m_new;
                l *= alpha;
                lq *= alpha;
#pragma unroll
                for (int c = 0; c < kRowsCols; ++c) o[c] *= alpha;
            }
            const float m_use = m == kNegInf ? 0.0f : m;
#pragma unroll
            for (int t = 0; t < 8; ++t) q[t] = fast_exp2(__builtin_fmaf(q[t], prm.scale_log2, -m_use));
            const float sum = ((q[0] + q[1]) + (q[2] + q[3])) + ((q[4] + q[5]) + (q[6] + q[7]));
            l += sum;                            // this lane's share of the row's sums, both
            uint32_t hi[4], lo[4] = {0u, 0u, 0u, 0u};
            float sum_q = 0.0f;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                hi[u] = cvt_bf16(q[2 * u], q[2 * u + 1]);
                const f32x2_t back = __builtin_convertvector(__builtin_bit_cast(bf16x2_t, hi[u]), f32x2_t);
                if (kLo) lo[u] = cvt_bf16(q[2 * u] - back[0], q[2 * u + 1] - back[1]);
                else sum_q += back[0] + back[1];
            }
            lq += kLo ? sum : sum_q;             // one bf16 per weight: normalised by the rounded weights, see mla_block
            const bf16x8_t ph = __builtin_bit_cast(bf16x8_t, u32x4_t{hi[0], hi[1], hi[2], hi[3]});
            const bf16x8_t plo = __builtin_bit_cast(bf16x8_t, u32x4_t{lo[0], lo[1], lo[2], lo[3]});
#pragma unroll
            for (int c = 0; c < kRowsCols; ++c)
                o[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[c], ph, o[c], 0, 0, 0);
            if constexpr (kLo) {
#pragma unroll
                for (int c = 0; c < kRowsCols; ++c)
                    o[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va[c], plo, o[c], 0, 0, 0);
            }
            cur_buf = cur_buf == kStages - 1 ? 0 : cur_buf + 1;
            next_buf = next_buf == kStages - 1 ? 0 : next_buf + 1;
        }
        // The wave's rows x 128 columns, rounded as in mla_decode_kernel (bf16 results; partial rows fp16
        // scaled to the largest magnitude of the whole row, which the tile's four waves agree on in LDS).
        if (!whole) {
            float amax = 0.0f;
#pragma unroll
            for (int c = 0; c < kRowsCols; ++c)
#pragma unroll
                for (int i = 0; i < 4; ++i) amax = fmaxf(amax, __builtin_fabsf(o[c][i]));
            amax = kb_max(amax);
            if (kb == 0) lds_amax[rt][quarter][n] = amax;
        }
        __syncthreads();                         // everyone is done with the block buffers: they stage the output now
        uint16_t* dst = whole ? prm.out + (long)b * rows_total * kDv : prm.part_o + slot * rows_total * kDv;
        const __amdgpu_buffer_rsrc_t rd = make_rsrc(uniform(static_cast<void*>(dst)), (uint32_t)rows_total * (kDv * 2));
        const float l_row = kb_sum(l), lq_row = kb_sum(lq);
        float sc, inv_scale = 0.0f;
        if (whole) {
            sc = lq_row > 0.0f ? 1.0f / lq_row : 0.0f;
        } else {
            const float amax = fmaxf(fmaxf(lds_amax[rt][0][n], lds_amax[rt][1][n]), fmaxf(lds_amax[rt][2][n], lds_amax[rt][3][n]));
            sc = amax > 0.0f ? fminf(32768.0f / amax, 0x1.0p100f) : 0.0f;
            inv_scale = amax > 0.0f ? 1.0f / sc : 0.0f;
        }
#pragma unroll
        for (int c = 0; c < kRowsCols; ++c) {
            const f32x4_t v = o[c] * sc;
            uint2 d;
            d.x = whole ? cvt_bf16(v[0], v[1]) : pack_f16(v[0], v[1]);
            d.y = whole ? cvt_bf16(v[2], v[3]) : pack_f16(v[2], v[3]);
            *reinterpret_cast<uint2*>(stage + n * kRowsStagePitch + (16 * c + 4 * kb) * 2) = d;
        }
        fence();
#pragma unroll
        for (int i = 0; i < 4; ++i) {        // rows 4 i .. 4 i + 3, 256 bytes each; rows past the last are dropped
            const int r = 4 * i + kb;
            const u32x4_t d = *reinterpret_cast<const u32x4_t*>(stage + r * kRowsStagePitch + n * 16);
            __builtin_amdgcn_raw_buffer_store_b128(d, rd, (16 * rt + r) * (kDv * 2) + quarter * (kRowsCols * 32) + n * 16, 0, 0);
        }
        fence();
        if (row < rows_total && kb == 0 && quarter == 0) {
            if (whole) {
                if (prm.lse) prm.lse[(long)b * rows_total + row] = l_row > 0.0f ? (m + __log2f(l_row)) * kLn2 : kNegInf;
            } else {
                reinterpret_cast<float4*>(prm.part_ml)[slot * rows_total + row] = make_float4(m, l_row, lq_row, inv_scale);
            }
        }
        __syncthreads();          // the next segment's first block goes to buffer 0, which staged output until here
    }
}

// kWaves waves per output row of 512 columns; lane holds columns 8*lane .. 8*lane+7.  A partial row is 512
// fp16 values times its own scale (the fourth value of its (m, l, lq, 1 / scale) record).  Bound by the partial rows'
// bytes in large calls and by its dependent steps in small ones: as merge_kernel, and 8 partial rows on their way
// instead of 4 (the whole call: 29 sequences of 131 to 262 tokens, 64 rows 20.2 -> 19.4 us; 64 of 1024 to 8192, 16
// rows 61.9 -> 60.9; 128 rows 109.6 -> 108.9).
// kRead = kReadOwn: non-temporal there, 1.5 to 2 us more of a large call.  kReadFarOnce, through the L2s before: 3 of 817 to 13076
// tokens, 64 rows 31.6 -> 30.4 us; 7 of 2216 to 17728, 72 rows 41.1 -> 39.9; one of 30000, 128 rows 37.6 -> 36.7.
template <int kWaves, int kRead>
__global__ __launch_bounds__(kWaves == 1 ? 256 : 64 * kWaves) void mla_merge_kernel(
        const int32_t* __restrict__ meta, const float* __restrict__ part_ml, const uint16_t* __restrict__ part_o, uint16_t* __restrict__ out,
        float* __restrict__ lse, int batch, uint32_t seq_rows, uint32_t per_xcd) {
    const int lane = threadIdx.x & 63;
    const int wave = uniform(threadIdx.x >> 6);
    const MergeRow mr = merge_row<kWaves, kRead>(meta, (uint32_t)batch, seq_rows, per_xcd, wave);
    const uint32_t row = mr.row, b = mr.b;
    const int n = mr.n;
    if (n == 1) return;
    const MergeShare sh = merge_share<kWaves>(n, wave);
    if (sh.alone && kWaves > 1 && wave > 0) return;       // few slots: the first wave does the row
    uint4* outp = reinterpret_cast<uint4*>(out + (long)row * kDv) + lane;
    if (n == 0) {
        *outp = make_uint4(0u, 0u, 0u, 0u);
        if (lse && lane == 0) lse[row] = kNegInf;
        return;
    }
    const long stride_rows = seq_rows, first_row = (long)mr.first_slot * stride_rows + (row - b * seq_rows);
    const float4* ml = reinterpret_cast<const float4*>(part_ml) + first_row;   // (m, l, lq, 1 / scale)
    const u32x4_t* po = reinterpret_cast<const u32x4_t*>(part_o + first_row * kDv) + lane;
    const long po_stride = stride_rows * (kDv / 8);
    auto record = [&](int s) {
        float4 r = make_float4(kNegInf, 0.0f, 0.0f, 0.0f);
        if (s < sh.end) r = ml[s * stride_rows];
        return r;
    };
    float M = kNegInf, l = 0.0f, lq = 0.0f;
    float acc[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
    if (sh.first < sh.end) {
        float4 mine = record(sh.first + lane);
        u32x4_t o[8];
        auto load = [&](int s0) {
#pragma unroll
            for (int u = 0; u < 8; ++u) o[u] = load_partial<kRead>(&po[(s0 + u < sh.end ? s0 + u : sh.end - 1) * po_stride]);
        };
        load(sh.first);
        M = mine.x;
        for (int base = sh.first + 64; base < sh.end; base += 64)
            if (base + lane < sh.end) M = fmaxf(M, ml[(base + lane) * stride_rows].x);
        M = wave_max(M);
        const float m_use = (M == kNegInf) ? 0.0f : M;
        float w = fast_exp2(mine.x - m_use);               // lanes past the end: 0
        l = mine.y * w;
        lq = mine.z * w;
        float ws = w * mine.w;                             // weight times the inverse of the row's scale
        for (int i0 = 0; sh.first + i0 < sh.end; i0 += 8) {
            const int s0 = sh.first + i0;
            if (i0 > 0) {
                if ((i0 & 63) == 0) {
                    mine = record(s0 + lane);
                    w = fast_exp2(mine.x - m_use);
                    l = __builtin_fmaf(mine.y, w, l);
                    lq = __builtin_fmaf(mine.z, w, lq);
                    ws = w * mine.w;
                }
                load(s0);
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const float ws_s = lane_value(ws, (i0 + u) & 63);
                if (s0 + u < sh.end) {                    // past the end: nothing, also where the row read is infinite
                    const uint32_t q[4] = {o[u].x, o[u].y, o[u].z, o[u].w};
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const f32x2_t v = __builtin_convertvector(__builtin_bit_cast(f16x2_t, q[c]), f32x2_t);
                        acc[2 * c] = __builtin_fmaf(v[0], ws_s, acc[2 * c]);
                        acc[2 * c + 1] = __builtin_fmaf(v[1], ws_s, acc[2 * c + 1]);
                    }
                }
            }
        }
        l = wave_sum(l);
        lq = wave_sum(lq);
    }
    if constexpr (kWaves > 1) {
        if (!sh.alone) {                                  // the waves' sums, each against its own maximum, meet in LDS
            __shared__ f32x4_t part[kWaves][2][64];
            __shared__ f32x4_t wave_ml[kWaves];
            part[wave][0][lane] = f32x4_t{acc[0], acc[1], acc[2], acc[3]};
            part[wave][1][lane] = f32x4_t{acc[4], acc[5], acc[6], acc[7]};
            if (lane == 0) wave_ml[wave] = f32x4_t{M, l, lq, 0.0f};
            __syncthreads();
            if (wave > 0) return;
#pragma unroll
            for (int w = 1; w < kWaves; ++w) M = fmaxf(M, wave_ml[w][0]);
            const float m_all = (M == kNegInf) ? 0.0f : M;
            l = lq = 0.0f;
#pragma unroll
            for (int c = 0; c < 8; ++c) acc[c] = 0.0f;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) {
                const float f = fast_exp2(wave_ml[w][0] - m_all);
                l = __builtin_fmaf(wave_ml[w][1], f, l);
                lq = __builtin_fmaf(wave_ml[w][2], f, lq);
#pragma unroll
                for (int c = 0; c < 8; ++c) acc[c] = __builtin_fmaf(part[w][c >> 2][lane][c & 3], f, acc[c]);
            }
        }
    }
    const float inv = lq > 0.0f ? 1.0f / lq : 0.0f;
    uint4 w;
    w.x = cvt_bf16(acc[0] * inv, acc[1] * inv);
    w.y = cvt_bf16(acc[2] * inv, acc[3] * inv);
    w.z = cvt_bf16(acc[4] * inv, acc[5] * inv);
    w.w = cvt_bf16(acc[6] * inv, acc[7] * inv);
    *outp = w;
    if (lse && lane == 0) lse[row] = l > 0.0f ? (M + __log2f(l)) * kLn2 : kNegInf;
}

// A decode kernel on its arguments: those of the plan ahead of prm, see split_decode_kernel.
template <typename Kernel>
hipError_t launch_mla(Kernel kernel, const MlaParams& prm, dim3 grid, int threads, hipStream_t stream) {
    return launch(kernel, grid, threads, stream, prm.kv_lens, prm.c_ptrs, prm.batch, prm.n_pieces, prm.min_piece_tokens, prm.few.pieces,
                  prm.few.min_piece, prm.xcd_skew, prm.q_len, prm.n_heads, prm);
}

template <int NW>
hipError_t launch_mla_16(const MlaParams& prm, dim3 grid, hipStream_t stream) {
    if (prm.weight_mode == 1) return launch_mla(mla_decode_kernel<NW, 1>, prm, grid, 64 * NW, stream);
    if (prm.weight_mode == 2) return launch_mla(mla_decode_kernel<NW, 2>, prm, grid, 64 * NW, stream);
    return launch_mla(mla_decode_kernel<NW, 0>, prm, grid, 64 * NW, stream);
}

hipError_t launch_mla_tile(const MlaParams& prm, hipStream_t stream) {
    const dim3 grid((unsigned)mla_tile_grid(prm.n_pieces, prm.q_len * prm.n_heads));
    if (prm.weight_mode == 1) return launch_mla(mla_tile_kernel<1>, prm, grid, 64 * kTileWaves, stream);
    if (prm.weight_mode == 2) return launch_mla(mla_tile_kernel<2>, prm, grid, 64 * kTileWaves, stream);
    return launch_mla(mla_tile_kernel<0>, prm, grid, 64 * kTileWaves, stream);
}

template <int RT>
hipError_t launch_mla_rows(const MlaParams& prm, dim3 grid, hipStream_t stream) {
    if (prm.weight_mode == 2) return launch_mla(mla_rows_kernel<RT, false>, prm, grid, 256 * RT, stream);
    return launch_mla(mla_rows_kernel<RT, true>, prm, grid, 256 * RT, stream);
}

}  // namespace

// Workgroup shape for rows_total = q_len * n_heads query rows per sequence: (waves, 16-row tiles per wave).  Up to 32
// rows mla_rows_kernel (one row group, as the shape given here), which has its line there; then mla_tile_kernel, 128
// rows per workgroup: at 33 rows already 69.3 us against 77.7 with a wave per 16 rows.  layout 1: waves of 16 rows, 4
// at most, for any number of rows; layout 2: as 1 up to 64 rows, then mla_tile_kernel.
void mla_block_shape(int rows_total, int layout, int* waves, int* tiles_per_wave) {
    const int tiles = (rows_total + 15) / 16;
    const bool tile32 = layout != 1 && tiles > (layout == 2 ? 4 : 2);
    *tiles_per_wave = tile32 ? 2 : 1;
    *waves = tile32 || tiles >= 3 ? 4 : tiles;
}

hipError_t launch_mla_decode(const MlaParams& prm, hipStream_t stream, hipEvent_t* events) {
    const int rows_total = prm.q_len * prm.n_heads;
    int nw = 1, rt = 1;
    mla_block_shape(rows_total, prm.layout, &nw, &rt);
    dim3 grid((unsigned)((prm.n_pieces + 7) / 8 * 8 * ((rows_total + 16 * rt * nw - 1) / (16 * rt * nw))));
    hipError_t e;
    if (events && (e = hipEventRecord(events[0], stream)) != hipSuccess) return e;
    if (prm.layout == 0 && rows_total <= 16) e = launch_mla_rows<1>(prm, grid, stream);
    else if (prm.layout == 0 && rows_total <= 32) e = launch_mla_rows<2>(prm, grid, stream);
    else if (rt == 2) e = launch_mla_tile(prm, stream);
    else if (nw == 4) e = launch_mla_16<4>(prm, grid, stream);
    else if (nw == 2) e = launch_mla_16<2>(prm, grid, stream);
    else e = launch_mla_16<1>(prm, grid, stream);
    if (e != hipSuccess) return e;
    if (events && (e = hipEventRecord(events[1], stream)) != hipSuccess) return e;
    const long rows = (long)prm.batch * rows_total;
    e = launch_merge<0>(rows, prm.batch, [&](auto waves, auto read, unsigned grid) {
        constexpr int kWaves = decltype(waves)::value;
        return launch(mla_merge_kernel<kWaves, decltype(read)::value>, dim3(grid), kWaves == 1 ? 256 : 64 * kWaves, stream, prm.meta, prm.part_ml,
                      prm.part_o, prm.out, prm.lse, prm.batch, (uint32_t)rows_total, grid >> 3);
    });
    if (e != hipSuccess) return e;
    if (events && (e = hipEventRecord(events[2], stream)) != hipSuccess) return e;
    return hipSuccess;
}

}  // namespace xattn
