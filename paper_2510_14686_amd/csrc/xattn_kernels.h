// Internal interface between the C-ABI host code and the gfx950 kernels.
#ifndef XATTN_KERNELS_H_
#define XATTN_KERNELS_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "xattn_plan.h"

namespace xattn {

constexpr int kHeadDim = 128;
// Default share (per mille) moved from the odd-numbered XCDs' parts of the token stream to the
// even-numbered ones: on MI355X the odd XCDs need about 7 % longer for the same bytes (measured per
// wave with clock stamps on several machines; rotating the data among the XCDs moves nothing), so
// equal parts leave the even XCDs idle at the end of the kernel.
constexpr int kDefaultXcdSkewGqa = 32;
constexpr int kDefaultXcdSkewMla = 0;
constexpr int kMaxWavesPerBlock = 8;   // KV heads times the waves that share a piece (matrix path) or the pieces (vector path)

// Workspace header: per sequence two int32 words, (first partial slot, number of segments and kSpreadRows), written
// by the decode kernel for the merge kernel.  0 segments = no keys; 1 = finished by the decode kernel.

struct DecodeParams {
    const uint16_t* q;               // bf16 [batch, q_len, n_q_heads, 128]
    const void* const* k_ptrs;       // device array[batch] of device pointers
    const void* const* v_ptrs;
    const int32_t* kv_lens;          // device int32[batch]
    int batch, q_len, n_q_heads, n_kv_heads, group;
    float inv_group;                 // 1 / group
    float scale_log2;                // scale * log2(e)
    uint16_t* out;                   // bf16 [batch, q_len, n_q_heads, 128]
    float* lse;                      // fp32 [batch, q_len, n_q_heads] or null
    float* part_o;                   // fp32 [slots, q_len * n_q_heads, 128]
    float* part_ml;                  // fp32 [slots, q_len * n_q_heads, 2]  (max, sum)
    int32_t* meta;                   // int32 [batch, 2]
    int n_pieces;                    // vector path: pieces the token stream is cut into (upper bound on active ones); both: what the
                                     // workspace has slots for
    int parts;                       // and pieces per workgroup: waves per workgroup / KV heads per workgroup
    int shared_pieces;               // matrix path: pieces, n_pieces at most; share.parts waves per KV head work on each
    PieceShare share;
    int min_piece_tokens;            // of the path's pieces, as `few`
    FewPieces few;                   // see plan_for_total
    int xcd_skew;                    // per mille: share taken from the odd XCDs' parts of the stream and given to the even ones
    int path;                        // kPathAuto, kPathVector or kPathMatrix
    int pv_mode;                     // matrix path: kPvBf16x3, kPvFp32 or kPvBf16
};

// How the matrix path multiplies the softmax weights p with V.
constexpr int kPvBf16x3 = 0;   // default: bf16 MFMA 16x16x16 three times, p as three bf16 parts (24 significant bits)
constexpr int kPvFp32 = 1;     // fp32 MFMA 16x16x4, p exact; 4x the matrix-core time, measurably slower
constexpr int kPvBf16 = 2;     // bf16 MFMA 16x16x16 once, p rounded to bf16; same speed as the default, less exact
constexpr int kPvBf16x3Apart = 3;      // internal, below 4 rows per KV head: as 0, and infinite values keep their sums

// Inner-loop choice: automatic = matrix path (see use_matrix_path); kPathMatrix also opens the weight modes to
// calls below 4 rows per KV head.
constexpr int kPathAuto = 0;
constexpr int kPathVector = 1;
constexpr int kPathMatrix = 2;

bool use_matrix_path(int path);

// Query rows one wave handles for a KV head with rows_total = group * q_len rows; more rows than that
// make row groups, workgroups that read the same pieces.
int rows_per_wave(int rows_total, int path);

// Enqueues the split-KV decode kernel and the merge kernel on `stream`.  If `events` is not null it
// holds three events, recorded before the decode kernel, between the kernels and after the merge.
hipError_t launch_decode(const DecodeParams& prm, hipStream_t stream, hipEvent_t* events);

// Waves per output row of the merge kernels: as many as keep the launch within what the chip holds at once
// (256 compute units of 32 waves).  Few rows mean few sequences, whose keys may be split into hundreds of
// slots; rows of up to kMergeAlone slots are summed by their first wave alone whatever this says.
constexpr int kMergeAlone = 8;
constexpr int merge_waves(long rows) { return rows <= 512 ? 16 : rows <= 2048 ? 4 : 1; }

// Whose partial rows an XCD reads.  From 8 sequences on it merges the x-th eighth of the output rows, as the decode kernels
// give it the x-th eighth of the token stream (kReadOwn): where the lengths are about even, most partial rows are then read through
// the L2 that they were written through.  (Round robin: 31 sequences of 41 to 666 tokens, 8 KV heads, 32 rows 26.2 -> 27.7 us;
// latent-KV, 128 rows 27.8 -> 29.5, 128 of 244 to 1958 71.3 -> 73.4; large GQA calls level.)  Where they are not, an XCD would be left
// with most of the work: the workgroups then turn to the rows round robin themselves (see spread_rows).  With fewer sequences than
// XCDs a long one's rows would all meet on one of them (latent-KV, 7 of 2216 to 17728, 72 rows 37.0 -> 37.8): always round robin.
// Those rows come from all XCDs, through the L2 (kReadFar) or past it (kReadFarOnce).
constexpr int kReadOwn = 0, kReadFar = 1, kReadFarOnce = 2;
// Workgroups of a merge kernel whose work is `n` of them in the order of the output rows: a multiple of the eight XCDs.
inline unsigned merge_grid(long n) { return (unsigned)((n + 7) / 8 * 8); }
// Returns launch(waves per row, kRead..., workgroups), the first two as types.  Of few sequences' rows, fewer than kCachedBelow are
// read through the L2s.
template <int kCachedBelow, typename Launch>
inline hipError_t launch_merge(long rows, int batch, Launch launch) {
    auto with_waves = [&](auto read) {
        switch (merge_waves(rows)) {
            case 16: return launch(std::integral_constant<int, 16>(), read, merge_grid(rows));
            case 4: return launch(std::integral_constant<int, 4>(), read, merge_grid(rows));
            default: return launch(std::integral_constant<int, 1>(), read, merge_grid((rows + 3) / 4));
        }
    };
    if (batch >= 8) return with_waves(std::integral_constant<int, kReadOwn>());
    if constexpr (kCachedBelow > 0) {
        static_assert(merge_waves(kCachedBelow) == 16, "one form of the kernel");
        if (rows < kCachedBelow) return launch(std::integral_constant<int, 16>(), std::integral_constant<int, kReadFar>(), merge_grid(rows));
    }
    return with_waves(std::integral_constant<int, kReadFarOnce>());
}

// Latent-KV (MLA-shaped) decode: every head reads the same cached row of 576 bf16 per token.
struct MlaParams {
    const uint16_t* q;               // bf16 [batch, q_len, n_heads, 576]
    const void* const* c_ptrs;       // device array[batch] of device pointers: bf16 [kv_len, 576]
    const int32_t* kv_lens;
    int batch, q_len, n_heads;
    float scale_log2;
    uint16_t* out;                   // bf16 [batch, q_len, n_heads, 512]
    float* lse;                      // fp32 [batch, q_len, n_heads] or null
    uint16_t* part_o;                // fp16 [slots, q_len * n_heads, 512]: partial rows, each times its own scale
    float* part_ml;                  // fp32 [slots, q_len * n_heads, 4]: (max, sum, sum of rounded weights, 1 / scale)
    int32_t* meta;                   // int32 [batch, 2]
    int n_pieces, min_piece_tokens;
    FewPieces few;
    int xcd_skew;                    // as in DecodeParams
    int layout;                      // 0 automatic, 1 one 16-row tile per wave, 2 32-row tiles from 65 rows on
    int weight_mode;                 // softmax weights in the value product: 0 default (hi + lo bf16 parts where a key
                                     // dominates, one bf16 elsewhere), 1 hi + lo everywhere, 2 one bf16 everywhere
};
void mla_block_shape(int rows_total, int layout, int* waves, int* tiles_per_wave);
// Enqueues the decode kernel and its merge kernel; events as for launch_decode.
hipError_t launch_mla_decode(const MlaParams& prm, hipStream_t stream, hipEvent_t* events);

// Appends q_len new K/V rows per sequence at rows [kv_lens[b] - q_len, kv_lens[b]).
struct WriteParams {
    const uint16_t* k_new;           // bf16 [batch, q_len, row_elems]
    const uint16_t* v_new;
    void* const* k_ptrs;
    void* const* v_ptrs;
    const int32_t* kv_lens;
    int batch, q_len;
    int row_bytes;                   // n_kv_heads * head_dim * 2
};
hipError_t launch_write_kvcache(const WriteParams& prm, hipStream_t stream);

}  // namespace xattn
#endif
