// The C-ABI layer (csrc/xattn_api.cpp) on a stand-in for the HIP runtime and the kernel launches: which
// workspace a call gets, how it splits the keys over it, and what a failed allocation leaves behind.
// As in the real runtime a failed call stays recorded until hipGetLastError takes it, and a launch
// reports whatever is recorded.  Prints "all scenarios ran" and exits with 0 if every check held.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <string>
#include <vector>

#include "../../include/xattn.h"
#include "../../paper_2510_14686_amd/csrc/xattn_host.h"
#include "../../paper_2510_14686_amd/csrc/xattn_kernels.h"

static hipError_t g_recorded = hipSuccess;      // the runtime's last error
static size_t g_free = (size_t)1 << 40;         // largest allocation that succeeds
static bool g_capturing = false;
static std::vector<size_t> g_allocs;            // sizes that succeeded
static int g_refused = 0;
static hipError_t record(hipError_t e) {
    if (e != hipSuccess) g_recorded = e;
    return e;
}

extern "C" {
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipMalloc(void** p, size_t bytes) {
    if (bytes > g_free) { ++g_refused; return record(hipErrorOutOfMemory); }
    g_allocs.push_back(bytes);
    *p = reinterpret_cast<void*>((uintptr_t)(g_allocs.size() << 44));      // never dereferenced
    return hipSuccess;
}
hipError_t hipGetLastError() { const hipError_t e = g_recorded; g_recorded = hipSuccess; return e; }
const char* hipGetErrorString(hipError_t) { return "stand-in error"; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
    *s = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t*) { return record(hipErrorUnknown); }
hipError_t hipEventSynchronize(hipEvent_t) { return record(hipErrorUnknown); }
hipError_t hipEventElapsedTime(float*, hipEvent_t, hipEvent_t) { return record(hipErrorUnknown); }
hipError_t hipMemcpy(void*, const void*, size_t, hipMemcpyKind) { return record(hipErrorUnknown); }
}

namespace xattn {
// What the last call launched.
static int g_decodes = 0, g_merges = 0;
static DecodeParams g_prm;
static MlaParams g_mla;

bool use_matrix_path(int path) { return path != kPathVector; }
int rows_per_wave(int rows_total, int) { return rows_total <= 16 ? 16 : 32; }
void mla_block_shape(int, int, int* waves, int* tiles) { *waves = 8; *tiles = 1; }
static hipError_t launch() {
    ++g_decodes;
    const hipError_t e = hipGetLastError();
    if (e == hipSuccess) ++g_merges;
    return e;
}
hipError_t launch_decode(const DecodeParams& prm, hipStream_t, hipEvent_t*) { g_prm = prm; return launch(); }
hipError_t launch_mla_decode(const MlaParams& prm, hipStream_t, hipEvent_t*) { g_mla = prm; return launch(); }
hipError_t launch_write_kvcache(const WriteParams&, hipStream_t) { return hipGetLastError(); }
}  // namespace xattn

static int g_failures = 0;
#define CHECK(cond)                                                                                        \
    do {                                                                                                   \
        if (!(cond)) {                                                                                     \
            std::fprintf(stderr, "CHECK failed at line %d: %s (%s)\n", __LINE__, #cond, xattn_last_error()); \
            ++g_failures;                                                                                  \
        }                                                                                                  \
    } while (0)

static const uintptr_t kMiB = (uintptr_t)1 << 20;

static int decode(intptr_t stream, int batch, int q_len, int hq, int hkv) {
    static int dummy __attribute__((aligned(16)));
    return xattn_decode(&dummy, reinterpret_cast<void**>(&dummy), reinterpret_cast<void**>(&dummy), &dummy, batch, q_len, hq, hkv,
                        128, 0.125f, &dummy, nullptr, reinterpret_cast<void*>(stream));
}
static int mla_decode(intptr_t stream, int batch, int q_len, int heads) {
    static int dummy __attribute__((aligned(16)));
    return xattn_mla_decode(&dummy, reinterpret_cast<void**>(&dummy), &dummy, batch, q_len, heads, 512, 64, 0.125f, &dummy, nullptr,
                            reinterpret_cast<void*>(stream));
}
// The last launch's slots, of either path, lie within `bytes` bytes from its table on.
static bool fits(size_t bytes) {
    const xattn::DecodeParams& p = xattn::g_prm;
    const size_t slots = (size_t)p.n_pieces + p.batch, rows = (size_t)p.q_len * p.n_q_heads;
    const char* base = reinterpret_cast<const char*>(p.meta);
    return p.shared_pieces <= p.n_pieces && reinterpret_cast<const char*>(p.part_ml) >= base + 8 * (size_t)p.batch &&
           reinterpret_cast<const char*>(p.part_o) >= reinterpret_cast<const char*>(p.part_ml) + slots * rows * 8 &&
           reinterpret_cast<const char*>(p.part_o) + slots * rows * 512 <= base + bytes;
}

template <typename Fn>
static bool fail_text_stays(Fn fn) {
    const std::string before = xattn_last_error();
    fn();
    return before == xattn_last_error();
}

// A call whose allocation fails reports it and leaves nothing recorded: the next call works.
static void a_failed_allocation_fails_one_call() {
    g_free = 0;
    const int before = xattn::g_decodes;
    CHECK(decode(1, 4, 1, 8, 8) == XATTN_ENOMEM);
    CHECK(mla_decode(1, 4, 1, 16) == XATTN_ENOMEM);
    CHECK(xattn::g_decodes == before);                     // nothing was enqueued
    g_free = (size_t)1 << 40;
    CHECK(decode(1, 4, 1, 8, 8) == XATTN_OK);
    CHECK(xattn::g_merges == xattn::g_decodes);
}

// Few KV heads: the split over several pieces per workgroup wants more than one piece per compute unit
// needs.  Where only the latter can be allocated the call runs on that.
static void a_call_runs_on_what_can_be_allocated() {
    g_free = 4 * kMiB;
    const int before = xattn::g_merges;
    for (int i = 0; i < 3; ++i) {
        CHECK(decode(2, 64, 1, 8, 2) == XATTN_OK);         // 320 slots of 8 rows: 1.3 MiB; four pieces per workgroup: 4.5
        CHECK(xattn::g_prm.parts == 1 && xattn::g_prm.n_pieces == 256);
        CHECK(g_allocs.back() <= 4 * kMiB && fits(g_allocs.back()));
    }
    CHECK(xattn::g_merges == before + 3);                  // both kernels of every call
    g_free = (size_t)1 << 40;
}

// The split of a call follows from its shape alone on the library's workspaces: whatever ran on the stream
// before, eager or captured, and the same as in xattn_decode_noalloc's fixed array.
static size_t g_fixed_asked;
static int fixed_workspace(const char*, int, size_t bytes, char** ws) {
    g_fixed_asked = bytes;
    *ws = reinterpret_cast<char*>((uintptr_t)1 << 60);
    return XATTN_OK;
}
static void the_split_does_not_depend_on_earlier_calls() {
    static int dummy __attribute__((aligned(16)));
    void** const ptrs = reinterpret_cast<void**>(&dummy);
    CHECK(xattn::decode_call("noalloc", fixed_workspace, &dummy, ptrs, ptrs, &dummy, 64, 1, 8, 2, 128, 0.125f, &dummy, nullptr, nullptr) == XATTN_OK);
    const int pieces = xattn::g_prm.n_pieces, parts = xattn::g_prm.parts;
    CHECK(parts == 4 && pieces == 1024 && fits(XATTN_NOALLOC_SCRATCH_BYTES));
    CHECK(fail_text_stays([&] {
        // first call of a stream; a latent-KV call, a small call or a large one before it; captured or not
        for (int first = 0; first < 4; ++first)
            for (int captured = 0; captured < (first == 0 ? 1 : 2); ++captured) {
                const intptr_t stream = 100 + 2 * first + captured;
                if (first == 1) CHECK(mla_decode(stream, 1, 1, 1) == XATTN_OK);
                if (first == 2) CHECK(decode(stream, 1, 1, 8, 8) == XATTN_OK);
                if (first == 3) CHECK(decode(stream, 512, 8, 64, 8) == XATTN_OK);
                const size_t allocs = g_allocs.size();
                g_capturing = captured != 0;
                CHECK(decode(stream, 64, 1, 8, 2) == XATTN_OK);
                g_capturing = false;
                CHECK(xattn::g_prm.parts == parts && xattn::g_prm.n_pieces == pieces);
                CHECK(!captured || g_allocs.size() == allocs);
                CHECK(fits(g_allocs.back()));
            }
    }));
    // a stream without a workspace: a capture cannot make one, and records nothing
    g_capturing = true;
    const int before = xattn::g_decodes;
    CHECK(decode(200, 64, 1, 8, 2) == XATTN_ENOMEM);
    CHECK(mla_decode(200, 64, 1, 16) == XATTN_ENOMEM);
    CHECK(xattn::g_decodes == before);
    g_capturing = false;
    // nor can it enlarge one
    CHECK(decode(201, 1, 1, 8, 8) == XATTN_OK);
    g_capturing = true;
    CHECK(decode(201, 4096, 8, 64, 8) == XATTN_ENOMEM);
    g_capturing = false;
}

// A caller's workspace: anything from one piece per compute unit on is used, as far as it goes, and a call that
// succeeds leaves the last failure's message alone.
static void a_caller_workspace_is_used_as_far_as_it_goes() {
    const int shapes[][4] = {{64, 1, 8, 2}, {7, 2, 5, 1}, {30, 16, 12, 3}, {200, 1, 32, 8}, {3, 4, 64, 4}};
    for (const auto& s : shapes) {
        CHECK(xattn_configure(XATTN_CFG_PIECES, 256) == XATTN_OK);
        const size_t least = xattn_workspace_bytes(s[0], s[1], s[2], s[3], 128);
        CHECK(xattn_configure(XATTN_CFG_PIECES, 0) == XATTN_OK);
        const size_t most = xattn_workspace_bytes(s[0], s[1], s[2], s[3], 128);
        CHECK(least <= most);
        int last_parts = 0;
        for (int step = 0; step <= 8; ++step) {
            const size_t bytes = least + (most - least) / 8 * step + (step == 8 ? (most - least) % 8 : 0);
            CHECK(xattn_set_workspace(reinterpret_cast<void*>((uintptr_t)1 << 61), bytes) == XATTN_OK);
            CHECK(fail_text_stays([&] { CHECK(decode(1, s[0], s[1], s[2], s[3]) == XATTN_OK); }));
            CHECK(fits(bytes) && xattn::g_prm.parts >= last_parts);
            last_parts = xattn::g_prm.parts;
        }
        CHECK(xattn_set_workspace(reinterpret_cast<void*>((uintptr_t)1 << 61), least - 1) == XATTN_OK);
        CHECK(decode(1, s[0], s[1], s[2], s[3]) == XATTN_ENOMEM);
        CHECK(xattn_set_workspace(nullptr, 0) == XATTN_OK);
        CHECK(decode(1, s[0], s[1], s[2], s[3]) == XATTN_OK);
        CHECK(xattn::g_prm.parts == last_parts);           // xattn_workspace_bytes is enough for the library's split
    }
}

int main() {
    a_failed_allocation_fails_one_call();
    a_call_runs_on_what_can_be_allocated();
    the_split_does_not_depend_on_earlier_calls();
    a_caller_workspace_is_used_as_far_as_it_goes();
    CHECK(g_recorded == hipSuccess);
    if (g_failures) return 1;
    std::puts("all scenarios ran");
    return 0;
}
