// Kernel launches (csrc/xattn_launch.h) on a stand-in for the HIP runtime with two devices: what a failed launch leaves
// behind, and whose function a stream gets.  As in the real runtime a failed call stays recorded until hipGetLastError takes it.  Prints "all
// scenarios ran" and exits with 0 if every check held.
#include <cstdint>
#include <cstdio>
#include <cstdlib>

#include "../../paper_2510_14686_amd/csrc/xattn_launch.h"

static hipError_t g_recorded = hipSuccess;      // the runtime's last error
static int g_device = 0;                        // the current device
static hipError_t g_device_fails = hipSuccess, g_lookup_fails = hipSuccess, g_launch_fails = hipSuccess;
static int g_launches = 0;
static uintptr_t g_launched = 0;                // the function of the last launch: kernel + 1 + its device
static int g_first, g_second;                   // the arguments of the last launch
static hipError_t record(hipError_t e) {
    if (e != hipSuccess) g_recorded = e;
    return e;
}

extern "C" {
hipError_t hipGetDevice(int* d) { *d = g_device; return record(g_device_fails); }
hipError_t hipSetDevice(int d) { g_device = d; return hipSuccess; }
// A stream is its device in the upper half; of the runtime's own handles (0, 1, 2) it is not asked.
hipError_t hipStreamGetDevice(hipStream_t s, int* d) {
    const uintptr_t handle = reinterpret_cast<uintptr_t>(s);
    if (handle <= 2) std::abort();
    *d = (int)(handle >> 32);
    return *d < 2 ? hipSuccess : record(hipErrorInvalidHandle);
}
hipError_t hipGetLastError() { const hipError_t e = g_recorded; g_recorded = hipSuccess; return e; }
hipError_t hipGetFuncBySymbol(hipFunction_t* f, const void* kernel) {
    if (g_lookup_fails != hipSuccess) return record(g_lookup_fails);
    *f = reinterpret_cast<hipFunction_t>(reinterpret_cast<uintptr_t>(kernel) + 1 + g_device);
    return hipSuccess;
}
hipError_t hipModuleLaunchKernel(hipFunction_t f, unsigned, unsigned, unsigned, unsigned, unsigned, unsigned, unsigned, hipStream_t,
                                 void**, void** extra) {
    if (g_launch_fails != hipSuccess) return record(g_launch_fails);
    ++g_launches;
    g_launched = reinterpret_cast<uintptr_t>(f);
    g_first = static_cast<const int*>(extra[1])[0];
    g_second = static_cast<const int*>(extra[1])[1];
    return hipSuccess;
}
}

static void kernel_a(int, int) {}
static void kernel_b(int, int) {}
static void kernel_c(int, int) {}

static int g_failures = 0;
#define CHECK(cond)                                                              \
    do {                                                                         \
        if (!(cond)) {                                                           \
            std::fprintf(stderr, "CHECK failed at line %d: %s\n", __LINE__, #cond); \
            ++g_failures;                                                        \
        }                                                                        \
    } while (0)

template <typename Kernel>
static hipError_t go(Kernel kernel, hipStream_t stream = nullptr) { return xattn::launch(kernel, dim3(3), 64, stream, 5, 7); }

// A launch that fails, wherever, reports it once: the thread's next check of its own work finds nothing.
static void a_failed_launch_leaves_nothing_recorded() {
    g_launch_fails = hipErrorInvalidConfiguration;
    CHECK(go(kernel_a) == hipErrorInvalidConfiguration && hipGetLastError() == hipSuccess);
    g_launch_fails = hipSuccess;
    g_lookup_fails = hipErrorInvalidDeviceFunction;
    CHECK(go(kernel_c) == hipErrorInvalidDeviceFunction && hipGetLastError() == hipSuccess);
    g_lookup_fails = hipSuccess;
    g_device_fails = hipErrorNoDevice;
    CHECK(go(kernel_a) == hipErrorNoDevice && hipGetLastError() == hipSuccess);
    g_device_fails = hipSuccess;
    CHECK(g_launches == 0);
    CHECK(go(kernel_a) == hipSuccess && go(kernel_b) == hipSuccess && g_launches == 2 && g_first == 5 && g_second == 7);
}

// A stream's launches use the function of the stream's device, whichever is current, and leave the current one alone.
static hipStream_t stream_of(int device) { return reinterpret_cast<hipStream_t>((uintptr_t)device << 32 | 0x1000u); }
template <typename Kernel>
static uintptr_t function_of(Kernel kernel, int device) { return reinterpret_cast<uintptr_t>(kernel) + 1 + device; }
static void a_stream_gets_its_own_devices_function() {
    for (int pass = 0; pass < 2; ++pass)                   // looked up, and from the table
        for (int current = 0; current < 2; ++current) {
            g_device = current;
            for (int device = 0; device < 2; ++device) {
                CHECK(go(kernel_a, stream_of(device)) == hipSuccess && g_launched == function_of(kernel_a, device) && g_device == current);
                CHECK(go(kernel_b, stream_of(device)) == hipSuccess && g_launched == function_of(kernel_b, device) && g_device == current);
            }
            for (uintptr_t handle = 0; handle <= 2; ++handle)      // the default streams: of the current device
                CHECK(go(kernel_a, reinterpret_cast<hipStream_t>(handle)) == hipSuccess && g_launched == function_of(kernel_a, current));
        }
    g_device = 0;
    g_lookup_fails = hipErrorInvalidDeviceFunction;
    CHECK(go(kernel_c, stream_of(1)) == hipErrorInvalidDeviceFunction && g_device == 0 && hipGetLastError() == hipSuccess);
    g_lookup_fails = hipSuccess;
    const int before = g_launches;
    CHECK(go(kernel_a, stream_of(5)) == hipErrorInvalidHandle && g_launches == before && hipGetLastError() == hipSuccess);
}

int main() {
    a_stream_gets_its_own_devices_function();
    g_launches = 0;
    a_failed_launch_leaves_nothing_recorded();
    if (g_failures) return 1;
    std::puts("all scenarios ran");
    return 0;
}
