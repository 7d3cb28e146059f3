// Kernel launches of libxattn.so (host code).
#ifndef XATTN_LAUNCH_H_
#define XATTN_LAUNCH_H_

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <type_traits>

namespace xattn {

// A short call is bound by the host's two launches, so a kernel's function is looked up once per thread and device, and its
// arguments go to the runtime as one packed buffer, laid out as the kernel takes them: two launches of 12 and 7 arguments 6.7 -> 6.35 us.
// The function is the one of the stream's device, which need not be the current one.
inline hipError_t look_up(const void* kernel, int dev, hipFunction_t* f) {
    int current = 0;
    hipError_t e = hipGetDevice(&current);
    if (e != hipSuccess || dev == current) return e != hipSuccess ? e : hipGetFuncBySymbol(f, kernel);
    if ((e = hipSetDevice(dev)) != hipSuccess) return e;
    e = hipGetFuncBySymbol(f, kernel);
    const hipError_t back = hipSetDevice(current);
    return e != hipSuccess ? e : back;
}
inline hipError_t function_for(const void* kernel, hipStream_t stream, hipFunction_t* f) {
    struct Entry {
        const void* kernel;
        int dev;
        hipFunction_t f;
    };
    static thread_local Entry table[64] = {};
    int dev = 0;
    const bool own = stream != nullptr && stream != hipStreamLegacy && stream != hipStreamPerThread;
    hipError_t e = own ? hipStreamGetDevice(stream, &dev) : hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uintptr_t k = reinterpret_cast<uintptr_t>(kernel);
    Entry& t = table[(k >> 3 ^ k >> 9 ^ (uintptr_t)dev) & 63];
    if (t.kernel != kernel || t.dev != dev) {
        hipFunction_t found;
        if ((e = look_up(kernel, dev, &found)) != hipSuccess) return e;
        t = Entry{kernel, dev, found};
    }
    *f = t.f;
    return hipSuccess;
}

// An error that the call returns is taken back from the runtime: the thread's next check of other work must not find it.
inline hipError_t taken_back(hipError_t e) {
    if (e != hipSuccess) (void)hipGetLastError();
    return e;
}

template <typename... P, typename... A>
hipError_t launch(void (*kernel)(P...), dim3 grid, int threads, hipStream_t stream, const A&... args) {
    static_assert(sizeof...(P) == sizeof...(A), "one value per parameter");
    hipFunction_t f;
    const hipError_t e = function_for(reinterpret_cast<const void*>(kernel), stream, &f);
    if (e != hipSuccess) return taken_back(e);
    alignas(16) char buffer[(0 + ... + (sizeof(P) + alignof(P)))];
    size_t bytes = 0;
    auto put = [&](const auto& value) {
        constexpr size_t align = alignof(std::decay_t<decltype(value)>);
        bytes = (bytes + align - 1) / align * align;
        memcpy(buffer + bytes, &value, sizeof value);
        bytes += sizeof value;
    };
    (put(static_cast<P>(args)), ...);
    void* extra[] = {HIP_LAUNCH_PARAM_BUFFER_POINTER, buffer, HIP_LAUNCH_PARAM_BUFFER_SIZE, &bytes, HIP_LAUNCH_PARAM_END};
    return taken_back(hipModuleLaunchKernel(f, grid.x, grid.y, grid.z, (unsigned)threads, 1, 1, 0, stream, nullptr, extra));
}

}  // namespace xattn
#endif
