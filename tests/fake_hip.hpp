// A HIP runtime for host tests: device memory is host memory, streams and
// events do nothing, and allocations can be made to fail.  A test program
// includes the library's host sources after this and defines the launches.
#pragma once

#include <hip/hip_runtime.h>

#include <atomic>
#include <chrono>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <thread>

#define __align__(n) __attribute__((aligned(n)))
#define HIP_SYMBOL(x) (x)

namespace fake {
inline long fail_in = -1;      // >= 0: allocations left before one fails
inline bool refuse() { return fail_in >= 0 && fail_in-- == 0; }
inline hipError_t alloc(void **p, size_t n) {
    if (refuse()) { *p = nullptr; return hipErrorOutOfMemory; }
    *p = std::malloc(n ? n : 1);
    return hipSuccess;
}
// Work that a stream still does after a call returned: the stream is busy until
// it has run (`late` of 5: it never runs, and the stream is idle).
inline int late = 0;
inline std::thread worker;
inline std::atomic<bool> busy{false};
inline void join() { if (worker.joinable()) worker.join(); }
inline void later(std::function<void()> work) {
    join();
    busy = true;
    worker = std::thread([work] {
        std::this_thread::sleep_for(std::chrono::milliseconds(3));
        work();
        busy = false;
    });
}
}  // namespace fake

extern "C" {
hipError_t hipMalloc(void **p, size_t n) { return fake::alloc(p, n); }
hipError_t hipFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return fake::alloc(p, n); }
hipError_t hipHostFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int) {
    *v = a == hipDeviceAttributeMultiprocessorCount ? 2 : 160 << 10;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **p, const void *s) { *p = const_cast<void *>(s); return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t e) { return e == hipSuccess ? "no error" : "error"; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) {
    *s = static_cast<hipStream_t>(std::malloc(1));
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s) { std::free(s); return hipSuccess; }
hipError_t hipStreamQuery(hipStream_t) { return fake::busy ? hipErrorNotReady : hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { fake::join(); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = nullptr; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 0.0f; return hipSuccess; }
}
