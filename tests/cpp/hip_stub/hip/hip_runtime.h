// The few HIP runtime calls of streams.hpp and pinned.hpp, on the host, with
// errors on demand (for drain_check.cpp).
#pragma once
#include <cstdlib>

typedef void* hipStream_t;
typedef void* hipEvent_t;
enum hipError_t { hipSuccess = 0, hipErrorUnknown = 999 };
enum { hipStreamNonBlocking = 1, hipEventDisableTiming = 2, hipHostMallocPortable = 1 };

inline hipError_t stub_sync_result = hipSuccess;
inline int stub_syncs = 0;
inline void (*stub_on_sync)() = nullptr;

inline hipError_t hipStreamSynchronize(hipStream_t) {
    ++stub_syncs;
    if (stub_on_sync) stub_on_sync();
    return stub_sync_result;
}
inline hipError_t hipHostMalloc(void** p, std::size_t n, unsigned) {
    *p = std::malloc(n);
    return *p ? hipSuccess : hipErrorUnknown;
}
inline hipError_t hipHostFree(void* p) {
    std::free(p);
    return hipSuccess;
}
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
inline hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    *s = std::malloc(1);
    return hipSuccess;
}
inline hipError_t hipStreamDestroy(hipStream_t s) {
    std::free(s);
    return hipSuccess;
}
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    *e = std::malloc(1);
    return hipSuccess;
}
inline hipError_t hipEventDestroy(hipEvent_t e) {
    std::free(e);
    return hipSuccess;
}
