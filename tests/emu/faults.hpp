// Included ahead of the library's sources (-include) in the build of
// tests/emu/faults.cpp: allocations and copies that fail when they are told to, and a count
// of what has been queued on a stream since a host thread last waited for it
// (the emulation itself runs everything at once).
#pragma once
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

struct EmuFaults {
    long mallocs = -1, pinned = -1;  // that many more succeed, the rest fail; < 0: all do
    long copies_left = -1;           // likewise, of the copies
    long failed = 0;                 // allocations and copies that failed
    long queued = 0;                 // copies and launches not waited for
    long copies = 0;                 // copies queued
    bool news = false;               // operator new fails
    bool news_after_wait = false;    // from the next wait for a stream on
    long most = -1;                  // device allocations at most, if >= 0
    long live = 0;                   // device allocations not freed
};
inline EmuFaults emu_faults;

inline bool emu_fails(long& left) {
    if (left < 0) return false;
    if (left > 0) {
        --left;
        return false;
    }
    ++emu_faults.failed;
    return true;
}
inline hipError_t emu_hipMalloc(void** p, size_t n) {
    const bool full = emu_faults.most >= 0 && emu_faults.live >= emu_faults.most;
    if (full || emu_fails(emu_faults.mallocs)) {
        *p = nullptr;
        return hipErrorOutOfMemory;
    }
    ++emu_faults.live;
    return hipMalloc(p, n);
}
inline hipError_t emu_hipFree(void* p) {
    emu_faults.live -= p != nullptr;
    return hipFree(p);
}
inline hipError_t emu_hipHostMalloc(void** p, size_t n, unsigned flags) {
    if (emu_fails(emu_faults.pinned)) {
        *p = nullptr;
        return hipErrorOutOfMemory;
    }
    return hipHostMalloc(p, n, flags);
}
inline hipError_t emu_hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t t) {
    if (emu_fails(emu_faults.copies_left)) return hipErrorInvalidValue;
    ++emu_faults.queued;
    ++emu_faults.copies;
    return hipMemcpyAsync(d, s, n, k, t);
}
inline hipError_t emu_hipStreamSynchronize(hipStream_t s) {
    emu_faults.queued = 0;
    if (emu_faults.news_after_wait) emu_faults.news = true;
    return hipStreamSynchronize(s);
}
inline hipError_t emu_hipDeviceSynchronize() {
    emu_faults.queued = 0;
    return hipDeviceSynchronize();
}
inline hipError_t emu_hipEventSynchronize(hipEvent_t e) {
    emu_faults.queued = 0;  // every event is recorded behind all of the call's work
    return hipEventSynchronize(e);
}
#define hipMalloc emu_hipMalloc
#define hipFree emu_hipFree
#define hipHostMalloc emu_hipHostMalloc
#define hipMemcpyAsync emu_hipMemcpyAsync
#define hipStreamSynchronize emu_hipStreamSynchronize
#define hipDeviceSynchronize emu_hipDeviceSynchronize
#define hipEventSynchronize emu_hipEventSynchronize
#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(k, g, b, sh, st, ...) \
    (++emu_faults.queued, emu_launch(k, dim3(g), dim3(b), __VA_ARGS__))
#undef hipExtLaunchKernelGGL
#define hipExtLaunchKernelGGL(k, g, b, sh, st, e0, e1, fl, ...) \
    hipLaunchKernelGGL(k, g, b, sh, st, __VA_ARGS__)
