// A stand-in for the HIP runtime that libhashgraph.so calls, for checks of its
// host paths on a machine without a GPU.  A program that includes this file and
// links the library with -rdynamic takes the runtime's place: its definitions come
// first in the symbol search.  Memory is only counted (pointers are never
// followed), kernels are not run, copies to the host give zeros.
#pragma once

#include <hip/hip_runtime.h>
#include <string.h>

#include <map>

namespace fake {

struct Block {
    size_t bytes;
    bool pooled;
};

struct State {
    std::map<void*, Block> live;
    uintptr_t next = 1ull << 40;
    size_t used = 0;             // bytes of live blocks
    size_t kept = 0;             // freed bytes that the pool still holds
    size_t capacity = ~(size_t)0;
    long allocs = 0;             // allocation calls that succeeded
    long fail_in = -1;           // the allocation call that many ahead fails (0: the next),
    long fail_times = 2;         // and so do those after it: that many in all (a retry too)
    long memsets = 0, memset_fail_in = -1, launches = 0, trims = 0, pools = 0;
    bool capturing = false;
};
inline State st;

inline bool fails(long& in) { return in >= 0 && in-- == 0; }

inline hipError_t alloc(void** p, size_t bytes, bool pooled) {
    if (st.fail_in == 0 && st.fail_times > 0) {
        --st.fail_times;
        return hipErrorOutOfMemory;
    }
    if (st.fail_in > 0) --st.fail_in;
    const size_t reuse = pooled ? (bytes < st.kept ? bytes : st.kept) : 0;
    if (bytes - reuse > st.capacity || st.used + st.kept > st.capacity - (bytes - reuse))
        return hipErrorOutOfMemory;
    st.kept -= reuse;
    st.used += bytes;
    *p = (void*)st.next;
    st.next += (bytes + 511) / 256 * 256;
    st.live[*p] = Block{bytes, pooled};
    ++st.allocs;
    return hipSuccess;
}

inline hipError_t release(void* p) {
    if (!p) return hipSuccess;
    auto it = st.live.find(p);
    if (it == st.live.end()) return hipErrorInvalidValue;
    st.used -= it->second.bytes;
    if (it->second.pooled) st.kept += it->second.bytes;
    st.live.erase(it);
    return hipSuccess;
}

}  // namespace fake

#define FAKE extern "C" __attribute__((visibility("default")))
FAKE hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
FAKE hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
FAKE hipError_t hipSetDevice(int) { return hipSuccess; }
FAKE hipError_t hipGetLastError() { return hipSuccess; }
FAKE hipError_t hipDeviceTotalMem(size_t* b, hipDevice_t) { *b = 288ull << 30; return hipSuccess; }
FAKE hipError_t hipDeviceSynchronize() { return hipSuccess; }
FAKE hipError_t hipMalloc(void** p, size_t b) { return fake::alloc(p, b, false); }
FAKE hipError_t hipMallocAsync(void** p, size_t b, hipStream_t) { return fake::alloc(p, b, false); }
FAKE hipError_t hipMallocFromPoolAsync(void** p, size_t b, hipMemPool_t, hipStream_t) {
    return fake::alloc(p, b, true);
}
FAKE hipError_t hipFree(void* p) { return fake::release(p); }
FAKE hipError_t hipFreeAsync(void* p, hipStream_t) { return fake::release(p); }
FAKE hipError_t hipMemPoolCreate(hipMemPool_t* p, const hipMemPoolProps*) {
    *p = (hipMemPool_t)(uintptr_t)++fake::st.pools;
    return hipSuccess;
}
FAKE hipError_t hipMemPoolDestroy(hipMemPool_t) { return hipSuccess; }
FAKE hipError_t hipMemPoolSetAttribute(hipMemPool_t, hipMemPoolAttr, void*) { return hipSuccess; }
FAKE hipError_t hipMemPoolTrimTo(hipMemPool_t, size_t) {
    ++fake::st.trims;
    fake::st.kept = 0;
    return hipSuccess;
}
FAKE hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) {
    if (fake::fails(fake::st.memset_fail_in)) return hipErrorInvalidValue;
    ++fake::st.memsets;
    return hipSuccess;
}
FAKE hipError_t hipMemcpyAsync(void* d, const void*, size_t n, hipMemcpyKind k, hipStream_t) {
    if (k == hipMemcpyDeviceToHost) memset(d, 0, n);
    return hipSuccess;
}
FAKE hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
FAKE hipError_t hipStreamGetDevice(hipStream_t, hipDevice_t* d) { *d = 0; return hipSuccess; }
FAKE hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
    *s = fake::st.capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
FAKE hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
FAKE hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) {
    ++fake::st.launches;
    return hipSuccess;
}
FAKE hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
FAKE hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* l, hipStream_t* s) {
    *g = *b = dim3(1);
    *l = 0;
    *s = nullptr;
    return hipSuccess;
}
#undef FAKE
