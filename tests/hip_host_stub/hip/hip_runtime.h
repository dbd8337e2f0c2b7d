// Host-only stand-in for <hip/hip_runtime.h> (test infrastructure): lets the
// library's host builder (api.cpp) compile with a plain C++ compiler.  Without
// SIMGPU_STUB_DEVICE there is no device: every device call fails, so a load
// runs the host expansion and stops at its first device call.  With it, device
// memory is host memory, an allocation of more than SIMGPU_STUB_ALLOC_MAX bytes
// fails (0 or unset: none does), and errors stay until hipGetLastError reads them.
#pragma once
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <cstring>

typedef int hipError_t;
typedef void *hipStream_t;
enum { hipSuccess = 0, hipErrorOutOfMemory = 2, hipErrorNoDevice = 100 };
enum hipMemcpyKind { hipMemcpyHostToDevice = 1, hipMemcpyDeviceToHost = 2 };
enum hipDeviceAttribute_t { hipDeviceAttributeMultiprocessorCount = 0 };
struct uint4 { unsigned x, y, z, w; };

inline bool stub_device() { return std::getenv("SIMGPU_STUB_DEVICE") != nullptr; }
inline hipError_t &stub_error() {
    static hipError_t e = hipSuccess;
    return e;
}
inline hipError_t stub_fail(hipError_t e) { return stub_error() = e; }

inline hipError_t hipGetDevice(int *d) {
    if (!stub_device()) return hipErrorNoDevice;
    *d = 0;
    return hipSuccess;
}
inline hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int) {
    if (!stub_device()) return hipErrorNoDevice;
    *v = 256;
    return hipSuccess;
}
inline hipError_t hipMalloc(void **p, size_t bytes) {
    *p = nullptr;
    if (!stub_device()) return hipErrorNoDevice;
    const char *ev = std::getenv("SIMGPU_STUB_ALLOC_MAX");
    const size_t most = ev ? (size_t)std::strtoull(ev, nullptr, 10) : 0;
    if (most && bytes > most) return stub_fail(hipErrorOutOfMemory);
    *p = std::malloc(bytes);
    return *p ? hipSuccess : stub_fail(hipErrorOutOfMemory);
}
inline hipError_t hipFree(void *p) {
    std::free(p);
    return hipSuccess;
}
inline hipError_t hipMemcpy(void *dst, const void *src, size_t bytes, hipMemcpyKind) {
    if (!stub_device()) return hipErrorNoDevice;
    std::memcpy(dst, src, bytes);
    return hipSuccess;
}
inline hipError_t hipGetLastError() {
    const hipError_t e = stub_error();
    stub_error() = hipSuccess;
    return e;
}
inline const char *hipGetErrorString(hipError_t) { return "stub device error (host-only build)"; }
