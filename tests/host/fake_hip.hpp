// A stand-in for the HIP runtime that lets the host code of libcrp.so run on the
// CPU: device memory is host memory, kernels are not run but handed to a hook, and
// copies from pinned memory take place when the stream is waited for (as late as
// the runtime may make them).  The definitions here come before those of
// libamdhip64 for everything that libcrp.so calls.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <string>
#include <vector>

namespace fake {

struct Copy {
    void* dst;
    const void* src;
    size_t bytes;
};
inline std::vector<Copy> pending;                    // copies from pinned memory not yet made
inline std::map<const char*, size_t> pinned;
inline hipError_t last = hipSuccess;
inline std::string fail_kernel;                      // launches of this kernel fail
inline float elapsed_ms = 1.0f;
inline int cus = 256;
// called for every launch: name, blocks, threads, arguments
inline std::function<void(const std::string&, dim3, dim3, void**)> on_launch;

// Filled while the library is loaded, before the globals above exist.
inline std::map<const void*, std::string>& kernels()      // host stub -> kernel name
{
    static std::map<const void*, std::string> m;
    return m;
}
inline std::map<const void*, size_t>& variables()         // host symbol -> bytes
{
    static std::map<const void*, size_t> m;
    return m;
}

inline void finish()
{
    for (const Copy& c : pending)
        std::memcpy(c.dst, c.src, c.bytes);
    pending.clear();
}

inline bool is_pinned(const void* p)
{
    for (const auto& m : pinned)
        if ((const char*)p >= m.first && (const char*)p < m.first + m.second)
            return true;
    return false;
}

inline hipError_t set(hipError_t e)
{
    if (e != hipSuccess)
        last = e;
    return e;
}

struct Config {
    dim3 grid, block;
    size_t shared;
    hipStream_t stream;
};
inline std::vector<Config> configs;

}  // namespace fake

extern "C" {

void** __hipRegisterFatBinary(const void*)
{
    static void* handle;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*,
                           void*, void*, void*, int*)
{
    fake::kernels()[host] = name;
}
void __hipRegisterVar(void**, void* var, char*, char*, int, size_t size, int, int)
{
    fake::variables()[var] = size;
}
hipError_t hipGetSymbolAddress(void** p, const void* symbol)
{
    *p = std::calloc(1, fake::variables().at(symbol));
    return hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t sh, hipStream_t s)
{
    fake::configs.push_back({g, b, sh, s});
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* sh, hipStream_t* s)
{
    const fake::Config c = fake::configs.back();
    fake::configs.pop_back();
    *g = c.grid;
    *b = c.block;
    *sh = c.shared;
    *s = c.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t, hipStream_t)
{
    const std::string& name = fake::kernels()[f];
    if (!fake::fail_kernel.empty() && name.find(fake::fail_kernel) != std::string::npos)
        return fake::set(hipErrorLaunchFailure);
    if (g.x == 0 || g.y == 0 || g.z == 0)
        return fake::set(hipErrorInvalidConfiguration);
    if (fake::on_launch)
        fake::on_launch(name, g, b, args);
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int block, size_t)
{
    *n = 512 / block;      // eight waves per compute unit
    return hipSuccess;
}

hipError_t hipMalloc(void** p, size_t n)
{
    *p = std::calloc(1, n ? n : 1);
    return *p ? hipSuccess : fake::set(hipErrorOutOfMemory);
}
hipError_t hipFree(void* p)
{
    fake::finish();
    std::free(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned)
{
    *p = std::calloc(1, n);
    fake::pinned[(const char*)*p] = n;
    return hipSuccess;
}
hipError_t hipHostFree(void* p)
{
    fake::finish();
    fake::pinned.erase((const char*)p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t)
{
    if (fake::is_pinned(s)) {
        fake::pending.push_back({d, s, n});
        return hipSuccess;
    }
    fake::finish();
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind)
{
    fake::finish();
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t)
{
    fake::finish();
    std::memset(d, v, n);
    return hipSuccess;
}
hipError_t hipMemset(void* d, int v, size_t n) { return hipMemsetAsync(d, v, n, nullptr); }
hipError_t hipStreamSynchronize(hipStream_t)
{
    fake::finish();
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipStreamSynchronize(nullptr); }

hipError_t hipEventCreate(hipEvent_t* e)
{
    *e = (hipEvent_t)std::calloc(1, 8);
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e)
{
    std::free((void*)e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipStreamSynchronize(nullptr); }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t)
{
    *ms = fake::elapsed_ms;
    return hipSuccess;
}

hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDevice(int* d)
{
    *d = 0;
    return hipSuccess;
}
int hipGetStreamDeviceId(hipStream_t) { return 0; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int)
{
    *v = a == hipDeviceAttributeWarpSize ? 64 : fake::cus;
    return hipSuccess;
}
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int)
{
    std::memset(p, 0, sizeof *p);
    p->multiProcessorCount = fake::cus;
    p->warpSize = 64;
    std::strcpy(p->gcnArchName, "gfx950");
    return hipSuccess;
}
hipError_t hipGetLastError()
{
    const hipError_t e = fake::last;
    fake::last = hipSuccess;
    return e;
}
const char* hipGetErrorString(hipError_t) { return "fake error"; }

}  // extern "C"
