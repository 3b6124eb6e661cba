// A HIP runtime for host-side checks of the library (no GPU use): a program that includes this and links libbubbly.so
// answers the library's runtime calls itself.  Device memory is host memory that no kernel ever touches, allocations
// are counted and can be bounded, launches are recorded by kernel name and not run.
#pragma once

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include <hip/hip_runtime_api.h>

struct FakeLaunch {
    std::string name;
    dim3 grid, block;
};

struct FakeHip {
    std::map<void *, size_t> mem;                  // live device allocations
    size_t limit = ~(size_t)0;                     // largest allocation that succeeds
    hipError_t last = hipSuccess;
    std::map<const void *, std::string> kernels;   // host stub -> mangled device name
    std::vector<FakeLaunch> launches;
    dim3 grid, block;
    size_t held() const
    {
        size_t n = 0;
        for (auto &m : mem) n += m.second;
        return n;
    }
};

inline FakeHip &fake()
{
    static FakeHip *f = new FakeHip;
    return *f;
}

inline hipError_t fake_ret(hipError_t e)
{
    if (e != hipSuccess) fake().last = e;
    return e;
}

extern "C" {

void **__hipRegisterFatBinary(const void *)
{
    static void *handle = nullptr;
    return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, const char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, dim3 *, dim3 *,
                           int *)
{
    fake().kernels[host] = name;
}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t, hipStream_t)
{
    fake().grid = g;
    fake().block = b;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *shared, hipStream_t *s)
{
    *g = fake().grid;
    *b = fake().block;
    *shared = 0;
    *s = nullptr;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **, size_t, hipStream_t)
{
    fake().launches.push_back({fake().kernels[f], g, b});
    return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n)
{
    if (n > fake().limit) return fake_ret(hipErrorOutOfMemory);
    // the address alone is used: one page stands for it
    *p = std::aligned_alloc(256, 4096);
    fake().mem[*p] = n;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    if (!fake().mem.erase(p)) std::abort();
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void *, const void *, size_t, hipMemcpyKind) { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipGetLastError()
{
    const hipError_t e = fake().last;
    fake().last = hipSuccess;
    return e;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int)
{
    std::memset((void *)p, 0, sizeof(*p));
    std::strcpy(p->gcnArchName, "gfx950:sramecc+:xnack-");
    return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *)
{
    std::memset((void *)a, 0, sizeof(*a));
    a->type = hipMemoryTypeDevice;
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return *p = std::calloc(1, n), hipSuccess; }
hipError_t hipHostFree(void *p) { return std::free(p), hipSuccess; }
hipError_t hipHostGetDevicePointer(void **d, void *h, unsigned) { return *d = h, hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return *e = (hipEvent_t)std::malloc(1), hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { return std::free(e), hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t)
{
    static float t = 1.0f;   // ever shorter: the last shape timed is the fastest
    return *ms = t *= 0.99f, hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { return *s = (hipStream_t)std::malloc(1), hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { return std::free(s), hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }

}  // extern "C"
