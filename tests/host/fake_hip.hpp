// A HIP runtime on host memory, for tests of the library's host code without a
// GPU: linked into an executable that exports its symbols, it takes the place
// of the runtime's functions below for libnufft_resample.so.  Kernel launches
// are recorded and not run; time passes by launches (fake_hip::cost), and the
// allocation numbered fake_hip::fail_at fails and, as in the runtime, leaves
// its error for hipGetLastError.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <string>
#include <vector>

namespace fake_hip {

struct Launch {
    std::string kernel;      // mangled name
    dim3 grid, block;
    size_t lds;
    std::vector<char> arg;   // the first argument's leading bytes
    bool is(const char* part) const { return kernel.find(part) != std::string::npos; }
};

inline std::vector<Launch> launches;
// (the library registers its kernels before this executable's own objects exist)
inline std::map<const void*, std::string>& names()
{
    static std::map<const void*, std::string> m;
    return m;
}
inline std::function<double(const Launch&)> cost = [](const Launch&) { return 1.0; };   // ms
inline double clock = 0.0;
inline int64_t allocations = 0, fail_at = -1;
inline size_t arg_bytes = 0;         // bytes of the first argument to keep
inline hipError_t last = hipSuccess;

struct Config {
    dim3 grid, block;
    size_t lds;
    hipStream_t stream;
};
inline std::vector<Config> configs;
struct Event {
    double at = 0.0;
};

}  // namespace fake_hip

extern "C" {

hipError_t hipMalloc(void** p, size_t n)
{
    if (fake_hip::allocations++ == fake_hip::fail_at) {
        *p = nullptr;
        return fake_hip::last = hipErrorOutOfMemory;
    }
    *p = std::calloc(1, n);
    return hipSuccess;
}
hipError_t hipFree(void* p)
{
    std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void* to, const void* from, size_t n, hipMemcpyKind)
{
    std::memcpy(to, from, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* to, const void* from, size_t n, hipMemcpyKind, hipStream_t)
{
    std::memcpy(to, from, n);
    return hipSuccess;
}
hipError_t hipMemset(void* p, int v, size_t n)
{
    std::memset(p, v, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void* p, int v, size_t n, hipStream_t)
{
    std::memset(p, v, n);
    return hipSuccess;
}
hipError_t hipGetLastError(void)
{
    const hipError_t e = fake_hip::last;
    fake_hip::last = hipSuccess;
    return e;
}
hipError_t hipPeekAtLastError(void) { return fake_hip::last; }

hipError_t hipEventCreate(hipEvent_t* e)
{
    *e = reinterpret_cast<hipEvent_t>(new fake_hip::Event());
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e)
{
    delete reinterpret_cast<fake_hip::Event*>(e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t)
{
    reinterpret_cast<fake_hip::Event*>(e)->at = fake_hip::clock;
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b)
{
    *ms = (float)(reinterpret_cast<fake_hip::Event*>(b)->at - reinterpret_cast<fake_hip::Event*>(a)->at);
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned)
{
    *s = reinterpret_cast<hipStream_t>(std::malloc(1));
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t s)
{
    std::free(s);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }

hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t st)
{
    fake_hip::configs.push_back({grid, block, lds, st});
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* st)
{
    const fake_hip::Config c = fake_hip::configs.back();
    fake_hip::configs.pop_back();
    *grid = c.grid;
    *block = c.block;
    *lds = c.lds;
    *st = c.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t lds, hipStream_t)
{
    fake_hip::Launch l{fake_hip::names()[f], grid, block, lds, {}};
    l.arg.assign((const char*)args[0], (const char*)args[0] + fake_hip::arg_bytes);
    // the limits of a real launch
    const bool fits = (uint64_t)grid.x * block.x < (uint64_t(1) << 32) && grid.x > 0 && grid.y > 0 && grid.z > 0;
    fake_hip::clock += fake_hip::cost(l);
    fake_hip::launches.push_back(std::move(l));
    if (!fits) fake_hip::last = hipErrorInvalidConfiguration;
    return fits ? hipSuccess : hipErrorInvalidConfiguration;
}
void** __hipRegisterFatBinary(const void*)
{
    static void* handle = nullptr;
    return &handle;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*)
{
    fake_hip::names()[f] = name;
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterManagedVar(void*, void**, void*, const char*, size_t, unsigned) {}

}  // extern "C"
