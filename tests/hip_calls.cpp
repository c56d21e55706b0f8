// Stand-ins for the HIP calls that the library's host path makes, loaded ahead
// of the runtime in a process without a GPU: every buffer is one large
// allocation, the device a 256-CU gfx950 on which two workgroups fit a CU, and
// launches and function attributes are recorded instead of carried out.
#include <hip/hip_runtime_api.h>

#include <mutex>
#include <string.h>

namespace {
struct Call {
    long long kind;  // 0: function attribute, 1: launch, 2: other driver query
    long long func, value;   // value: attribute value, or a launch's dynamic LDS
    long long gx, gy, block;
};
constexpr int kMax = 1 << 16;
Call calls[kMax];
int ncalls;
std::mutex mu;

void record(long long kind, const void *f, long long value, dim3 g = dim3(0, 0, 0), dim3 b = dim3(0, 0, 0))
{
    std::lock_guard<std::mutex> l(mu);
    if (ncalls < kMax)
        calls[ncalls++] = Call{kind, (long long)(size_t)f, value, g.x, g.y, b.x};
}
}  // namespace

extern "C" {
int shim_calls(Call *out, int most)
{
    std::lock_guard<std::mutex> l(mu);
    const int n = ncalls < most ? ncalls : most;
    memcpy(out, calls, sizeof(Call) * n);
    ncalls = 0;
    return n;
}

hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipMemGetAddressRange(hipDeviceptr_t *base, size_t *size, hipDeviceptr_t)
{
    *base = nullptr;
    *size = (size_t)1 << 62;
    return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_t *p, int)
{
    memset(p, 0, sizeof *p);
    strcpy(p->gcnArchName, "gfx950");
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t, int)
{
    record(2, nullptr, 0);
    *v = 256;
    return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute, int value)
{
    record(0, f, value);
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t)
{
    record(2, nullptr, 0);
    *n = 2;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **, size_t lds, hipStream_t)
{
    record(1, f, (long long)lds, g, b);
    return hipSuccess;
}
}
