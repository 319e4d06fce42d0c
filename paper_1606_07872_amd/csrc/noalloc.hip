// The peak search of asp_find_peak for callers that cannot allocate device
// memory (code under HIP graph capture, serving loops, harnesses that forbid
// hipMalloc): no context, no allocation.  Its scratch -- one packed key per
// work-group of the scan -- is a file-scope device array, one copy per GPU,
// kept until the process ends.
#include <stdio.h>

#include <mutex>

#include "asp_device.h"
#include "cycle.h"

namespace asp {
namespace {

// The packed keys (|v| bits << 32) | (0xFFFFFFFF - idx), 2 KiB per GPU.  A call's
// scan writes the key of each of its work-groups and its second kernel reads
// just those: nothing is cleared (a launch of its own) and no call sees what
// another left.  One work-group of 16 waves per CU leaves few keys to read: 4096 x
// 4096 in 12.4 us, 2048 x 2048 in 6.9, 16384 x 16384 in 163, against 13.4, 9.6 and
// 193 with eight work-groups of 4 waves per CU and an atomic maximum.
constexpr int kNaT = 1024, kNaKeys = 256;
__device__ __align__(256) unsigned long long scratch[kNaKeys];

constexpr int kMaxDevices = 64;
std::mutex g_lock;
unsigned long long *g_scratch[kMaxDevices];   // device address of `scratch` per GPU

__global__ __launch_bounds__(kNaT) void k_na_scan(const float *__restrict__ R, int64_t n,
                                                 unsigned long long *keys)
{
    const unsigned long long k = peak_key<kNaT / 64>(R, n, blockIdx.x, gridDim.x);
    if (threadIdx.x == 0) keys[blockIdx.x] = k;
}

// One wave: the maximum of the first m keys (all are read, and the rest not
// counted), decoded into the pixel index and the residual value there.  Without
// a key (every pixel NaN) there is no pixel: index 2^32 - 1 and NaN.
__global__ __launch_bounds__(64) void k_na_out(const float *__restrict__ R,
                                               const unsigned long long *keys, int m,
                                               int64_t *idx_out, float *value_out)
{
    constexpr int U = kNaKeys / 128;
    static_assert(128 * U == kNaKeys, "two keys to a load, whole rounds");
    const int t = threadIdx.x;
    ulonglong2 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = reinterpret_cast<const ulonglong2 *>(keys)[t + 64 * u];
    unsigned long long k = 0ull;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int i = 2 * (t + 64 * u);
        k = i < m && v[u].x > k ? v[u].x : k;
        k = i + 1 < m && v[u].y > k ? v[u].y : k;
    }
    k = wave_max_u64(k);
    if (t == 0) {
        const int64_t idx = (int64_t)(0xFFFFFFFFu - (uint32_t)(k & 0xFFFFFFFFull));
        *idx_out = idx;
        *value_out = k ? R[idx] : __builtin_nanf("");
    }
}

// The device address of `scratch` on the current GPU, resolved once per GPU.
hipError_t scratch_on_device(unsigned long long **out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> guard(g_lock);
    if (!g_scratch[dev]) {
        void *ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch[dev] = static_cast<unsigned long long *>(ptr);
    }
    *out = g_scratch[dev];
    return hipSuccess;
}

}  // namespace
}  // namespace asp

extern "C" asp_status asp_find_peak_noalloc(const float *R, int64_t H, int64_t W,
                                            int64_t *idx_out, float *value_out, void *stream)
{
    if (!R || !idx_out || !value_out || H <= 0 || W <= 0) return ASP_ERR_INVALID_ARG;
    if ((double)H * (double)W >= 4294967295.0) {
        fprintf(stderr, "asp_find_peak_noalloc: %lld x %lld pixels exceed the maximum of "
                        "2^32 - 2 (the packed key holds a 32-bit index)\n",
                (long long)H, (long long)W);
        return ASP_ERR_INVALID_ARG;
    }
    if (reinterpret_cast<uintptr_t>(R) % 16 != 0) {
        fprintf(stderr, "asp_find_peak_noalloc: the image must be 16-byte aligned\n");
        return ASP_ERR_INVALID_ARG;
    }
    unsigned long long *keys = nullptr;
    if (asp::scratch_on_device(&keys) != hipSuccess) return ASP_ERR_DEVICE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) != hipSuccess) return ASP_ERR_DEVICE;
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    const int64_t n = H * W;
    const int64_t need = (n / 4 + asp::kNaT - 1) / asp::kNaT;
    const int64_t cap = cus < asp::kNaKeys ? cus : asp::kNaKeys;
    const int grid = (int)(need < 1 ? 1 : (need < cap ? need : cap));
    hipLaunchKernelGGL(asp::k_na_scan, dim3(grid), dim3(asp::kNaT), 0, s, R, n, keys);
    hipLaunchKernelGGL(asp::k_na_out, dim3(1), dim3(64), 0, s, R, keys, grid, idx_out, value_out);
    return hipGetLastError() == hipSuccess ? ASP_OK : ASP_ERR_DEVICE;
}
