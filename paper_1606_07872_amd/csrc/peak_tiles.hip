// Incremental peak search (Sect. 2 step 1): the largest |R|, the lowest
// row-major index winning ties, from per-tile maxima kept on the device.
//
// A residual update changes R only inside its windows, so only the 64 x 64
// tiles those windows touch can change their maximum.  The update lists each
// such tile once (its stale flag going from 0 to 1); here a fixed grid rescans
// the listed tiles, and one work-group reduces all tile keys into the peak
// key.  The packed key (|v| bits << 32) | (0xFFFFFFFF - idx) is the one of the
// full scan, so the result is the same pixel bit for bit.
#include "asp_device.h"
#include "cycle.h"

namespace asp {
namespace {

constexpr int kT = 256;
constexpr int kReduceT = 1024;
constexpr int kTileGrid = 1024;

__global__ __launch_bounds__(kT) void k_peak_tiles(Params p)
{
    if (p.st->stop) return;
    peak_tiles_scan(p, blockIdx.x, gridDim.x);
}

// The tile pass has finished.
__global__ __launch_bounds__(kReduceT) void k_peak_reduce(Params p)
{
    if (p.st->stop) return;
    peak_tiles_reduce(p);
}

__global__ __launch_bounds__(kT) void k_peak_mark_all(Params p)
{
    const PeakTiles K = p.st->pk;
    const int ntiles = K.tiles_x * K.tiles_y;
    for (int i = blockIdx.x * kT + threadIdx.x; i < ntiles; i += gridDim.x * kT) {
        K.dirty[i] = 1;
        K.list[i] = i;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) K.count[0] = (unsigned int)ntiles;
}

}  // namespace

hipError_t launch_peak_tiles(const Params &p, int ntiles, hipStream_t s)
{
    const int grid = ntiles < kTileGrid ? ntiles : kTileGrid;
    hipLaunchKernelGGL(k_peak_tiles, dim3(grid), dim3(kT), 0, s, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_peak_reduce, dim3(1), dim3(kReduceT), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_peak_mark_all(const Params &p, hipStream_t s)
{
    hipLaunchKernelGGL(k_peak_mark_all, dim3(64), dim3(kT), 0, s, p);
    return hipGetLastError();
}

}  // namespace asp
