// Per-step launch of a tiled step (tile_dev.hpp): four wave tiles a block.
#include <hip/hip_runtime.h>

#include "kernels.hpp"
#include "tile_dev.hpp"

namespace htn {
namespace kern {

__global__ __launch_bounds__(kBlk) __attribute__((amdgpu_waves_per_eu(2))) void k_tile(
    const void *__restrict__ A, int ta, const void *__restrict__ B, int tb, void *__restrict__ C, int tc,
    const int2 *__restrict__ tab, TileArgs t) {
    tile_wave_any(A, ta, B, tb, C, tc, tab, t, __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6)));
}

hipError_t launch_tile(const void *A, int ta, const void *B, int tb, void *C, int tc, const int2 *tab,
                       const TileArgs &t, void *part, hipStream_t st) {
    if (ta < 0 || ta > 2 || tb < 0 || tb > 2 || tc < 0 || tc > 2) return hipErrorInvalidValue;
    if ((ta == 0) != (tb == 0) || (ta == 0 && tc != 0)) return hipErrorInvalidValue;
    if (t.M < 1 || t.N < 1 || t.K < 1 || t.ksplit < 1 || (t.ksplit > 1 && (!part || tc == 2)))
        return hipErrorInvalidValue;
    const int64_t units = (int64_t)t.tiles_m * t.tiles_n * t.ksplit;
    if (units > (int64_t(1) << 30)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_tile, dim3((unsigned)((units + 3) / 4)), dim3(kBlk), 0, st, A, ta, B, tb,
                       t.ksplit > 1 ? part : C, tc, tab, t);
    if (t.ksplit > 1) return launch_ksum(part, C, tc, t.total, t.ksplit, st);
    return hipGetLastError();
}

}  // namespace kern
}  // namespace htn
