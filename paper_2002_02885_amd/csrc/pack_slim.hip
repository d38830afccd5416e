// Launches of the slim form of the dense products (gemm_slim_device.h).
#include "gemm_slim_device.h"

namespace packk {

template <int MODE, typename T, int TM, int TN>
__global__ __launch_bounds__(64 * SLIM_WAVES) void slim_kernel(const GemmProb* __restrict__ probs, const TileRef* __restrict__ tiles,
                                                               const void* __restrict__ x) {
    __shared__ __attribute__((aligned(16))) char lds[SlimCfg<(int)sizeof(T), MODE != LIN_FWD, TM, TN>::LDS_BYTES];
    const TileRef tr = tiles[blockIdx.x];
    if (tr.prob < 0) return;
    slim_body<MODE, T, TM, TN>(probs[tr.prob], tr, x, lds);
}

hipError_t launch_slim(int mode, bool bf16, int tile_cfg, const GemmProb* probs, const TileRef* tiles, int n, const void* x, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    const dim3 grid(n), block(64 * SLIM_WAVES);
    const bool big = tile_cfg == GEMM_CFG_SLIM64;
    if (big && !(bf16 && mode == LIN_FWD)) return hipErrorInvalidValue;
    if (mode == LIN_FWD) {
        if (!bf16) hipLaunchKernelGGL((slim_kernel<LIN_FWD, float, 1, 1>), grid, block, 0, st, probs, tiles, x);
        else if (big) hipLaunchKernelGGL((slim_kernel<LIN_FWD, bf16_t, 2, 2>), grid, block, 0, st, probs, tiles, x);
        else hipLaunchKernelGGL((slim_kernel<LIN_FWD, bf16_t, 1, 1>), grid, block, 0, st, probs, tiles, x);
    } else if (mode == LIN_DX) {
        if (bf16) hipLaunchKernelGGL((slim_kernel<LIN_DX, bf16_t, 1, 1>), grid, block, 0, st, probs, tiles, x);
        else hipLaunchKernelGGL((slim_kernel<LIN_DX, float, 1, 1>), grid, block, 0, st, probs, tiles, x);
    } else {
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace packk
