// sw2d_block.hip - the single-grid step by register tiles (sw2d_block.h).
#include <hip/hip_runtime.h>

#include "sw2d_block.h"
#include "sw2d_internal.h"

namespace sw2d {

template <int K, int R>
__global__ __launch_bounds__(kWave * kBlockWaves) void sw2d_block_kernel(
    const float* __restrict__ eta, const float* __restrict__ u, const float* __restrict__ v,
    const float* __restrict__ hp, float* __restrict__ eta_o, float* __restrict__ u_o, float* __restrict__ v_o,
    FoldPartial* __restrict__ part, BlockGeometry geo, StepCoef k) {
    constexpr int W = kBlockWaves;
    __shared__ BlockShared<W> sh;
    __shared__ BlockFoldShared<W> fsh;
    // workgroup b runs on XCD b % 8: each XCD takes a contiguous range of tiles
    const int q = geo.nblocks / kXcds, rem = geo.nblocks % kXcds;
    const int x = blockIdx.x % kXcds;
    const int tile = x * q + min(x, rem) + (int)blockIdx.x / kXcds;
    const int band = tile / geo.strips, strip = tile - band * geo.strips;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
    constexpr int T = W * R;
    const int r0 = band * (T - 4 * K), cb = strip * (kBlockCols - 4 * K);
    const int j0 = band > 0 ? r0 + 2 * K : 0, j1 = band + 1 < geo.bands ? r0 + T - 2 * K : geo.ny;
    const int c0 = cb + 2 * lane;
    const bool owned = (strip == 0 || lane >= K) && (strip + 1 == geo.strips ? c0 < geo.nx : lane < kWave - K);

    BlockFolds F[K];
    block_pass<K, R, W>(eta, u, v, hp, eta_o, u_o, v_o, geo.nx, geo.ny, r0 + wave * R, wave, lane, c0, owned,
                               j0, j1, k, sh, F);
    block_fold<K, W>(F, wave, lane, fsh, part + blockIdx.x, geo.nblocks);
}

hipError_t launch_block(int K, const float* eta, const float* u, const float* v, const float* hp, float* eta_o,
                        float* u_o, float* v_o, FoldPartial* part, const BlockGeometry& geo, const StepCoef& k,
                        hipStream_t s) {
    const dim3 grid(geo.nblocks), block(kWave * kBlockWaves);
#define SW2D_BLOCK_CASE(KK, RR)                                                                                       \
    if (K == (KK) && geo.rows == (RR)) {                                                                             \
        hipLaunchKernelGGL((sw2d_block_kernel<KK, RR>), grid, block, 0, s, eta, u, v, hp, eta_o, u_o, v_o, part, geo, k); \
        return hipGetLastError();                                                                                    \
    }
    SW2D_BLOCK_CASE(1, kBlockRowsLow)
    SW2D_BLOCK_CASE(2, kBlockRowsLow)
    SW2D_BLOCK_CASE(3, kBlockRowsLow)
    SW2D_BLOCK_CASE(4, kBlockRowsLow)
    SW2D_BLOCK_CASE(3, kBlockRowsMid)
    SW2D_BLOCK_CASE(4, kBlockRowsMid)
    SW2D_BLOCK_CASE(4, kBlockRowsHigh)
#undef SW2D_BLOCK_CASE
    return hipErrorInvalidValue;
}

}  // namespace sw2d
