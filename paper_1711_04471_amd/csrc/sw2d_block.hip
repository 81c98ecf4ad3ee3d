// sw2d_block.hip - the single-grid step by register tiles (sw2d_block.h).
#include <hip/hip_runtime.h>

#include "sw2d_block.h"
#include "sw2d_internal.h"

namespace sw2d {

template <int K, int R, bool kWide>
__global__ __launch_bounds__(kWave * kBlockWaves) void sw2d_block_kernel(
    const float* __restrict__ eta, const float* __restrict__ u, const float* __restrict__ v,
    const float* __restrict__ hp, float* __restrict__ eta_o, float* __restrict__ u_o, float* __restrict__ v_o,
    FoldPartial* __restrict__ part, BlockGeometry geo, StepCoef k) {
    constexpr int W = kBlockWaves;
    __shared__ BlockShared<W> sh;
    __shared__ double s_disp[K][W];
    __shared__ float s_mu[K][W], s_mv[K][W];
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
    block_pass<K, R, W, kWide>(eta, u, v, hp, eta_o, u_o, v_o, geo.nx, geo.ny, r0 + wave * R, wave, lane, c0, owned,
                               j0, j1, k, sh, F);
#pragma unroll
    for (int s = 0; s < K; ++s) {
        double d = F[s].disp;
        float mu = F[s].max_u, mv = F[s].max_v;
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) {
            d += __shfl_xor(d, off, kWave);
            mu = fmaxf(mu, __shfl_xor(mu, off, kWave));
            mv = fmaxf(mv, __shfl_xor(mv, off, kWave));
        }
        if (lane == 0) {
            s_disp[s][wave] = d;
            s_mu[s][wave] = mu;
            s_mv[s][wave] = mv;
        }
    }
    __syncthreads();
    if (threadIdx.x < K) {
        const int s = threadIdx.x;
        double d = 0.0;
        float mu = 0.f, mv = 0.f;
        for (int i = 0; i < W; ++i) {
            d += s_disp[s][i];
            mu = fmaxf(mu, s_mu[s][i]);
            mv = fmaxf(mv, s_mv[s][i]);
        }
        FoldPartial* o = part + (size_t)s * geo.nblocks + blockIdx.x;
        o->disp = d;
        o->mu = mu;
        o->mv = mv;
    }
}

hipError_t launch_block(int K, const float* eta, const float* u, const float* v, const float* hp, float* eta_o,
                        float* u_o, float* v_o, FoldPartial* part, const BlockGeometry& geo, const StepCoef& k,
                        hipStream_t s) {
    const dim3 grid(geo.nblocks), block(kWave * kBlockWaves);
    // 8-byte row accesses: a pair never straddles a row end, and every row starts on 8 bytes
    uintptr_t low = reinterpret_cast<uintptr_t>(hp);
    for (const float* p : {eta, u, v, (const float*)eta_o, (const float*)u_o, (const float*)v_o})
        low |= reinterpret_cast<uintptr_t>(p);
    const bool wide = geo.nx % 2 == 0 && low % 8 == 0;
#define SW2D_BLOCK_CASE(KK, RR)                                                                                        \
    if (K == (KK) && geo.rows == (RR)) {                                                                              \
        if (wide)                                                                                                     \
            hipLaunchKernelGGL((sw2d_block_kernel<KK, RR, true>), grid, block, 0, s, eta, u, v, hp, eta_o, u_o, v_o,  \
                               part, geo, k);                                                                         \
        else                                                                                                          \
            hipLaunchKernelGGL((sw2d_block_kernel<KK, RR, false>), grid, block, 0, s, eta, u, v, hp, eta_o, u_o, v_o, \
                               part, geo, k);                                                                         \
        return hipGetLastError();                                                                                     \
    }
    SW2D_BLOCK_CASE(1, kBlockRowsLow)
    SW2D_BLOCK_CASE(2, kBlockRowsLow)
    SW2D_BLOCK_CASE(3, kBlockRowsLow)
    SW2D_BLOCK_CASE(4, kBlockRowsLow)
    SW2D_BLOCK_CASE(2, kBlockRowsHigh)
    SW2D_BLOCK_CASE(3, kBlockRowsHigh)
    SW2D_BLOCK_CASE(4, kBlockRowsHigh)
#undef SW2D_BLOCK_CASE
    return hipErrorInvalidValue;
}

}  // namespace sw2d
