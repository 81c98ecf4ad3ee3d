// sw2d_block.hip - the single-grid step by register tiles (sw2d_block.h).
#include <hip/hip_runtime.h>

#include "sw2d_block.h"
#include "sw2d_internal.h"

namespace sw2d {

template <int K, int R, int kVar>
__global__ __launch_bounds__(kWave * kBlockWaves) void sw2d_block_kernel(
    const float* __restrict__ eta, const float* __restrict__ u, const float* __restrict__ v,
    const float* __restrict__ hp, float* __restrict__ eta_o, float* __restrict__ u_o, float* __restrict__ v_o,
    FoldPartial* __restrict__ part, BlockGeometry geo, StepCoef k) {
    constexpr int W = kBlockWaves;
    __shared__ BlockShared<W, kVar> sh;
    __shared__ BlockFoldShared<W> fsh;
    // workgroup b runs on XCD b % 8: each XCD takes a contiguous range of tiles, or, of a grid read from
    // HBM (which takes the highest tiles), runs of kBlockRun tiles in turn
    const int b = blockIdx.x, x = b % kXcds;
    int tile;
    if (R < 8 || geo.contiguous) {
        const int q = geo.nblocks / kXcds, rem = geo.nblocks % kXcds;
        tile = x * q + min(x, rem) + b / kXcds;
    } else {
        constexpr int kTurn = kBlockRun * kXcds;
        tile = b < geo.nblocks / kTurn * kTurn ? b / kTurn * kTurn + x * kBlockRun + b % kTurn / kXcds : b;
    }
    const int band = tile / geo.strips, strip = tile - band * geo.strips;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
    constexpr int T = W * R, kSouth = block_south(kVar) * K, kNorth = 2 * K, kWest = block_west_lanes(K, kVar);
    const int r0 = band * (T - kSouth - kNorth), cb = strip * (kBlockCols - 2 * (kWest + K));
    const int j0 = band > 0 ? r0 + kSouth : 0, j1 = band + 1 < geo.bands ? r0 + T - kNorth : geo.ny;
    const int c0 = cb + 2 * lane;
    const bool owned = (strip == 0 || lane >= kWest) && (strip + 1 == geo.strips ? c0 < geo.nx : lane < kWave - K);

    BlockFolds F[K];
    block_pass<K, R, W, kVar>(eta, u, v, hp, eta_o, u_o, v_o, geo.nx, geo.ny, r0 + wave * R, wave, lane, c0, owned,
                              j0, j1, k, sh, F);
    block_fold<K, W>(F, wave, lane, fsh, part + blockIdx.x, geo.nblocks);
}

// The correction of a row's cells: the network's planes and the mask bytes of the pair, of its east
// neighbour and of the row above, as the correction kernel reads them.
struct BlockCorrect {
    StepCorrection c;
    int nx, ny, c0;
    __device__ __forceinline__ void operator()(const BlockIO& io, int row, float (&e)[2], float (&u)[2],
                                               float (&v)[2]) const {
        const size_t plane = (size_t)nx * ny;
        float d[3][2];
#pragma unroll
        for (int f = 0; f < 3; ++f) io.load(c.delta + f * plane, row, d[f]);
        const uint8_t* const at = c.mask + (size_t)row * nx;
        bool w[3], n[2];
#pragma unroll
        for (int i = 0; i < 3; ++i) w[i] = at[min(c0 + i, nx - 1)] != 0 && c0 + i < nx;
#pragma unroll
        for (int i = 0; i < 2; ++i) n[i] = at[(row + 1 < ny ? nx : 0) + min(c0 + i, nx - 1)] != 0 && row + 1 < ny;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            if (!w[i]) continue;
            e[i] = fmaf(c.scale[0], d[0][i], e[i]);
            if (w[i + 1]) u[i] = fmaf(c.scale[1], d[1][i], u[i]);
            if (n[i]) v[i] = fmaf(c.scale[2], d[2][i], v[i]);
        }
    }
};

// A corrected step of a small grid costs its launches. With the correction as one of its own after the
// step, five corrected steps of a 300 x 221 grid took 98.3 us; added as the step stores its state, 93.2.
template <int R>
__global__ __launch_bounds__(kWave * kBlockWaves) void sw2d_block_correct_kernel(
    const float* __restrict__ eta, const float* __restrict__ u, const float* __restrict__ v,
    const float* __restrict__ hp, float* __restrict__ eta_o, float* __restrict__ u_o, float* __restrict__ v_o,
    FoldPartial* __restrict__ part, BlockGeometry geo, StepCoef k, StepCorrection fix) {
    constexpr int W = kBlockWaves, K = 1, T = W * R;
    __shared__ BlockShared<W> sh;
    __shared__ BlockFoldShared<W> fsh;
    const int b = blockIdx.x, x = b % kXcds, q = geo.nblocks / kXcds, rem = geo.nblocks % kXcds;
    const int tile = x * q + min(x, rem) + b / kXcds;
    const int band = tile / geo.strips, strip = tile - band * geo.strips;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
    const int r0 = band * (T - 4 * K), c0 = strip * (kBlockCols - 4 * K) + 2 * lane;
    const int j0 = band > 0 ? r0 + 2 * K : 0, j1 = band + 1 < geo.bands ? r0 + T - 2 * K : geo.ny;
    const bool owned = (strip == 0 || lane >= K) && (strip + 1 == geo.strips ? c0 < geo.nx : lane < kWave - K);
    BlockFolds F[K];
    block_pass<K, R, W, 0>(eta, u, v, hp, eta_o, u_o, v_o, geo.nx, geo.ny, r0 + wave * R, wave, lane, c0, owned, j0, j1,
                           k, sh, F, BlockCorrect{fix, geo.nx, geo.ny, c0});
    block_fold<K, W>(F, wave, lane, fsh, part + blockIdx.x, geo.nblocks);
}

hipError_t launch_block_corrected(const float* eta, const float* u, const float* v, const float* hp, float* eta_o,
                                  float* u_o, float* v_o, FoldPartial* part, const BlockGeometry& geo,
                                  const StepCoef& k, const StepCorrection& fix, hipStream_t s) {
    static_assert(block_shape(1, 3, 0) && !block_shape(1, 5, 0), "one height at K = 1");
    hipLaunchKernelGGL(sw2d_block_correct_kernel<3>, dim3(geo.nblocks), dim3(kWave * kBlockWaves), 0, s, eta, u, v, hp,
                       eta_o, u_o, v_o, part, geo, k, fix);
    return hipGetLastError();
}

template <int kVar>
hipError_t launch_variant(int K, const float* eta, const float* u, const float* v, const float* hp, float* eta_o,
                          float* u_o, float* v_o, FoldPartial* part, const BlockGeometry& geo, const StepCoef& k,
                          hipStream_t s) {
    const dim3 grid(geo.nblocks), block(kWave * kBlockWaves);
#define SW2D_BLOCK_CASE(KK, RR)                                                                                   \
    if constexpr (block_shape(KK, RR, kVar)) {                                                                    \
        if (K == (KK) && geo.rows == (RR)) {                                                                      \
            hipLaunchKernelGGL((sw2d_block_kernel<KK, RR, kVar>), grid, block, 0, s, eta, u, v, hp, eta_o, u_o, v_o, \
                               part, geo, k);                                                                     \
            return hipGetLastError();                                                                             \
        }                                                                                                         \
    }
#define SW2D_BLOCK_ROWS(RR) \
    SW2D_BLOCK_CASE(1, RR) SW2D_BLOCK_CASE(2, RR) SW2D_BLOCK_CASE(3, RR) SW2D_BLOCK_CASE(4, RR)
    SW2D_BLOCK_ROWS(3)
    SW2D_BLOCK_ROWS(5)
    SW2D_BLOCK_ROWS(7)
    SW2D_BLOCK_ROWS(8)
#undef SW2D_BLOCK_ROWS
#undef SW2D_BLOCK_CASE
    return hipErrorInvalidValue;
}

hipError_t launch_block(int K, int kvar, const float* eta, const float* u, const float* v, const float* hp,
                        float* eta_o, float* u_o, float* v_o, FoldPartial* part, const BlockGeometry& geo,
                        const StepCoef& k, hipStream_t s) {
    switch (kvar) {
#define SW2D_BLOCK_VAR(V) \
    case V: return launch_variant<V>(K, eta, u, v, hp, eta_o, u_o, v_o, part, geo, k, s);
        SW2D_BLOCK_VAR(0)
        SW2D_BLOCK_VAR(1)
        SW2D_BLOCK_VAR(2)
        SW2D_BLOCK_VAR(3)
        SW2D_BLOCK_VAR(4)
        SW2D_BLOCK_VAR(5)
        SW2D_BLOCK_VAR(6)
        SW2D_BLOCK_VAR(7)
        SW2D_BLOCK_VAR(kVarWetDry)
#undef SW2D_BLOCK_VAR
    }
    return hipErrorInvalidValue;
}

}  // namespace sw2d
