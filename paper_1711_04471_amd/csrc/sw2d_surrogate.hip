// sw2d_surrogate.hip - kernels of the learned coarse-step surrogate of the 2DSW model.
//
// The surrogate advances a 4x-coarsened state of the model of Sect. 6.2 with the same
// fused step on the coarse grid (4 dx, 4 dt) and adds a correction predicted by a small
// convolutional network: 3x3 'same' convolutions 5 -> 32 -> 32 -> 32 -> 3 with ReLU after
// the first three. The plain fine model is its judge and fallback.
//
// Kernels here:
//   * restrict4      fine (eta, u, v, H, mask) -> coarse, 4x4 blocks;
//   * pack_input     coarse state -> normalised BF16 NHWC input (5 channels padded to 16);
//   * conv3x3        implicit GEMM on BF16 MFMA (v_mfma_f32_32x32x16_bf16), FP32 accumulate:
//                    out[p][n] = sum over taps t and channels k of in[p + off_t][k] Wk[t][n][k];
//                    used for the forward layers (bias + ReLU + BF16 store, or bias + FP32
//                    planar store of 3 channels) and for the data gradient (flipped,
//                    transposed weights; fused ReLU-mask of the layer input);
//   * backward       a layer's weight gradient dW[t][o][c] = sum_p dY[p][o] X[p + off_t][c] on MFMA
//                    (FP32 partials, then a fixed-order reduction), with the data gradient beside it;
//   * mse_grad       masked squared error and its gradient (BF16 NHWC, 32 or 4 channels);
//   * adam           Adam on FP32 master weights and their BF16 working copies in the forward
//                    and data-gradient layouts;
//   * correct        state += activity * t_std * out;
//   * rmse           sum over water of (a - b)^2 in FP64, fixed-order.
// Feature maps are NHWC BF16 with 16 or 32 channels: a pixel's channels are one 32/64 B
// row, so one lane's MFMA operand (8 consecutive channels) is one 16 B load.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "sw2d_internal.h"
#include "sw2d_surrogate.h"

namespace sw2d {
namespace sur {

typedef __attribute__((__vector_size__(8 * sizeof(short)))) short bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

// FP32 -> BF16, round to nearest even (one hardware conversion).
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

// Two values to BF16, packed with a in the low half.
__device__ __forceinline__ uint32_t f2bf2(float a, float b) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2_t){a, b}, bf16x2_t));
}

__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

// ------------------------------------------------------------------------------ restrict4
__global__ __launch_bounds__(256) void restrict4_kernel(const float* __restrict__ eta, const float* __restrict__ u,
                                                        const float* __restrict__ v, const float* __restrict__ H,
                                                        const uint8_t* __restrict__ mask, int NX, int NY,
                                                        float* __restrict__ eta_c, float* __restrict__ u_c,
                                                        float* __restrict__ v_c, float* __restrict__ H_c,
                                                        uint8_t* __restrict__ mask_c) {
    const int nx = NX / 4, ny = NY / 4;
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= nx * ny) return;
    const int J = idx / nx, I = idx - J * nx;
    auto wet_count = [&](int JJ, int II) -> int {
        if (JJ < 0 || II < 0 || JJ >= ny || II >= nx) return 0;
        int n = 0;
        for (int r = 0; r < 4; ++r)
            for (int c = 0; c < 4; ++c) n += mask[(size_t)(4 * JJ + r) * NX + 4 * II + c] != 0;
        return n;
    };
    int n = 0;
    float se = 0.f, sh = 0.f;
    for (int r = 0; r < 4; ++r)
        for (int c = 0; c < 4; ++c) {
            const size_t f = (size_t)(4 * J + r) * NX + 4 * I + c;
            if (mask[f]) {
                ++n;
                se += eta[f];
                sh += H[f];
            }
        }
    const bool wc = n >= 8;
    eta_c[idx] = wc ? se / (float)n : 0.f;
    H_c[idx] = n > 0 ? sh / (float)n : 0.f;
    mask_c[idx] = wc ? 1 : 0;
    const bool au = wc && wet_count(J, I + 1) >= 8;
    const bool av = wc && wet_count(J + 1, I) >= 8;
    float su = 0.f, sv = 0.f;
    for (int r = 0; r < 4; ++r) su += u[(size_t)(4 * J + r) * NX + 4 * I + 3];
    for (int c = 0; c < 4; ++c) sv += v[(size_t)(4 * J + 3) * NX + 4 * I + c];
    u_c[idx] = au ? 0.25f * su : 0.f;
    v_c[idx] = av ? 0.25f * sv : 0.f;
}

// ------------------------------------------------------------------------------ pack_input
// SplitMix64 (Steele, Lea & Flood, 2014) of the counter seed + (i + 1) * golden gamma, mapped
// to a uniform float in [-1, 1): the training-noise generator, keyed by (seed, element).
__device__ __forceinline__ float splitmix_uniform(uint64_t seed, uint64_t i) {
    uint64_t z = seed + (i + 1ull) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    return (float)(z >> 40) * (1.0f / 8388608.0f) - 1.0f;
}

// The 16 BF16 input channels of one pixel from its raw values x = (eta, u, v, H, mask):
// normalised, plus the training noise on channels 0..2, then 11 zero channels; two 16 B
// chunks. p is the pixel's index (the noise counter).
__device__ __forceinline__ void pack_values(const float (&x)[5], size_t p, const InputNorm& nrm, uint4& a,
                                            uint4& b) {
    uint16_t o[16];
#pragma unroll
    for (int c = 0; c < 16; ++c) o[c] = 0;
#pragma unroll
    for (int c = 0; c < 5; ++c) {
        float y = (x[c] - nrm.mean[c]) * nrm.inv_std[c];
        if (c < 3 && nrm.noise_amp > 0.f) y += nrm.noise_amp * splitmix_uniform(nrm.noise_seed, (uint64_t)p * 3 + c);
        o[c] = f2bf(y);
    }
    a.x = o[0] | ((uint32_t)o[1] << 16);
    a.y = o[2] | ((uint32_t)o[3] << 16);
    a.z = o[4] | ((uint32_t)o[5] << 16);
    a.w = o[6] | ((uint32_t)o[7] << 16);
    b.x = o[8] | ((uint32_t)o[9] << 16);
    b.y = o[10] | ((uint32_t)o[11] << 16);
    b.z = o[12] | ((uint32_t)o[13] << 16);
    b.w = o[14] | ((uint32_t)o[15] << 16);
}

__device__ __forceinline__ void pack_pixel(const float* __restrict__ eta, const float* __restrict__ u,
                                           const float* __restrict__ v, const float* __restrict__ H,
                                           const uint8_t* __restrict__ mask, size_t p, const InputNorm& nrm,
                                           uint4& a, uint4& b) {
    const float x[5] = {eta[p], u[p], v[p], H[p], mask[p] ? 1.f : 0.f};
    pack_values(x, p, nrm, a, b);
}

__global__ __launch_bounds__(256) void pack_input_kernel(const float* __restrict__ eta, const float* __restrict__ u,
                                                         const float* __restrict__ v, const float* __restrict__ H,
                                                         const uint8_t* __restrict__ mask, int npix, InputNorm nrm,
                                                         uint16_t* __restrict__ out) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= npix) return;
    uint4 a, b;
    pack_pixel(eta, u, v, H, mask, (size_t)p, nrm, a, b);
    uint4* dst = reinterpret_cast<uint4*>(out + (size_t)p * 16);
    dst[0] = a;
    dst[1] = b;
}

// ------------------------------------------------------------------------------ conv3x3
// Tile: kConvTH rows x 32 columns of output pixels per workgroup (4 waves, TH/4 rows each);
// the (TH+2) x 34 input patch is staged in LDS with a padded pixel stride.
constexpr int kConvTH = 8;
constexpr int kConvRowsPerWave = kConvTH / 4;
constexpr int kConvTW = 32;
constexpr int kConvThreads = 256;

template <int KIN>
struct ConvLds {
    static constexpr int kStride = KIN * 2 + 16;  // bytes per pixel, 16 B aligned, spreads banks
    static constexpr int kCols = kConvTW + 2;
    static constexpr int kRows = kConvTH + 2;
    static constexpr int kBytes = kRows * kCols * kStride;
};

template <int KIN, int MODE, bool kRaw = false>
__global__ __launch_bounds__(kConvThreads) void conv3x3_kernel(const uint16_t* __restrict__ in,
                                                               const uint16_t* __restrict__ Wk,
                                                               const float* __restrict__ bias,
                                                               uint16_t* __restrict__ out_bf,
                                                               float* __restrict__ out_f,
                                                               const uint16_t* __restrict__ relu_src, int H,
                                                               int W, int nimg, RawIn raw, InputNorm nrm,
                                                               CorrectOut co) {
    using L = ConvLds<KIN>;
    __shared__ __attribute__((aligned(16))) unsigned char patch[L::kBytes];
    const int tiles_x = (W + kConvTW - 1) / kConvTW;
    const int tiles_y = (H + kConvTH - 1) / kConvTH;
    const int per_img = tiles_x * tiles_y;
    const int total = per_img * nimg;

    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int half = lane / 32;  // which 8-channel group of a 16-channel chunk
    const int j = lane % 32;     // pixel within the 32-column block; also the A row (n)

    // A operands (weights), one per tap and 16-channel chunk: Wk[t][n = j][k0 + 8 half + 0..7],
    // loaded once and kept in registers while the workgroup walks its tiles
    constexpr int kK = KIN / 16;
    bf16x8 a[9][kK];
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int kc = 0; kc < kK; ++kc)
            a[t][kc] = *reinterpret_cast<const bf16x8*>(Wk + ((size_t)t * 32 + j) * KIN + kc * 16 + half * 8);
    // the bias is the accumulators' initial value (lane: output channels 8 q + 4 half + e)
    f32x16 binit;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) binit[4 * q + e] = MODE == kConvDgradMask ? 0.f : bias[8 * q + 4 * half + e];

    // The next tile's input patch is fetched into registers while the current one is
    // multiplied, then written to LDS: every load of a patch is in flight at once.
    constexpr int kChunks = KIN / 8;  // 16 B chunks per pixel
    constexpr int kPatchChunks = L::kRows * L::kCols * kChunks;
    constexpr int kPer = (kPatchChunks + kConvThreads - 1) / kConvThreads;
    uint4 pre[kPer];
    auto fetch = [&](int tile_g) {
        const int img = tile_g / per_img;
        const int tile = tile_g - img * per_img;
        const int ty = tile / tiles_x, tx = tile - ty * tiles_x;
        const int y0 = ty * kConvTH, x0 = tx * kConvTW;
        const size_t img_off = (size_t)img * H * W;
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const int e = threadIdx.x + q * kConvThreads;
            const int pix = e / kChunks, ch = e - pix * kChunks;
            const int r = pix / L::kCols, c = pix - r * L::kCols;
            const int gy = y0 + r - 1, gx = x0 + c - 1;
            pre[q] = make_uint4(0u, 0u, 0u, 0u);
            if (e < kPatchChunks && gy >= 0 && gy < H && gx >= 0 && gx < W) {
                if constexpr (kRaw) {  // pack the raw state here (KIN = 16: chunk 0 or 1)
                    uint4 a, b;
                    pack_pixel(raw.eta, raw.u, raw.v, raw.H, raw.mask, img_off + (size_t)gy * W + gx, nrm, a, b);
                    pre[q] = ch == 0 ? a : b;
                } else {
                    pre[q] = reinterpret_cast<const uint4*>(in + (img_off + (size_t)gy * W + gx) * KIN)[ch];
                }
            }
        }
    };
    auto commit = [&]() {
#pragma unroll
        for (int q = 0; q < kPer; ++q) {
            const int e = threadIdx.x + q * kConvThreads;
            const int pix = e / kChunks, ch = e - pix * kChunks;
            if (e < kPatchChunks) *reinterpret_cast<uint4*>(patch + pix * L::kStride + ch * 16) = pre[q];
        }
    };

    if ((int)blockIdx.x < total) fetch(blockIdx.x);
    for (int tile_g = blockIdx.x; tile_g < total; tile_g += gridDim.x) {
        const int img = tile_g / per_img;
        const int tile = tile_g - img * per_img;
        const int ty = tile / tiles_x, tx = tile - ty * tiles_x;
        const int y0 = ty * kConvTH, x0 = tx * kConvTW;
        const size_t img_off = (size_t)img * H * W;

        __syncthreads();  // the previous tile's patch is no longer read
        commit();
        __syncthreads();
        if (tile_g + (int)gridDim.x < total) fetch(tile_g + gridDim.x);

        f32x16 acc[kConvRowsPerWave];
#pragma unroll
        for (int b = 0; b < kConvRowsPerWave; ++b) acc[b] = binit;

#pragma unroll
        for (int b = 0; b < kConvRowsPerWave; ++b) {
            const int r = wave * kConvRowsPerWave + b;  // output row within the tile
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                const int ky = t / 3, kx = t - 3 * (t / 3);
                const unsigned char* src = patch + ((r + ky) * L::kCols + (j + kx)) * L::kStride + half * 16;
#pragma unroll
                for (int kc = 0; kc < kK; ++kc) {
                    const bf16x8 bv = *reinterpret_cast<const bf16x8*>(src + kc * 32);
                    acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[t][kc], bv, acc[b], 0, 0, 0);
                }
            }
        }

        // epilogue: lane holds pixel j, output channels n = 8 (q) + 4 half + (0..3), q = 0..3
#pragma unroll
        for (int b = 0; b < kConvRowsPerWave; ++b) {
            const int gy = y0 + wave * kConvRowsPerWave + b, gx = x0 + j;
            if (gy >= H || gx >= W) continue;
            const size_t p = img_off + (size_t)gy * W + gx;
            if constexpr (MODE == kConvRelu || MODE == kConvDgradMask) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int n0 = 8 * q + 4 * half;
                    uint16_t o[4];
                    if constexpr (MODE == kConvRelu) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) o[e] = f2bf(fmaxf(acc[b][4 * q + e], 0.f));
                    } else {
                        const uint2 m = *reinterpret_cast<const uint2*>(relu_src + p * 32 + n0);
                        const uint16_t mv[4] = {(uint16_t)(m.x & 0xffff), (uint16_t)(m.x >> 16),
                                                (uint16_t)(m.y & 0xffff), (uint16_t)(m.y >> 16)};
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            o[e] = (bf2f(mv[e]) > 0.f) ? f2bf(acc[b][4 * q + e]) : (uint16_t)0;
                    }
                    uint2 w;
                    w.x = o[0] | ((uint32_t)o[1] << 16);
                    w.y = o[2] | ((uint32_t)o[3] << 16);
                    *reinterpret_cast<uint2*>(out_bf + p * 32 + n0) = w;
                }
            } else if constexpr (MODE == kConvCorrect) {
                // the state += activity * (output * scale), as the correction kernel does
                if (half == 0 && co.mask[p] != 0) {
                    co.eta[p] = fmaf(co.s0, acc[b][0], co.eta[p]);
                    if (gx + 1 < W && co.mask[p + 1]) co.u[p] = fmaf(co.s1, acc[b][1], co.u[p]);
                    if (gy + 1 < H && co.mask[p + W]) co.v[p] = fmaf(co.s2, acc[b][2], co.v[p]);
                }
            } else {  // kConvLinear3: channels 0..2 as FP32 planes [img][3][H][W]
                if (half == 0) {
#pragma unroll
                    for (int e = 0; e < 3; ++e)
                        out_f[((size_t)img * 3 + e) * H * W + (size_t)gy * W + gx] = acc[b][e];
                }
            }
        }
    }
}

// ------------------------------------------------------------------------------ fused forward
// The four layers of one image in one pass (inference). A workgroup owns a TH x kFuTW tile
// of output pixels and computes every layer over the tile grown by the receptive field still
// ahead of it: layer 1 over (TH + 6) x (TW + 6) pixels of the (TH + 8) x (TW + 8) packed input,
// layer 2 over (TH + 4) x (TW + 4), layer 3 over (TH + 2) x (TW + 2), layer 4 over the tile.
// The maps stay in LDS, two buffers used in turn; a map's pixels outside the image are stored
// as 0, which is the next layer's zero padding. A layer's pixels are taken 32 at a time along the
// pairs of rows of its region (the lane's address carries the wrap), two rows per block, so that an
// input row's operands serve both. Taps, channel chunks, the packing of the input and the epilogues
// are those of the layer-by-layer kernels: the output is bitwise theirs.
// Bound by the matrix cores and the barriers between the layers: a 16 x 32 tile takes 21,000 cycles
// with 11,500 of products on the busiest SIMD (26,700 with one row per block, weights read by all
// waves with bank conflicts and waits behind the output's stores); a 1024^2 image 78-85 us (before
// 106), of which its 21 MB take 5.
constexpr int kFuTW = 32;
constexpr int kFuThreads = 512;
constexpr int kFuWaves = kFuThreads / 64;

template <int TH, int L>  // the region of layer L's output; L = 0 is the packed input
struct FuRegion {
    static constexpr int kHalo = 4 - L;
    static constexpr int kRows = TH + 2 * kHalo;
    static constexpr int kCols = kFuTW + 2 * kHalo;
    static constexpr int kPix = kRows * kCols;
    static constexpr int kStride = (L == 0 ? 32 : 64) + 16;  // bytes per pixel, 16 B aligned, spreads banks
    static constexpr int kBytes = kPix * kStride;
};
constexpr int kFuWSlot = 9 * 32 * 32 * 2;  // one layer's BF16 weights (the widest)

template <int TH>
struct FuLds {
    // buffer A holds layer 1's map, then layer 3's; buffer B the packed input, then layer 2's map
    static constexpr int kBufA = FuRegion<TH, 1>::kBytes;
    static constexpr int kBufB =
        FuRegion<TH, 0>::kBytes > FuRegion<TH, 2>::kBytes ? FuRegion<TH, 0>::kBytes : FuRegion<TH, 2>::kBytes;
    static_assert(FuRegion<TH, 3>::kBytes + 9 * 32 * 16 * 2 <= kBufA, "layer 3 map and layer 1 weights in buffer A");
    static constexpr int kBytes = kBufA + kBufB + 2 * kFuWSlot + 4 * 32 * 4;
};

typedef short i16x2 __attribute__((ext_vector_type(2)));

// ReLU of two packed BF16 values: a BF16 with its sign bit set is a negative 16-bit integer,
// so the signed maximum with 0 zeroes exactly the negative values (and -0). Rounding then
// clamping equals clamping then rounding, since rounding keeps the sign.
__device__ __forceinline__ uint32_t relu_bf2(uint32_t w) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(i16x2, w), (i16x2){0, 0}));
}

// The bias pattern of a lane (output channels 8 q + 4 half + e) as an accumulator value.
__device__ __forceinline__ f32x16 bias_pattern(const float* __restrict__ bias, int half) {
    f32x16 b;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) b[4 * q + e] = bias[8 * q + 4 * half + e];
    return b;
}

// Output of a block row: pixel (ry, rx) of the region, channels 8 q + 4 half + (0..3) of this lane.
template <int TH, int L, bool kLast>
__device__ __forceinline__ void fused_store(const f32x16& acc, unsigned char* __restrict__ out_lds,
                                            float* __restrict__ out_f, int ry, int rx, bool valid, int y0, int x0,
                                            int H, int W, int half) {
    using Out = FuRegion<TH, L>;
    const int gy = y0 - Out::kHalo + ry, gx = x0 - Out::kHalo + rx;
    const bool inside = valid && gy >= 0 && gy < H && gx >= 0 && gx < W;
    if constexpr (!kLast) {
        // A lane has 4 of every 8 channels; exchanging halves of the wave gives each lane all 8 of
        // every second group (half h: groups h and 2 + h), written 16 B at a time.
#pragma unroll
        for (int q = 0; q < 4; q += 2) {
            unsigned w[2][2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                unsigned x = relu_bf2(f2bf2(acc[4 * q + 2 * i], acc[4 * q + 2 * i + 1]));
                unsigned y = relu_bf2(f2bf2(acc[4 * q + 4 + 2 * i], acc[4 * q + 4 + 2 * i + 1]));
                const auto r = __builtin_amdgcn_permlane32_swap(x, y, false, false);
                w[0][i] = r[0];
                w[1][i] = r[1];
            }
            uint4 o = make_uint4(w[0][0], w[0][1], w[1][0], w[1][1]);
            if (!inside) o = make_uint4(0u, 0u, 0u, 0u);
            if (valid)
                *reinterpret_cast<uint4*>(out_lds + (ry * Out::kCols + rx) * Out::kStride + (q + half) * 16) = o;
        }
    } else {
        if (inside && half == 0) {
#pragma unroll
            for (int e = 0; e < 3; ++e) out_f[(size_t)e * H * W + (size_t)gy * W + gx] = acc[e];
        }
    }
}

// A operands of one layer from its LDS slot, where tap t's and 16-channel chunk kc's operands lie in
// lane order (16 B each), so a read touches every bank once.
template <int KIN>
__device__ __forceinline__ void fused_weights(bf16x8 (&a)[9][2], const unsigned char* __restrict__ slot, int lane) {
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int kc = 0; kc < KIN / 16; ++kc)
            a[t][kc] = *reinterpret_cast<const bf16x8*>(slot + ((t * (KIN / 16) + kc) * 64 + lane) * 16);
}

// One layer over its region: input map in_lds (region L - 1), output map out_lds (region L),
// or, for the last layer, channels 0..2 to the FP32 planes out_f [3][H][W]. A block is 32 columns
// of two rows (the region's row pairs end to end): input row i of its four feeds tap row i of the
// upper output row and tap row i - 1 of the lower one, so 24 operand reads serve 36 products
// (at 32 channels), in two independent chains, each in tap order. The next input row's operands
// (or the next block's first) are read while the current row's products run. The weights a are
// replaced by the next layer's (KNEXT channels, in next_slot) once the wave's last products are
// issued, beside its last stores.
template <int TH, int L, int KIN, bool kLast, int KNEXT>
__device__ __forceinline__ void fused_layer(const unsigned char* __restrict__ in_lds, unsigned char* __restrict__ out_lds,
                                            bf16x8 (&a)[9][2], const unsigned char* __restrict__ next_slot, const float* __restrict__ bias_lds,
                                            float* __restrict__ out_f, int y0, int x0, int H, int W, int wave,
                                            int half, int j) {
    using In = FuRegion<TH, L - 1>;
    using Out = FuRegion<TH, L>;
    constexpr int kK = KIN / 16;
    constexpr int kPairs = Out::kRows / 2 * Out::kCols;
    constexpr int kBlocks = (kPairs + 31) / 32;
    static_assert(Out::kRows % 2 == 0, "row pairs");
    const f32x16 bias = bias_pattern(bias_lds, half);
    bf16x8 b[2][3][kK];
    auto place = [&](int blk, int& ry, int& rx) {
        const int P = blk * 32 + j;
        const int Pc = P < kPairs ? P : kPairs - 1;  // the last block's spare lanes read a real pixel
        ry = 2 * (Pc / Out::kCols);
        rx = Pc % Out::kCols;
        return in_lds + (ry * In::kCols + rx) * In::kStride + half * 16;
    };
    auto read = [&](const unsigned char* base, int i) {
#pragma unroll
        for (int kx = 0; kx < 3; ++kx)
#pragma unroll
            for (int kc = 0; kc < kK; ++kc)
                b[i & 1][kx][kc] = *reinterpret_cast<const bf16x8*>(base + (i * In::kCols + kx) * In::kStride + kc * 32);
    };
    int ry, rx;
    const unsigned char* base = place(wave, ry, rx);
    read(base, 0);
    for (int blk = wave; blk < kBlocks; blk += kFuWaves) {
        f32x16 up = bias, low = bias;
        const int cy = ry, cx = rx;
        const bool valid = blk * 32 + j < kPairs;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (i < 3) {
                read(base, i + 1);
            } else if (blk + kFuWaves < kBlocks) {
                base = place(blk + kFuWaves, ry, rx);
                read(base, 0);
            }
#pragma unroll
            for (int kx = 0; kx < 3; ++kx)
#pragma unroll
                for (int kc = 0; kc < kK; ++kc) {
                    if (i < 3)
                        up = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[3 * (i < 3 ? i : 0) + kx][kc], b[i & 1][kx][kc], up, 0, 0, 0);
                    if (i > 0)
                        low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[3 * (i > 0 ? i - 1 : 0) + kx][kc], b[i & 1][kx][kc], low, 0, 0, 0);
                }
        }
        if (blk + kFuWaves >= kBlocks) {
            fused_weights<KNEXT>(a, next_slot, 32 * half + j);
            if constexpr (kLast) __builtin_amdgcn_s_waitcnt(0);  // the staged weights, before the stores
        }
        fused_store<TH, L, kLast>(up, out_lds, out_f, cy, cx, valid, y0, x0, H, W, half);
        fused_store<TH, L, kLast>(low, out_lds, out_f, cy + 1, cx, valid, y0, x0, H, W, half);
    }
    if (kBlocks < kFuWaves && wave >= kBlocks) {  // a wave without a block
        fused_weights<KNEXT>(a, next_slot, 32 * half + j);
        if constexpr (kLast) __builtin_amdgcn_s_waitcnt(0);  // the staged weights here too
    }
}

template <int TH>
__global__ __launch_bounds__(kFuThreads) void cnn_fused_kernel(RawIn raw, InputNorm nrm, FusedNet net,
                                                               float* __restrict__ out_f, int H, int W) {
    __shared__ __attribute__((aligned(16))) unsigned char lds[FuLds<TH>::kBytes];
    unsigned char* bufA = lds;
    unsigned char* bufB = lds + FuLds<TH>::kBufA;
    unsigned char* wslot[2] = {lds + FuLds<TH>::kBufA + FuLds<TH>::kBufB, lds + FuLds<TH>::kBufA + FuLds<TH>::kBufB + kFuWSlot};
    float* bias_lds = reinterpret_cast<float*>(lds + FuLds<TH>::kBufA + FuLds<TH>::kBufB + 2 * kFuWSlot);
    constexpr int kFuRawPer = (FuRegion<TH, 0>::kPix + kFuThreads - 1) / kFuThreads;  // input pixels per thread
    const int tiles_x = (W + kFuTW - 1) / kFuTW;
    const int total = tiles_x * ((H + TH - 1) / TH);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
    const int half = lane / 32, j = lane % 32;
    if (threadIdx.x < 128) bias_lds[threadIdx.x] = net.bias[threadIdx.x / 32][threadIdx.x % 32];

    // the packed input of a tile: raw values fetched into registers (a pixel outside the image reads
    // the first one, so that no load sits in a branch and all are in flight together), packed into
    // buffer B
    float rx_[kFuRawPer][4];
    unsigned rm_[kFuRawPer];
    auto raw_pixel = [&](int tile, int q, bool& in) -> unsigned {
        const int ty = tile / tiles_x, tx = tile - ty * tiles_x;
        const int e = threadIdx.x + q * kFuThreads;
        const int r = e / FuRegion<TH, 0>::kCols, c = e - r * FuRegion<TH, 0>::kCols;
        const int gy = ty * TH - FuRegion<TH, 0>::kHalo + r, gx = tx * kFuTW - FuRegion<TH, 0>::kHalo + c;
        in = e < FuRegion<TH, 0>::kPix && gy >= 0 && gy < H && gx >= 0 && gx < W;
        return in ? (unsigned)gy * (unsigned)W + (unsigned)gx : 0u;
    };
    auto fetch = [&](int tile) {
#pragma unroll
        for (int q = 0; q < kFuRawPer; ++q) {
            bool in;
            const unsigned p = raw_pixel(tile, q, in);
            rx_[q][0] = raw.eta[p];
            rx_[q][1] = raw.u[p];
            rx_[q][2] = raw.v[p];
            rx_[q][3] = raw.H[p];
            rm_[q] = raw.mask[p];
        }
    };
    auto commit = [&](int tile) {
#pragma unroll
        for (int q = 0; q < kFuRawPer; ++q) {
            const int e = threadIdx.x + q * kFuThreads;
            bool in;
            raw_pixel(tile, q, in);
            if (e < FuRegion<TH, 0>::kPix) {
                const float x[5] = {rx_[q][0], rx_[q][1], rx_[q][2], rx_[q][3], rm_[q] ? 1.f : 0.f};
                uint4 ca, cb;
                pack_values(x, 0, nrm, ca, cb);  // no noise at inference
                if (!in) ca = cb = make_uint4(0u, 0u, 0u, 0u);
                uint4* dst = reinterpret_cast<uint4*>(bufB + e * FuRegion<TH, 0>::kStride);
                dst[0] = ca;
                dst[1] = cb;
            }
        }
    };
    // The next layer's weights go from global memory straight into the free LDS slot while
    // the current layer runs, one tap and 16-channel chunk per wave and load (this lane: output
    // channel j, channels 8 half.. of the chunk); the wait and the barrier after the layer publish
    // them, and each wave then reads its A operands from LDS.
    auto wstage = [&](int layer, unsigned char* slot) {
        const int chunks = layer == 0 ? 1 : 2, kin = 16 * chunks;
        unsigned off = (unsigned)(j * kin + half * 8);
        asm volatile("" : "+v"(off));  // formed here, not kept across the layers as 64-bit addresses
#pragma unroll
        for (int q = 0; q < (18 + kFuWaves - 1) / kFuWaves; ++q) {
            const int g = q * kFuWaves + wave;  // wave-uniform: tap and chunk
            if (g < 9 * chunks) {
                const int t = g / chunks, kc = g - t * chunks;
                const uint16_t* group = net.wk[layer] + t * 32 * kin + kc * 16;  // wave-uniform
                __builtin_amdgcn_global_load_lds(group + off,
                                                 reinterpret_cast<uint4*>(slot) + g * 64, 16, 0, 0);
            }
        }
    };
    auto publish = [&]() {
        __builtin_amdgcn_s_waitcnt(0);  // this wave's copies (and loads) have landed
        __syncthreads();
    };

    // Staging: a layer's weights are in LDS, landed and published by a barrier, before the layer in
    // front of it ends (each wave reads them then); a slot is refilled once a barrier has passed since
    // its last read. Layers 2-4 take two slots in turn, whose roles swap from tile to tile; layer 1
    // has the tail of buffer A, free from layer 3 on. All copies land beside a long layer, and none
    // is waited for behind layer 4's stores.
    unsigned char* const s1 = bufA + FuRegion<TH, 3>::kBytes;
    bf16x8 w[9][2];
    wstage(0, s1);
    wstage(1, wslot[0]);
    wstage(2, wslot[1]);
    if ((int)blockIdx.x < total) {
        fetch(blockIdx.x);
        commit(blockIdx.x);
    }
    publish();
    fused_weights<16>(w, s1, lane);
    for (int tile = blockIdx.x; tile < total; tile += gridDim.x) {
        const int ty = tile / tiles_x, tx = tile - ty * tiles_x;
        const int y0 = ty * TH, x0 = tx * kFuTW;
        const int next = tile + (int)gridDim.x;
        __syncthreads();  // packed input, layer 2's and 3's weights in place; the last tile's layer 4 done
        fused_layer<TH, 1, 16, false, 32>(bufB, bufA, w, wslot[0], bias_lds, nullptr, y0, x0, H, W, wave, half, j);
        __syncthreads();
        wstage(3, wslot[0]);
        fetch(next < total ? next : tile);  // no branch: its loads stay in flight
        fused_layer<TH, 2, 32, false, 32>(bufA, bufB, w, wslot[1], bias_lds + 32, nullptr, y0, x0, H, W, wave, half, j);
        publish();
        wstage(0, s1);
        fused_layer<TH, 3, 32, false, 32>(bufB, bufA, w, wslot[0], bias_lds + 64, nullptr, y0, x0, H, W, wave, half, j);
        publish();
        wstage(1, wslot[1]);
        wstage(2, wslot[0]);
        // buffer B is free: layer 4 reads buffer A only. One half of the waves packs the next input
        // before its products, the other after, so the two share a SIMD's units.
        if (next < total && wave < kFuWaves / 2) commit(next);
        fused_layer<TH, 4, 32, true, 16>(bufA, nullptr, w, s1, bias_lds + 96, out_f, y0, x0, H, W, wave, half, j);
        if (next < total && wave >= kFuWaves / 2) commit(next);
        unsigned char* const t = wslot[0];
        wslot[0] = wslot[1];
        wslot[1] = t;
    }
}

// ------------------------------------------------------------------------------ training tiles
// The kernels of a training step walk kBwTH x kBwTW tiles, kBwThreads threads to a workgroup.
constexpr int kBwTH = 16, kBwTW = 32;
constexpr int kBwThreads = 512, kBwWaves = kBwThreads / 64;

// One map's tile with a rim of kRim pixels as a workgroup loads it, kChunks x 16 B per pixel: the 32
// inner columns a few rows at a time (all threads), then what rows are left and the rim's columns in
// one more load. A row's bytes times the tile's rows stay below kBwRange; wider images take other
// kernels.
constexpr unsigned kBwRange = 1u << 30;
constexpr int kBwWide = (kBwRange >> 6) / (kBwTH + 4);  // widest row of 64 B pixels

template <int kChunks, int kRim, int kStride>
struct BwMap {
    static constexpr int kRows = kBwTH + 2 * kRim, kCols = kBwTW + 2 * kRim;
    static constexpr int kStep = kBwThreads / (kBwTW * kChunks);  // rows per load
    static constexpr int kFull = kRows / kStep;
    static constexpr int kTail = kRows % kStep * kBwTW * kChunks, kSides = 2 * kRim * kRows * kChunks;
    static constexpr int kLoads = kFull + (kTail + kSides > 0 ? 1 : 0);
    static_assert(kTail + kSides <= kBwThreads, "one load for the rest");
    int row, col, lrow, lcol, ch;  // this thread's first pixel, and its last load's
    bool last;                     // it has one

    __device__ __forceinline__ explicit BwMap(int tid) {
        ch = tid % kChunks;
        row = tid / (kBwTW * kChunks);
        col = kRim + tid / kChunks % kBwTW;
        const int i = (tid - kTail) / kChunks, side = i / kRows;  // of the rim's columns
        const bool tail = tid < kTail;
        lrow = tail ? kFull * kStep + row : i % kRows;
        lcol = tail ? col : side < kRim ? side : kBwTW + side;
        last = tid < kTail + kSides;
    }

    // The tile at (y0, x0) of image img. Rows outside the image lie outside the buffer resource, and a
    // column outside it is given an offset there: both read zeros.
    __device__ __forceinline__ void fetch(const uint16_t* __restrict__ map, int img, int y0, int x0, int H, int W,
                                          u32x4 (&regs)[kLoads]) const {
        const int yb = max(y0 - kRim, 0), down = y0 - kRim - yb;  // < 0: the tile starts above the image
        const unsigned pitch = (unsigned)W * (16u * kChunks);
        const uint64_t left = (uint64_t)(H - yb) * pitch;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<uint16_t*>(map) + ((size_t)img * H + yb) * W * (8 * kChunks), 0,
            (int)(left < kBwRange ? (unsigned)left : kBwRange), 0x00020000);
        auto offset = [&](int r, int c) {
            const int gx = x0 - kRim + c;
            return (unsigned)gx < (unsigned)W ? (unsigned)(r + down) * pitch + (unsigned)(gx * kChunks + ch) * 16u
                                              : 2u * kBwRange;
        };
        const unsigned off = offset(row, col);
#pragma unroll
        for (int q = 0; q < kFull; ++q)
            regs[q] = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(off + (unsigned)(q * kStep) * pitch), 0, 0);
        if constexpr (kLoads > kFull)
            regs[kFull] = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)(last ? offset(lrow, lcol) : 2u * kBwRange), 0, 0);
    }
    __device__ __forceinline__ void commit(unsigned char* tile, const u32x4 (&regs)[kLoads]) const {
        unsigned char* const at = tile + (row * kCols + col) * kStride + ch * 16;
#pragma unroll
        for (int q = 0; q < kFull; ++q) *reinterpret_cast<u32x4*>(at + q * kStep * kCols * kStride) = regs[q];
        if constexpr (kLoads > kFull)
            if (last) *reinterpret_cast<u32x4*>(tile + (lrow * kCols + lcol) * kStride + ch * 16) = regs[kFull];
    }
};

// The tiles of a workgroup of a persistent grid. Workgroup b runs on XCD b % 8: each XCD walks a
// contiguous range of tiles, whose shared rims its L2 then holds.
struct BwWalk {
    int tiles_x, per_img, first, last, stride;
    __device__ __forceinline__ BwWalk(int nimg, int H, int W) {
        tiles_x = (W + kBwTW - 1) / kBwTW;
        per_img = tiles_x * ((H + kBwTH - 1) / kBwTH);
        const int total = per_img * nimg, groups = gridDim.x, xcd = blockIdx.x % kXcds;
        const int lead = min(groups, kXcds);  // XCDs in use
        stride = groups / kXcds + (xcd < groups % kXcds ? 1 : 0);
        first = (int)((int64_t)total * xcd / lead) + (int)blockIdx.x / kXcds;
        last = (int)((int64_t)total * (xcd + 1) / lead);
    }
    struct Place {
        int img, y0, x0;
    };
    __device__ __forceinline__ Place place(int tile) const {
        const int img = tile / per_img, t = tile - img * per_img;
        const int ty = t / tiles_x;
        return Place{img, ty * kBwTH, (t - ty * tiles_x) * kBwTW};
    }
};

// Two output rows of 32 pixels from an LDS map of kCols pixels per row: the lane's pixel of the upper
// row starts at base, kIn / 16 16-channel chunks each. Each output is a chain in tap order; an input
// row's operands serve both. weight(t, kc) is the A operand.
template <int KIN, int kCols, int kStride, typename Weight>
__device__ __forceinline__ void two_rows(const unsigned char* base, Weight&& weight, f32x16& up, f32x16& low) {
    constexpr int kK = KIN / 16;
    bf16x8 b[2][3][kK];
    auto read = [&](int i) {
#pragma unroll
        for (int kx = 0; kx < 3; ++kx)
#pragma unroll
            for (int kc = 0; kc < kK; ++kc)
                b[i & 1][kx][kc] = *reinterpret_cast<const bf16x8*>(base + (i * kCols + kx) * kStride + kc * 32);
    };
    read(0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (i < 3) read(i + 1);
#pragma unroll
        for (int kx = 0; kx < 3; ++kx)
#pragma unroll
            for (int kc = 0; kc < kK; ++kc) {
                if (i < 3)
                    up = __builtin_amdgcn_mfma_f32_32x32x16_bf16(weight(3 * (i < 3 ? i : 0) + kx, kc), b[i & 1][kx][kc],
                                                                 up, 0, 0, 0);
                if (i > 0)
                    low = __builtin_amdgcn_mfma_f32_32x32x16_bf16(weight(3 * (i > 0 ? i - 1 : 0) + kx, kc),
                                                                  b[i & 1][kx][kc], low, 0, 0, 0);
            }
    }
}

// 8 channels (group q + half of four) of a lane's pixel from an accumulator after the ReLU, as BF16: a
// lane holds 4 of every 8 channels, and exchanging halves of the wave completes one group of each two.
__device__ __forceinline__ u32x4 relu_group(const f32x16& acc, int q) {
    u32x2 w[2];
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int h = 0; h < 2; ++h)
            w[g][h] = f2bf2(fmaxf(acc[4 * (q + g) + 2 * h], 0.f), fmaxf(acc[4 * (q + g) + 2 * h + 1], 0.f));
    const auto r0 = __builtin_amdgcn_permlane32_swap(w[0][0], w[1][0], false, false);
    const auto r1 = __builtin_amdgcn_permlane32_swap(w[0][1], w[1][1], false, false);
    return (u32x4){r0[0], r1[0], r0[1], r1[1]};
}

// ------------------------------------------------------------------------------ forward pairs
// Two layers of the training forward in one pass over their input, both maps written for the backward:
// layers 1 and 2 (kFirst: 16 -> 32 -> 32 channels, ReLU) or 3 and 4 (32 -> 32, ReLU, -> 3 FP32 planes).
// The first of the two is computed over the tile and a rim of one pixel into LDS (pixels outside the
// image as the zero padding) and its tile's own pixels also to memory, so the second reads no map from
// there. Waves 0-3 take the first layer of a tile while waves 4-7 take the second of the tile before
// (one of each per SIMD, whose products and epilogues overlap), each with its layer's weights in
// registers. The next input tile is fetched meanwhile. Every output is bitwise that of conv3x3_kernel.
// 4 x 1024^2 pixels take 157 us for layers 1 and 2 (670 MB, 145 us at a large copy's rate) and 191 for
// 3 and 4 (586 MB, 127 us), a launch per layer 111 + 127 and 127 + 88. The barriers and the first
// layer's uneven blocks (10 for 4 waves) hold it: matrix cores are busy 47 % of the time, and fetching
// two tiles ahead changes nothing. All eight waves in one layer after the other took 174 and 193.
template <bool kFirst>
struct PairLds {
    static constexpr int kIn = kFirst ? 16 : 32;
    static constexpr int kInStride = kIn * 2 + 16, kMidStride = 64 + 16;
    using Map = BwMap<kIn / 8, 2, kInStride>;
    static constexpr int kMidRows = kBwTH + 2, kMidCols = kBwTW + 2;
    static constexpr int kInBytes = Map::kRows * Map::kCols * kInStride;
    static constexpr int kMidBytes = kMidRows * kMidCols * kMidStride;
};

template <bool kFirst>
__global__ __launch_bounds__(kBwThreads) void forward_pair_kernel(
    const uint16_t* __restrict__ in, const uint16_t* __restrict__ wa, const float* __restrict__ ba,
    const uint16_t* __restrict__ wb, const float* __restrict__ bb, uint16_t* __restrict__ mid_out,
    uint16_t* __restrict__ out_bf, float* __restrict__ out_f, int nimg, int H, int W) {
    using L = PairLds<kFirst>;
    using Map = typename L::Map;
    constexpr int kK = L::kIn / 16;
    __shared__ __attribute__((aligned(16))) unsigned char ins[L::kInBytes];
    __shared__ __attribute__((aligned(16))) unsigned char mids[2][L::kMidBytes];
    __shared__ float bias[2][32];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
    const int half = lane / 32, j = lane % 32;
    const BwWalk walk(nimg, H, W);
    const int first = walk.first, last = walk.last, stride = walk.stride;
    if (first >= last) return;

    u32x4 rin[Map::kLoads];
    auto thread = [&]() {  // the loads' places are formed where they are used, not kept in registers
        int t = threadIdx.x;
        asm volatile("" : "+v"(t));
        return t;
    };
    auto fetch = [&](int tile) {
        const BwWalk::Place p = walk.place(tile);
        Map(thread()).fetch(in, p.img, p.y0, p.x0, H, W, rin);
    };
    auto weights = [&](auto& a, const uint16_t* __restrict__ w, auto kin) {
        constexpr int kIn = kin.value;
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int kc = 0; kc < kIn / 16; ++kc)
                a[t][kc] = *reinterpret_cast<const bf16x8*>(w + ((size_t)t * 32 + j) * kIn + kc * 16 + half * 8);
        __builtin_amdgcn_s_waitcnt(0);  // here: else the loop would wait for them, and the next tile
    };
    if (threadIdx.x < 64) bias[threadIdx.x / 32][threadIdx.x % 32] = (threadIdx.x < 32 ? ba : bb)[threadIdx.x % 32];
    fetch(first);
    Map(thread()).commit(ins, rin);
    // Iteration i: the first layer of tile i into mids[i % 2], the second of tile i - 1 from the other.
    // Both roles pass two barriers per iteration and commit the next input between them and the next
    // iteration's first, in loops of their own, so that a wave waits for its loads alone, not its stores.
    if (wave < kBwWaves / 2) {
        bf16x8 a[9][kK];
        weights(a, wa, std::integral_constant<int, L::kIn>{});
        int buf = 0;
        for (int tile = first; tile < last; tile += stride, buf ^= 1) {
            const BwWalk::Place p = walk.place(tile);
            __syncthreads();
            if (tile + stride < last) fetch(tile + stride);
            // the row pairs of the tile with its rim, end to end, 32 pixels at a time
            constexpr int kPairs = L::kMidRows / 2 * L::kMidCols, kBlocks = (kPairs + 31) / 32;
#pragma unroll
            for (int blk0 = 0; blk0 < kBlocks; blk0 += kBwWaves / 2) {
                const int blk = blk0 + wave;
                if (blk >= kBlocks) break;  // wave-uniform
                const int P = blk * 32 + j;
                const bool valid = P < kPairs;
                const int Pc = valid ? P : kPairs - 1;  // the last block's spare lanes read a real pixel
                const int ry = 2 * (Pc / L::kMidCols), rx = Pc % L::kMidCols;
                f32x16 acc[2];
                acc[0] = acc[1] = bias_pattern(bias[0], half);
                two_rows<L::kIn, Map::kCols, L::kInStride>(ins + (ry * Map::kCols + rx) * L::kInStride + half * 16,
                                                           [&](int t, int kc) { return a[t][kc]; }, acc[0], acc[1]);
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int r = ry + i, gy = p.y0 - 1 + r, gx = p.x0 - 1 + rx;
                    const bool inside = ((unsigned)gy < (unsigned)H) & ((unsigned)gx < (unsigned)W);
                    const bool own = valid & inside & ((unsigned)(r - 1) < (unsigned)kBwTH) &
                                     ((unsigned)(rx - 1) < (unsigned)kBwTW);
                    u32x4* const to =
                        reinterpret_cast<u32x4*>(mid_out) + (((int64_t)p.img * H + gy) * W + gx) * 4 + half;
                    unsigned char* const at = mids[buf] + (r * L::kMidCols + rx) * L::kMidStride + half * 16;
#pragma unroll
                    for (int q = 0; q < 4; q += 2) {
                        u32x4 o = relu_group(acc[i], q);
                        if (own) to[q] = o;
                        if (!inside) o = (u32x4){0u, 0u, 0u, 0u};
                        if (valid) *reinterpret_cast<u32x4*>(at + q * 16) = o;
                    }
                }
            }
            __syncthreads();
            if (tile + stride < last) Map(thread()).commit(ins, rin);
        }
        __syncthreads();
    } else {
        bf16x8 a[9][2];
        weights(a, wb, std::integral_constant<int, 32>{});
        auto second = [&](int tile, const unsigned char* mid) {
            const BwWalk::Place p = walk.place(tile);
#pragma unroll
            for (int pair = 0; pair < 2; ++pair) {
                const int ry = 2 * (wave - kBwWaves / 2 + pair * (kBwWaves / 2));
                f32x16 acc[2];
                acc[0] = acc[1] = bias_pattern(bias[1], half);
                two_rows<32, L::kMidCols, L::kMidStride>(mid + (ry * L::kMidCols + j) * L::kMidStride + half * 16,
                                                         [&](int t, int kc) { return a[t][kc]; }, acc[0], acc[1]);
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int gy = p.y0 + ry + i, gx = p.x0 + j;
                    const bool inside = gy < H && gx < W;
                    if constexpr (kFirst) {
                        u32x4* const to =
                            reinterpret_cast<u32x4*>(out_bf) + (((int64_t)p.img * H + gy) * W + gx) * 4 + half;
#pragma unroll
                        for (int q = 0; q < 4; q += 2) {
                            const u32x4 o = relu_group(acc[i], q);
                            if (inside) to[q] = o;
                        }
                    } else if (inside && half == 0) {
#pragma unroll
                        for (int e = 0; e < 3; ++e)
                            out_f[((size_t)p.img * 3 + e) * H * W + (size_t)gy * W + gx] = acc[i][e];
                    }
                }
            }
        };
        int buf = 0;
        for (int tile = first; tile < last; tile += stride, buf ^= 1) {
            __syncthreads();
            if (tile + stride < last) fetch(tile + stride);
            if (tile > first) second(tile - stride, mids[buf ^ 1]);
            __syncthreads();
            if (tile + stride < last) Map(thread()).commit(ins, rin);
        }
        __syncthreads();
        second(first + (last - first - 1) / stride * stride, mids[buf ^ 1]);
    }
}

// ------------------------------------------------------------------------------ backward
// One layer's backward over its input map x and output gradient dY (both NHWC), each read once:
//   dW[t][o][c] = sum_p dY[p][o] x[p + off_t][c]   (MFMA, K = pixels),  db[o] = sum_p dY[p][o];
//   dX[p][c] = sum_t,o dY[p + off_t][o] Wd[t][c][o] where x[p][c] > 0   (kDgrad; K = channels).
// A workgroup walks kBwTH x kBwTW tiles. A tile of x (with its 1-pixel rim) and of dY (with the rim
// when the data gradient reads it) lies in LDS as it does in memory, a pixel's channels contiguous;
// the next tile is fetched into registers while the current one is multiplied. With kDgrad the
// workgroup's waves 0-3 take the data gradient and waves 4-7 the weight gradient (one of each per
// SIMD, 72 products each per tile), otherwise all eight the weight gradient.
//   * data gradient: blocks of 32 columns x 2 rows as in the fused forward (an operand of an input
//     row serves both output rows), each output a chain in tap order: bitwise the data gradient of
//     conv3x3_kernel;
//   * weight gradient: both operands are 8 consecutive pixels of one channel per lane, read by the
//     LDS transpose read (ds_read_b64_tr_b16: 16 lanes address 4 pixels x 16 channels, each receives
//     4 pixels of its channel). A row of x serves the dY rows above, at and below it. With 16 input
//     channels a product takes two taps (columns 0-15 the first, 16-31 the second).
// The last layer has three outputs: its dY may come with 4 channels per pixel (kDch = 4, 8 B in place
// of 64), which are laid into the LDS tile's pixels, whose other channels stay zero.
// Bound by memory: 805 MB for 4 x 1024^2 pixels of 32 + 32 channels, 174 us at a large copy's rate,
// take 205 us (the separate data and weight gradients 176 + 165, reading both maps twice); the last
// layer's thin dY 180, 16 input channels 96 (before 341 and 137). A thread's loads of a tile lie at
// fixed distances (BwMap), so that fetching and staging a tile takes a few vector instructions per
// load: with a division and a 64-bit address for each they took as long as the products (221 us).
// Each workgroup's partial [9][32][KIN] (and the bias partial [32]) goes to global memory.

__device__ const u32x4 kBwZeros = {0u, 0u, 0u, 0u};  // what a pixel outside the image reads

// A tile of a map with 4 channels (8 B) per pixel, one pixel per load.
template <int kRim, int kStride>
struct BwThinMap {
    static constexpr int kCols = kBwTW + 2 * kRim, kPix = (kBwTH + 2 * kRim) * kCols;
    static constexpr int kLoads = (kPix + kBwThreads - 1) / kBwThreads;
    int tid;
    __device__ __forceinline__ explicit BwThinMap(int t) : tid(t) {}
    __device__ __forceinline__ void fetch(const uint16_t* __restrict__ map, int img, int y0, int x0, int H, int W,
                                          u32x2 (&regs)[kLoads]) const {
        const int yb = max(y0 - kRim, 0), down = y0 - kRim - yb;
        const unsigned pitch = (unsigned)W * 8u;
        const uint64_t left = (uint64_t)(H - yb) * pitch;
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(map) + ((size_t)img * H + yb) * W * 4, 0,
                                              (int)(left < kBwRange ? (unsigned)left : kBwRange), 0x00020000);
#pragma unroll
        for (int q = 0; q < kLoads; ++q) {
            const int pix = tid + q * kBwThreads, r = pix / kCols, gx = x0 - kRim + pix % kCols;
            const bool in = (pix < kPix) & ((unsigned)gx < (unsigned)W);
            regs[q] = __builtin_amdgcn_raw_buffer_load_b64(
                rs, (int)(in ? (unsigned)(r + down) * pitch + (unsigned)gx * 8u : 2u * kBwRange), 0, 0);
        }
    }
    __device__ __forceinline__ void commit(unsigned char* tile, const u32x2 (&regs)[kLoads]) const {
#pragma unroll
        for (int q = 0; q < kLoads; ++q) {
            const int pix = tid + q * kBwThreads;
            if (pix < kPix) *reinterpret_cast<u32x2*>(tile + pix * kStride) = regs[q];
        }
    }
};

template <int KIN, bool kDgrad>
struct BwLds {
    static constexpr int kXStride = KIN * 2 + 16, kDStride = 64 + 16;  // bytes per pixel, spreads banks
    static constexpr int kXCols = kBwTW + 2, kXPix = (kBwTH + 2) * kXCols;
    static constexpr int kRim = kDgrad ? 1 : 0;
    static constexpr int kDCols = kBwTW + 2 * kRim, kDPix = (kBwTH + 2 * kRim) * kDCols;
    static constexpr int kXBytes = kXPix * kXStride, kDBytes = kDPix * kDStride;
    static constexpr int kAcc = KIN == 32 ? 9 : 5;  // 32 x 32 products of a wave
    static constexpr int kSum = kAcc * 32 * 32, kBias = kBwWaves * 64;  // floats
    static constexpr int kBytes = kXBytes + kDBytes + (kSum + kBias) * 4;
};

typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;

// 8 pixels of one channel per lane from the LDS map whose lane's pixel and channels start at src.
template <int kStride>
__device__ __forceinline__ bf16x8 read_transposed(const unsigned char* src) {
    const i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)src);
    const i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(src + 4 * kStride));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

template <int KIN, bool kDgrad, int kDch, bool kWide>
__global__ __launch_bounds__(kBwThreads) void backward_kernel(const uint16_t* __restrict__ x,
                                                              const uint16_t* __restrict__ dy,
                                                              const uint16_t* __restrict__ wd,
                                                              uint16_t* __restrict__ dx, int nimg, int H, int W,
                                                              float* __restrict__ part_w, float* __restrict__ part_b) {
    static_assert(KIN == 32 || (KIN == 16 && !kDgrad), "data gradients exist for 32-channel inputs only");
    using L = BwLds<KIN, kDgrad>;
    __shared__ __attribute__((aligned(16))) unsigned char lds[L::kBytes];
    unsigned char* const xs = lds;
    unsigned char* const ds = lds + L::kXBytes;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), lane = threadIdx.x % 64;
    const int half = lane / 32, j = lane % 32;

    const BwWalk walk(nimg, H, W);
    using Place = BwWalk::Place;
    const int first = walk.first, last = walk.last, stride = walk.stride;
    auto place = [&](int tile) { return walk.place(tile); };

    using XMap = BwMap<KIN / 8, 1, L::kXStride>;
    using DMap = std::conditional_t<kDch == 32, BwMap<4, L::kRim, L::kDStride>, BwThinMap<L::kRim, L::kDStride>>;
    // The items' places are formed where they are used: kept across the loop they would not fit the
    // registers beside the sums.
    auto thread = [&]() {
        int t = threadIdx.x;
        asm volatile("" : "+v"(t));
        return t;
    };
    // A wide image's chunk at a time: one that lies outside the image reads kBwZeros.
    auto each = [&](auto item, const uint16_t* map, const Place& p, auto chunks_c, auto rim_c, int e) {
        using Item = decltype(item);
        constexpr int kChunks = chunks_c.value, kRim = rim_c.value, kCols = kBwTW + 2 * kRim;
        const int pix = e / kChunks, ch = e % kChunks, r = pix / kCols, c = pix % kCols;
        const bool in = (r < kBwTH + 2 * kRim) & ((unsigned)(p.y0 - kRim + r) < (unsigned)H) &
                        ((unsigned)(p.x0 - kRim + c) < (unsigned)W);
        const Item* const base = reinterpret_cast<const Item*>(map) +
                                 (((int64_t)p.img * H + p.y0 - kRim) * W + p.x0 - kRim) * kChunks;
        const Item* const src = base + ((uint64_t)(unsigned)r * (unsigned)W * kChunks + (unsigned)(c * kChunks + ch));
        return *(in ? src : reinterpret_cast<const Item*>(&kBwZeros));
    };
    constexpr int kXWide = (L::kXPix * (KIN / 8) + kBwThreads - 1) / kBwThreads;
    constexpr int kDChunks = kDch == 32 ? 4 : 1, kDWide = (L::kDPix * kDChunks + kBwThreads - 1) / kBwThreads;
    u32x4 rx[kWide ? kXWide : XMap::kLoads];
    std::conditional_t<kDch == 32, u32x4, u32x2> rd[kWide ? kDWide : DMap::kLoads];
    auto fetch = [&](int tile) {
        const Place p = place(tile);
        const int tid = thread();
        constexpr std::integral_constant<int, KIN / 8> xchunks{};
        constexpr std::integral_constant<int, kDChunks> dchunks{};
        if constexpr (kWide) {
#pragma unroll
            for (int q = 0; q < kXWide; ++q)
                rx[q] = each(u32x4{}, x, p, xchunks, std::integral_constant<int, 1>{}, tid + q * kBwThreads);
        } else {
            XMap(tid).fetch(x, p.img, p.y0, p.x0, H, W, rx);
        }
        if constexpr (kWide) {
#pragma unroll
            for (int q = 0; q < kDWide; ++q)
                rd[q] = each(rd[0], dy, p, dchunks, std::integral_constant<int, L::kRim>{}, tid + q * kBwThreads);
        } else {
            DMap(tid).fetch(dy, p.img, p.y0, p.x0, H, W, rd);
        }
    };
    auto commit = [&]() {
        const int tid = thread();
        if constexpr (kWide) {
#pragma unroll
            for (int q = 0; q < kXWide; ++q) {
                const int e = tid + q * kBwThreads, pix = e / (KIN / 8);
                if (pix < L::kXPix) *reinterpret_cast<u32x4*>(xs + pix * L::kXStride + e % (KIN / 8) * 16) = rx[q];
            }
        } else {
            XMap(tid).commit(xs, rx);
        }
        if constexpr (kWide) {
#pragma unroll
            for (int q = 0; q < kDWide; ++q) {
                const int e = tid + q * kBwThreads, pix = e / kDChunks;
                if (pix < L::kDPix)
                    *reinterpret_cast<std::remove_reference_t<decltype(rd[0])>*>(ds + pix * L::kDStride +
                                                                                e % kDChunks * 16) = rd[q];
            }
        } else {
            DMap(tid).commit(ds, rd);
        }
    };

    constexpr int kWgradWaves = kDgrad ? kBwWaves / 2 : kBwWaves;
    // [kAcc][q][lane][e] as the accumulators lie: output 8 q + 4 (lane / 32) + e, column lane % 32
    float* const sums = reinterpret_cast<float*>(lds + L::kXBytes + L::kDBytes);
    float* const bsums = sums + L::kSum;                                          // [waves][64]
    for (int e = threadIdx.x; e < L::kSum + L::kBias; e += kBwThreads) sums[e] = 0.f;

    if constexpr (kDch < 32) {
        for (int e = threadIdx.x; e < L::kDPix * 4; e += kBwThreads)
            *reinterpret_cast<u32x4*>(ds + e / 4 * L::kDStride + e % 4 * 16) = (u32x4){0u, 0u, 0u, 0u};
        __syncthreads();
    }
    if (first < last) fetch(first);
    // Both roles pass the same barriers: one before and one after each commit, one before the sums
    // and one after each wave's turn. Each commits in its own loop, so that a wave waits for its
    // loads alone, not for its stores.
    if (kDgrad && wave < kBwWaves / 2) {
        bf16x8 a[9][2];
#pragma unroll
        for (int t = 0; t < 9; ++t)
#pragma unroll
            for (int kc = 0; kc < 2; ++kc)
                a[t][kc] = *reinterpret_cast<const bf16x8*>(wd + ((size_t)t * 32 + j) * 32 + kc * 16 + half * 8);
        __builtin_amdgcn_s_waitcnt(0);  // the weights: else the loop would wait for them, and the next tile
        for (int tile = first; tile < last; tile += stride) {
            __syncthreads();
            commit();
            __syncthreads();
            if (tile + stride < last) fetch(tile + stride);
            const Place p = place(tile);
            u32x4* const to = reinterpret_cast<u32x4*>(dx) + (((size_t)p.img * H + p.y0) * W + p.x0 + j) * 4 + half;
#pragma unroll
            for (int pair = 0; pair < 2; ++pair) {
                const int ry = 4 * wave + 2 * pair;
                f32x16 acc[2];
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[0][e] = acc[1][e] = 0.f;
                two_rows<32, L::kDCols, L::kDStride>(ds + (ry * L::kDCols + j) * L::kDStride + half * 16,
                                                     [&](int t, int kc) { return a[t][kc]; }, acc[0], acc[1]);
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const unsigned char* m = xs + ((ry + i + 1) * L::kXCols + j + 1) * L::kXStride + half * 8;
                    const bool in = p.y0 + ry + i < H && p.x0 + j < W;
#pragma unroll
                    for (int q = 0; q < 4; q += 2) {
                        unsigned w[2][2];  // [group q, q + 1][pair of channels]
#pragma unroll
                        for (int g = 0; g < 2; ++g) {
                            const uint2 mv = *reinterpret_cast<const uint2*>(m + (q + g) * 16);
                            const unsigned mw[2] = {mv.x, mv.y};
#pragma unroll
                            for (int h = 0; h < 2; ++h) {
                                const float lo = acc[i][4 * (q + g) + 2 * h], hi = acc[i][4 * (q + g) + 2 * h + 1];
                                w[g][h] = f2bf2(__uint_as_float(mw[h] << 16) > 0.f ? lo : 0.f,
                                                __uint_as_float(mw[h] & 0xffff0000u) > 0.f ? hi : 0.f);
                            }
                        }
                        // exchanging halves of the wave gives each lane all 8 channels of group q + half
                        const auto r0 = __builtin_amdgcn_permlane32_swap(w[0][0], w[1][0], false, false);
                        const auto r1 = __builtin_amdgcn_permlane32_swap(w[0][1], w[1][1], false, false);
                        if (in) to[(size_t)(ry + i) * W * 4 + q] = (u32x4){r0[0], r1[0], r0[1], r1[1]};
                    }
                }
            }
        }
        __syncthreads();
        for (int r = 0; r < kWgradWaves; ++r) __syncthreads();
    } else {
        constexpr int kRows = kBwTH / kWgradWaves;
        constexpr int kAcc = L::kAcc;
        const int turn = kDgrad ? wave - kBwWaves / 2 : wave, row0 = turn * kRows;
        // the lane's pixel and channels in a transpose read: 4 pixels x 16 channels per 16 lanes
        const int tp = 8 * half + lane % 16 / 4, tc = 4 * (lane % 4), upper = lane / 16 % 2;
        const unsigned char* const dbase =
            ds + ((row0 + L::kRim) * L::kDCols + tp + L::kRim) * L::kDStride + (16 * upper + tc) * 2;
        const unsigned char* const xbase =
            xs + (row0 * L::kXCols + tp) * L::kXStride + (KIN == 32 ? 16 * upper + tc : tc) * 2;
        f32x16 acc[kAcc];
#pragma unroll
        for (int t = 0; t < kAcc; ++t)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;
        float bsum = 0.f;  // this lane's channel and pixels
        auto read_d = [&](int d, int kb) {
            const bf16x8 av = read_transposed<L::kDStride>(dbase + (d * L::kDCols + 16 * kb) * L::kDStride);
            const u32x4 w = __builtin_bit_cast(u32x4, av);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                bsum += __uint_as_float(w[q] << 16);
                bsum += __uint_as_float(w[q] & 0xffff0000u);
            }
            return av;
        };
        // the wave's sums onto the workgroup's, 16 B per lane and access
        auto add_sums = [&]() {
            f32x4* const at = reinterpret_cast<f32x4*>(sums) + lane;
#pragma unroll
            for (int t = 0; t < kAcc; ++t) {
                f32x4 sum[4];  // a product's reads in flight together
#pragma unroll
                for (int q = 0; q < 4; ++q) sum[q] = at[(t * 4 + q) * 64];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) sum[q][e] += acc[t][4 * q + e];
                    at[(t * 4 + q) * 64] = sum[q];
                }
            }
            bsums[turn * 64 + lane] += bsum;
        };
        // A wave sums at most kChain pixels in one chain, whatever the image: each adds its sums in a tile of
        // its own, two after the wave's before it, whose barriers keep the additions apart and in a fixed
        // order. With one chain per launch the error grew with the image (dW against 64 bits, zero-mean
        // maps, 4 x 1024^2 and 16 x 1024^2 pixels: 2.5e-7 and 5.4e-7; so 1.6e-7 and 2.2e-7, with the
        // partials added in FP64); it costs 5 us of 128 per gradient of 4 x 1024^2, 0.9 % of a training step.
        constexpr int kChain = 1024, kPeriod = kChain / (kRows * kBwTW);
        static_assert(kPeriod == 2 * kWgradWaves, "a tile per wave and none beside it");
        int left = 2 * turn + 1;
        for (int tile = first; tile < last; tile += stride) {
            __syncthreads();
            commit();
            __syncthreads();
            if (tile + stride < last) fetch(tile + stride);
#pragma unroll
            for (int kb = 0; kb < kBwTW / 16; ++kb) {
                if constexpr (KIN == 32) {
                    bf16x8 av[kRows], b[2][3];
                    auto read_x = [&](int r) {
#pragma unroll
                        for (int kx = 0; kx < 3; ++kx)
                            b[r & 1][kx] =
                                read_transposed<L::kXStride>(xbase + (r * L::kXCols + 16 * kb + kx) * L::kXStride);
                    };
                    read_x(0);
#pragma unroll
                    for (int r = 0; r < kRows + 2; ++r) {  // rows of x from the one below row0 on
                        if (r < kRows) av[r < kRows ? r : 0] = read_d(r, kb);
                        if (r + 1 < kRows + 2) read_x(r + 1);
#pragma unroll
                        for (int ky = 0; ky < 3; ++ky) {
                            const int d = r - ky;
                            if (d < 0 || d >= kRows) continue;
#pragma unroll
                            for (int kx = 0; kx < 3; ++kx)
                                acc[3 * ky + kx] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                                    av[d < 0 || d >= kRows ? 0 : d], b[r & 1][kx], acc[3 * ky + kx], 0, 0, 0);
                        }
                    }
                } else {
#pragma unroll
                    for (int d = 0; d < kRows; ++d) {
                        const bf16x8 av = read_d(d, kb);
#pragma unroll
                        for (int q = 0; q < kAcc; ++q) {
                            const int t0 = 2 * q, t1 = q + 1 < kAcc ? 2 * q + 1 : t0;  // taps of the two halves
                            const int o0 = t0 / 3 * L::kXCols + t0 % 3, o1 = t1 / 3 * L::kXCols + t1 % 3;
                            const bf16x8 b = read_transposed<L::kXStride>(
                                xbase + (d * L::kXCols + 16 * kb + (upper ? o1 : o0)) * L::kXStride);
                            acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, b, acc[q], 0, 0, 0);
                        }
                    }
                }
            }
            if (--left == 0) {  // wave-uniform
                add_sums();
#pragma unroll
                for (int t = 0; t < kAcc; ++t)
#pragma unroll
                    for (int e = 0; e < 16; ++e) acc[t][e] = 0.f;
                bsum = 0.f;
                left = kPeriod;
            }
        }
        __syncthreads();
        // what is left, in wave order
#pragma unroll 1  // one copy of the code, in the instruction cache after the first wave's turn
        for (int r = 0; r < kWgradWaves; ++r) {
            if (r == turn) add_sums();
            __syncthreads();
        }
    }
    float* const out = part_w + (size_t)blockIdx.x * 9 * 32 * KIN;
    for (int e = threadIdx.x; e < 9 * 32 * KIN; e += kBwThreads) {
        const int t = e / (32 * KIN), o = e / KIN % 32, c = e % KIN;
        const int product = KIN == 32 ? t : t / 2, col = KIN == 32 ? c : t % 2 * 16 + c;
        out[e] = sums[((product * 4 + o / 8) * 64 + o / 4 % 2 * 32 + col) * 4 + o % 4];
    }
    if (threadIdx.x < 32) {
        float s = 0.f;
        for (int r = 0; r < kWgradWaves; ++r) s += bsums[r * 64 + threadIdx.x] + bsums[r * 64 + 32 + threadIdx.x];
        part_b[(size_t)blockIdx.x * 32 + threadIdx.x] = s;
    }
}

// dW[i] = sum over chunks of part[chunk][i] in FP64, in a fixed order: a workgroup takes 32
// weights, its 32 slices of 32 threads add the chunks k = slice (mod 32) in increasing k, and
// the 32 slice sums are added in slice order. Entries nw .. nw+31 are the bias.
constexpr int kRedW = 32, kRedSlices = 32;

__global__ __launch_bounds__(kRedW* kRedSlices) void wgrad_reduce_kernel(const float* __restrict__ part_w,
                                                                        const float* __restrict__ part_b,
                                                                        int chunks, int nw, float* __restrict__ dW,
                                                                        float* __restrict__ db) {
    __shared__ double red[kRedSlices][kRedW];
    const int w = threadIdx.x % kRedW, slice = threadIdx.x / kRedW;
    const int i = blockIdx.x * kRedW + w;
    double acc = 0.0;
    if (i < nw) {
#pragma unroll 8
        for (int k = slice; k < chunks; k += kRedSlices) acc += part_w[(size_t)k * nw + i];
    } else if (i < nw + 32) {
        for (int k = slice; k < chunks; k += kRedSlices) acc += part_b[(size_t)k * 32 + (i - nw)];
    }
    red[slice][w] = acc;
    __syncthreads();
    if (slice == 0) {
        double t = red[0][w];
#pragma unroll
        for (int q = 1; q < kRedSlices; ++q) t += red[q][w];
        if (i < nw)
            dW[i] = (float)t;
        else if (i < nw + 32)
            db[i - nw] = (float)t;
    }
}

// ------------------------------------------------------------------------------ mse_grad
// out, target: FP32 planes [img][3][H][W]; mask: coarse water mask [img][H][W].
// d_out (BF16 NHWC, kDch = 32 or 4 channels, 3.. zero) = 2 act (out - target) * inv_n;
// partial[block] = sum act (out - target)^2.
// Bound by memory: 4 x 1024^2 pixels take 29 us with 4 channels (138 MB). A lane takes a pixel; of
// the 64 B that 32 channels take, the wave writes 16 pixels at a time, four lanes to a pixel (1 KB
// contiguous per store). One lane writing its own pixel's four chunks, one pixel at a time and with
// 64-bit divisions, took 136 us (372 MB).
template <int kDch>
__global__ __launch_bounds__(256) void mse_grad_kernel(const float* __restrict__ out, const float* __restrict__ target,
                                                       const uint8_t* __restrict__ mask, int nimg, int H, int W,
                                                       float inv_n, float ts0, float ts1, float ts2,
                                                       uint16_t* __restrict__ d_out, double* __restrict__ partial) {
    const float tscale[3] = {ts0, ts1, ts2};
    __shared__ double lds[256];
    const unsigned plane = (unsigned)H * W, npix = nimg * plane;  // < 2^31
    const int lane = threadIdx.x % 64;
    double s = 0.0;
    // A wave takes 4 x 64 pixels at a time. No load depends on another, so that all are in flight
    // together; whole waves stay in the loop: their lanes write each other's pixels.
    constexpr int kPer = 4;
    for (unsigned q0 = (blockIdx.x * 256 + threadIdx.x - lane) * kPer; q0 < npix; q0 += gridDim.x * 256 * kPer) {
        float r[kPer][3];
        unsigned m[kPer][3];
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const unsigned q = min(q0 + 64 * k + lane, npix - 1);
            const unsigned img = q / plane, pin = q - img * plane;
            const int y = (int)(pin / W), x = (int)(pin - (unsigned)y * W);
            const uint8_t* const at = mask + (size_t)img * plane + pin;
            const bool east = x + 1 < W, north = y + 1 < H;
            m[k][0] = at[0];
            m[k][1] = at[east ? 1 : 0];
            m[k][2] = at[north ? W : 0];
            if (!east) m[k][1] = 0;
            if (!north) m[k][2] = 0;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const size_t f = ((size_t)img * 3 + c) * plane + pin;
                r[k][c] = out[f] - target[f] * tscale[c];
            }
        }
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const unsigned q = q0 + 64 * k + lane;
            uint16_t g[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const bool act = q < npix && m[k][0] != 0 && (c == 0 || m[k][c] != 0);
                const float e = act ? r[k][c] : 0.f;
                s += (double)e * (double)e;
                g[c] = f2bf(2.f * e * inv_n);
            }
            const uint2 o = make_uint2(g[0] | ((uint32_t)g[1] << 16), g[2]);
            if constexpr (kDch == 4) {
                if (q < npix) *reinterpret_cast<uint2*>(d_out + (size_t)q * 4) = o;
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int from = 16 * i + lane / 4;
                    const unsigned a = __shfl(o.x, from), b = __shfl(o.y, from);
                    const bool head = lane % 4 == 0;
                    const unsigned first = q0 + 64 * k + 16 * i;
                    if (first + lane / 4 < npix)
                        reinterpret_cast<uint4*>(d_out)[(size_t)first * 4 + lane] =
                            make_uint4(head ? a : 0u, head ? b : 0u, 0u, 0u);
                }
            }
        }
    }
    lds[threadIdx.x] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) lds[threadIdx.x] += lds[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = lds[0];
}

// Sum over a workgroup of 256 threads, in thread 0: by lane swaps in each wave, then over its four waves
// (a tree through LDS has eight barriers, and these kernels are little else).
__device__ __forceinline__ double group_sum(double s) {
    __shared__ double lds[4];
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (threadIdx.x % 64 == 0) lds[threadIdx.x / 64] = s;
    __syncthreads();
    return (lds[0] + lds[1]) + (lds[2] + lds[3]);
}

__global__ __launch_bounds__(256) void sum_partials_kernel(const double* __restrict__ partial, int n,
                                                           double* __restrict__ out) {
    double s = 0.0;
#pragma unroll 4
    for (int i = threadIdx.x; i < n; i += 256) s += partial[i];
    s = group_sum(s);
    if (threadIdx.x == 0) *out = s;
}

// ------------------------------------------------------------------------------ adam
// BF16 working copies of weight i of one layer: forward Wk[t][n][k] and data-gradient Wd[t'][k][n] with
// t' = 8 - t (flipped taps), from the FP32 master in forward layout [9][32][kin].
__device__ __forceinline__ void cast_weight(float w, int i, int kin, int dkin, uint16_t* __restrict__ wk,
                                            uint16_t* __restrict__ wd) {
    const int t = i / (32 * kin), rem = i - t * 32 * kin;
    const int n = rem / kin, k = rem - n * kin;
    const uint16_t b = f2bf(w);
    wk[i] = b;
    // data gradient: output channels are the forward input channels k (32 of them, kin
    // may be 16 or 32), reduced channels are the forward outputs n (dkin of them)
    if (wd && n < dkin) wd[((size_t)(8 - t) * 32 + k) * dkin + n] = b;
}

// With copies, each updated weight is also laid out for the next forward and backward pass: a launch
// of their own per layer would take longer than all of this kernel (four of 4.5 us beside 4.7 us).
__global__ __launch_bounds__(256) void adam_kernel(float* __restrict__ theta, const float* __restrict__ grad,
                                                   float* __restrict__ m, float* __restrict__ v, int n,
                                                   AdamHyper hp, NetCopies copies) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float g = grad[i];
    const float mi = hp.beta1 * m[i] + (1.f - hp.beta1) * g;
    const float vi = hp.beta2 * v[i] + (1.f - hp.beta2) * g * g;
    m[i] = mi;
    v[i] = vi;
    const float w = theta[i] - hp.lr * (mi * hp.inv_bc1) / (sqrtf(vi * hp.inv_bc2) + hp.eps);
    theta[i] = w;
#pragma unroll
    for (int l = 0; l < NetCopies::kMax; ++l) {
        const int at = i - copies.begin[l];
        if (l < copies.layers && at >= 0 && at < 9 * 32 * copies.cin[l])
            cast_weight(w, at, copies.cin[l], 32, copies.wk[l], copies.wd[l]);
    }
}

__global__ __launch_bounds__(256) void cast_weights_kernel(const float* __restrict__ master, int kin, int dkin,
                                                           uint16_t* __restrict__ wk, uint16_t* __restrict__ wd) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < 9 * 32 * kin) cast_weight(master[i], i, kin, dkin, wk, wd);
}

// ------------------------------------------------------------------------------ correct
__global__ __launch_bounds__(256) void correct_kernel(float* __restrict__ eta, float* __restrict__ u,
                                                      float* __restrict__ v, const float* __restrict__ out,
                                                      const uint8_t* __restrict__ mask, int H, int W, float s0,
                                                      float s1, float s2) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= H * W) return;
    const int y = p / W, x = p - y * W;
    const bool wet = mask[p] != 0;
    if (!wet) return;
    const size_t plane = (size_t)H * W;
    eta[p] = fmaf(s0, out[p], eta[p]);
    if (x + 1 < W && mask[p + 1]) u[p] = fmaf(s1, out[plane + p], u[p]);
    if (y + 1 < H && mask[p + W]) v[p] = fmaf(s2, out[2 * plane + p], v[p]);
}

// ------------------------------------------------------------------------------ rmse
// Four cells in a row of memory; the planes may begin at any cell.
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef uint8_t u8x4_any __attribute__((ext_vector_type(4), aligned(1)));

// Four cells per thread at a time, all loaded before the mask is looked at (1024^2: 6.0 -> 4.7 us).
__global__ __launch_bounds__(256) void sqdiff_kernel(const float* __restrict__ a, const float* __restrict__ b,
                                                     const uint8_t* __restrict__ mask, int n,
                                                     double* __restrict__ partial) {
    double s = 0.0;
    const int64_t groups = n / 4;
    const int64_t first = (int64_t)blockIdx.x * 256 + threadIdx.x, step = (int64_t)gridDim.x * 256;
    for (int64_t g = first; g < groups; g += step) {
        const u8x4_any m = *(const u8x4_any*)(mask + 4 * g);
        const f32x4_any x = *(const f32x4_any*)(a + 4 * g), y = *(const f32x4_any*)(b + 4 * g);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const double d = (double)x[i] - (double)y[i];
            s += m[i] ? d * d : 0.0;
        }
    }
    if (first < n - 4 * groups && mask[4 * groups + first]) {
        const double d = (double)a[4 * groups + first] - (double)b[4 * groups + first];
        s += d * d;
    }
    s = group_sum(s);
    if (threadIdx.x == 0) partial[blockIdx.x] = s;
}

// ------------------------------------------------------------------------------ sub3
// out[c][p] = a_c[p] - b_c[p] for the three fields (training target: fine ahead minus coarse).
__global__ __launch_bounds__(256) void sub3_kernel(const float* __restrict__ a0, const float* __restrict__ a1,
                                                   const float* __restrict__ a2, const float* __restrict__ b0,
                                                   const float* __restrict__ b1, const float* __restrict__ b2,
                                                   int n, float* __restrict__ out) {
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= n) return;
    out[p] = a0[p] - b0[p];
    out[(size_t)n + p] = a1[p] - b1[p];
    out[2 * (size_t)n + p] = a2[p] - b2[p];
}

// ------------------------------------------------------------------------------ moments
// partial[block] = (sum x, sum x^2) in double over entries with mask != 0 (all if no mask).
__global__ __launch_bounds__(256) void moments_kernel(const float* __restrict__ x, const uint8_t* __restrict__ mask,
                                                      int64_t n, double* __restrict__ partial) {
    __shared__ double l1[256], l2[256];
    double s1 = 0.0, s2 = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        if (!mask || mask[i]) {
            const double v = (double)x[i];
            s1 += v;
            s2 += v * v;
        }
    l1[threadIdx.x] = s1;
    l2[threadIdx.x] = s2;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) {
            l1[threadIdx.x] += l1[threadIdx.x + h];
            l2[threadIdx.x] += l2[threadIdx.x + h];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        partial[2 * blockIdx.x] = l1[0];
        partial[2 * blockIdx.x + 1] = l2[0];
    }
}

__global__ __launch_bounds__(256) void moments_final_kernel(const double* __restrict__ partial, int n,
                                                            double* __restrict__ out) {
    __shared__ double l1[256], l2[256];
    double s1 = 0.0, s2 = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) {
        s1 += partial[2 * i];
        s2 += partial[2 * i + 1];
    }
    l1[threadIdx.x] = s1;
    l2[threadIdx.x] = s2;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) {
            l1[threadIdx.x] += l1[threadIdx.x + h];
            l2[threadIdx.x] += l2[threadIdx.x + h];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        out[0] = l1[0];
        out[1] = l2[0];
    }
}

// ------------------------------------------------------------------------------ launchers
hipError_t launch_sub3(const float* a0, const float* a1, const float* a2, const float* b0, const float* b1,
                       const float* b2, int n, float* out, hipStream_t s) {
    hipLaunchKernelGGL(sub3_kernel, dim3((n + 255) / 256), dim3(256), 0, s, a0, a1, a2, b0, b1, b2, n, out);
    return hipGetLastError();
}

hipError_t launch_moments(const float* x, const uint8_t* mask, int64_t n, double* partial, int nblocks, double* out,
                          hipStream_t s) {
    hipLaunchKernelGGL(moments_kernel, dim3(nblocks), dim3(256), 0, s, x, mask, n, partial);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(moments_final_kernel, dim3(1), dim3(256), 0, s, partial, nblocks, out);
    return hipGetLastError();
}

hipError_t launch_restrict4(const float* eta, const float* u, const float* v, const float* H,
                            const uint8_t* mask, int NX, int NY, float* eta_c, float* u_c, float* v_c,
                            float* H_c, uint8_t* mask_c, hipStream_t s) {
    const int n = (NX / 4) * (NY / 4);
    hipLaunchKernelGGL(restrict4_kernel, dim3((n + 255) / 256), dim3(256), 0, s, eta, u, v, H, mask, NX, NY,
                       eta_c, u_c, v_c, H_c, mask_c);
    return hipGetLastError();
}

hipError_t launch_pack_input(const float* eta, const float* u, const float* v, const float* H,
                             const uint8_t* mask, int npix, const InputNorm& nrm, uint16_t* out,
                             hipStream_t s) {
    hipLaunchKernelGGL(pack_input_kernel, dim3((npix + 255) / 256), dim3(256), 0, s, eta, u, v, H, mask, npix, nrm,
                       out);
    return hipGetLastError();
}

// Workgroups of `kernel` the current device holds at once (CUs x occupancy), cached per
// device and kernel; 0 when the query fails.
int resident_groups(const void* kernel, int threads) {
    constexpr int kDevs = 16, kSlots = 32;
    static thread_local const void* keys[kDevs][kSlots] = {};
    static thread_local int vals[kDevs][kSlots] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kDevs) return 0;
    for (int i = 0; i < kSlots; ++i)
        if (keys[dev][i] == kernel) return vals[dev][i];
    int cus = 0, per_cu = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess) return 0;
    const int v = cus * (per_cu > 0 ? per_cu : 1);
    for (int i = 0; i < kSlots; ++i)
        if (!keys[dev][i]) {
            keys[dev][i] = kernel;
            vals[dev][i] = v;
            break;
        }
    return v;
}

hipError_t launch_conv3x3_raw(const RawIn& raw, const InputNorm& nrm, const uint16_t* Wk, const float* bias,
                              uint16_t* out_bf, int H, int W, hipStream_t s) {
    const int tiles = ((W + kConvTW - 1) / kConvTW) * ((H + kConvTH - 1) / kConvTH);
    const int cap = resident_groups(reinterpret_cast<const void*>(&conv3x3_kernel<16, kConvRelu, true>), kConvThreads);
    if (cap < 1) return hipErrorInvalidDeviceFunction;
    hipLaunchKernelGGL((conv3x3_kernel<16, kConvRelu, true>), dim3(tiles < cap ? tiles : cap), dim3(kConvThreads), 0, s,
                       nullptr, Wk, bias, out_bf, nullptr, nullptr, H, W, 1, raw, nrm, CorrectOut{});
    return hipGetLastError();
}

hipError_t launch_conv3x3_correct(const uint16_t* in, const uint16_t* Wk, const float* bias, const CorrectOut& co,
                                  int H, int W, hipStream_t s) {
    const int tiles = ((W + kConvTW - 1) / kConvTW) * ((H + kConvTH - 1) / kConvTH);
    const int cap = resident_groups(reinterpret_cast<const void*>(&conv3x3_kernel<32, kConvCorrect>), kConvThreads);
    if (cap < 1) return hipErrorInvalidDeviceFunction;
    hipLaunchKernelGGL((conv3x3_kernel<32, kConvCorrect>), dim3(tiles < cap ? tiles : cap), dim3(kConvThreads), 0, s,
                       in, Wk, bias, nullptr, nullptr, nullptr, H, W, 1, RawIn{}, InputNorm{}, co);
    return hipGetLastError();
}

// The tile height. A tile takes about as long as 10 rows and its own (a round of 256 workgroups, the
// whole corrected step around it: 23.5 us at 16 rows, 22.1 at 12, 21.4 at 10, 18.9 at 6), so higher
// tiles recompute less and lower ones serve images that leave CUs idle or a last round nearly empty
// (us per corrected step at 16, 12, 10 and 6 rows: 64^2 21.3, 20.6, 20.0, 19.0; 300 x 221 23.5, 22.1,
// 21.4, 26.7; 400^2 34.2, 31.9, 37.3, 41.0; 450^2 35.2, 40.3, 38.6, 48.0).
hipError_t launch_cnn_fused(const RawIn& raw, const InputNorm& nrm, const FusedNet& net, float* out_f, int H,
                            int W, hipStream_t s) {
    auto tiles = [&](int th) { return (int64_t)((W + kFuTW - 1) / kFuTW) * ((H + th - 1) / th); };
    auto go = [&](auto kernel, int th) {
        const int cap = resident_groups(reinterpret_cast<const void*>(kernel), kFuThreads);
        if (cap < 1) return hipErrorInvalidDeviceFunction;
        const int64_t n = tiles(th);
        hipLaunchKernelGGL(kernel, dim3(n < cap ? (int)n : cap), dim3(kFuThreads), 0, s, raw, nrm, net, out_f, H, W);
        return hipGetLastError();
    };
    int th = 0;
    int64_t least = 0;
    for (const int h : {16, 12, 10, 6}) {
        const int64_t cost = (tiles(h) + kCus - 1) / kCus * (h + 10);
        if (th == 0 || cost < least) {
            th = h;
            least = cost;
        }
    }
    if (th == 6) return go(&cnn_fused_kernel<6>, 6);
    if (th == 10) return go(&cnn_fused_kernel<10>, 10);
    if (th == 12) return go(&cnn_fused_kernel<12>, 12);
    return go(&cnn_fused_kernel<16>, 16);
}

hipError_t launch_conv3x3(int kin, int mode, const uint16_t* in, const uint16_t* Wk, const float* bias,
                          uint16_t* out_bf, float* out_f, const uint16_t* relu_src, int nimg, int H, int W,
                          hipStream_t s) {
    // A persistent grid of as many workgroups as the device holds at once: each loads the
    // weights once and walks tiles (measured faster than a second round of workgroups).
    const int tiles = ((W + kConvTW - 1) / kConvTW) * ((H + kConvTH - 1) / kConvTH) * nimg;
    const dim3 block(kConvThreads);
#define SW2D_CONV_CASE(K, M)                                                                          \
    if (kin == K && mode == M) {                                                                      \
        const int cap = resident_groups(reinterpret_cast<const void*>(&conv3x3_kernel<K, M>), kConvThreads); \
        if (cap < 1) return hipErrorInvalidDeviceFunction;                                            \
        const dim3 grid(tiles < cap ? tiles : cap);                                                   \
        hipLaunchKernelGGL((conv3x3_kernel<K, M>), grid, block, 0, s, in, Wk, bias, out_bf, out_f, relu_src, H, \
                           W, nimg, RawIn{}, InputNorm{}, CorrectOut{});                              \
        return hipGetLastError();                                                                      \
    }
    SW2D_CONV_CASE(16, kConvRelu)
    SW2D_CONV_CASE(32, kConvRelu)
    SW2D_CONV_CASE(32, kConvLinear3)
    SW2D_CONV_CASE(32, kConvDgradMask)
#undef SW2D_CONV_CASE
    return hipErrorInvalidValue;
}

bool forward_pairs_ok(int W) { return W <= kBwWide; }

hipError_t launch_forward_pairs(const uint16_t* x16, const FusedNet& net, uint16_t* const* acts, float* out, int nimg,
                                int H, int W, hipStream_t s) {
    const int64_t tiles = backward_tiles(nimg, H, W);
    auto go = [&](auto kernel, const uint16_t* in, int l, uint16_t* mid, uint16_t* out_bf, float* out_f) {
        const int cap = resident_groups(reinterpret_cast<const void*>(kernel), kBwThreads);
        if (cap < 1) return hipErrorInvalidDeviceFunction;
        hipLaunchKernelGGL(kernel, dim3(tiles < cap ? (int)tiles : cap), dim3(kBwThreads), 0, s, in, net.wk[l],
                           net.bias[l], net.wk[l + 1], net.bias[l + 1], mid, out_bf, out_f, nimg, H, W);
        return hipGetLastError();
    };
    const hipError_t e = go(&forward_pair_kernel<true>, x16, 0, acts[0], acts[1], nullptr);
    return e != hipSuccess ? e : go(&forward_pair_kernel<false>, acts[1], 2, acts[2], nullptr, out);
}

int64_t backward_tiles(int nimg, int H, int W) {
    return (int64_t)((W + kBwTW - 1) / kBwTW) * ((H + kBwTH - 1) / kBwTH) * nimg;
}

hipError_t launch_backward(int kin, const uint16_t* x, const uint16_t* dy, int dch, const uint16_t* wd, uint16_t* dx,
                           int nimg, int H, int W, float* part, int max_parts, float* dW, float* db, hipStream_t s) {
    if (max_parts < 1) return hipErrorInvalidValue;
    const int64_t tiles = backward_tiles(nimg, H, W);
    const int nw = 9 * 32 * kin;
    auto go = [&](auto kernel) {
        int groups = resident_groups(reinterpret_cast<const void*>(kernel), kBwThreads);
        if (groups < 1) return hipErrorInvalidDeviceFunction;
        if (groups > max_parts) groups = max_parts;
        if (groups > tiles) groups = (int)tiles;
        hipLaunchKernelGGL(kernel, dim3(groups), dim3(kBwThreads), 0, s, x, dy, wd, dx, nimg, H, W, part,
                           part + (size_t)groups * nw);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(wgrad_reduce_kernel, dim3((nw + 32 + kRedW - 1) / kRedW), dim3(kRedW * kRedSlices), 0, s,
                           part, part + (size_t)groups * nw, groups, nw, dW, db);
        return hipGetLastError();
    };
    const bool wide = W > kBwWide;
    if (dch == 4) {
        if (kin != 32 || !dx) return hipErrorInvalidValue;
        return wide ? go(&backward_kernel<32, true, 4, true>) : go(&backward_kernel<32, true, 4, false>);
    }
    if (kin == 16 && !dx)
        return wide ? go(&backward_kernel<16, false, 32, true>) : go(&backward_kernel<16, false, 32, false>);
    if (kin == 32 && dx)
        return wide ? go(&backward_kernel<32, true, 32, true>) : go(&backward_kernel<32, true, 32, false>);
    if (kin == 32)
        return wide ? go(&backward_kernel<32, false, 32, true>) : go(&backward_kernel<32, false, 32, false>);
    return hipErrorInvalidValue;
}

hipError_t launch_mse_grad(const float* out, const float* target, const uint8_t* mask, int nimg, int H, int W,
                           float inv_n, const float* tscale, uint16_t* d_out, int dch, double* partial, int nblocks,
                           double* loss, hipStream_t s) {
    hipLaunchKernelGGL((dch == 4 ? mse_grad_kernel<4> : mse_grad_kernel<32>), dim3(nblocks), dim3(256), 0, s, out,
                       target, mask, nimg, H, W, inv_n, tscale[0], tscale[1], tscale[2], d_out, partial);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(sum_partials_kernel, dim3(1), dim3(256), 0, s, partial, nblocks, loss);
    return hipGetLastError();
}

hipError_t launch_adam(float* theta, const float* grad, float* m, float* v, int n, const AdamHyper& hp,
                       const NetCopies& copies, hipStream_t s) {
    hipLaunchKernelGGL(adam_kernel, dim3((n + 255) / 256), dim3(256), 0, s, theta, grad, m, v, n, hp, copies);
    return hipGetLastError();
}

hipError_t launch_cast_weights(const float* master, int kin, int dkin, uint16_t* wk, uint16_t* wd, hipStream_t s) {
    const int n = 9 * 32 * kin;
    hipLaunchKernelGGL(cast_weights_kernel, dim3((n + 255) / 256), dim3(256), 0, s, master, kin, dkin, wk, wd);
    return hipGetLastError();
}

hipError_t launch_correct(float* eta, float* u, float* v, const float* out, const uint8_t* mask, int H, int W,
                          const float* t_std, hipStream_t s) {
    hipLaunchKernelGGL(correct_kernel, dim3((H * W + 255) / 256), dim3(256), 0, s, eta, u, v, out, mask, H, W,
                       t_std[0], t_std[1], t_std[2]);
    return hipGetLastError();
}

hipError_t launch_sqdiff(const float* a, const float* b, const uint8_t* mask, int n, double* partial, int nblocks,
                         double* out, hipStream_t s) {
    hipLaunchKernelGGL(sqdiff_kernel, dim3(nblocks), dim3(256), 0, s, a, b, mask, n, partial);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(sum_partials_kernel, dim3(1), dim3(256), 0, s, partial, nblocks, out);
    return hipGetLastError();
}

}  // namespace sur
}  // namespace sw2d
