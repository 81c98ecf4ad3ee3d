// sw2d_sor.hip - red-black successive over-relaxation for the pressure Poisson equation of
// the paper's second workload (Sect. 6.3: SOR takes most of its GPU time), with the residual
// of every iteration folded on the device.
//
// Arrays [nz][ny][nx] FP32; the outermost layer holds fixed (Dirichlet) values. One
// iteration = a sweep over the red cells ((i + j + k) even), then over the black ones; a
// cell becomes p + omega (g - p), g = (cx (pE + pW) + cy (pN + pS) + cz (pU + pD) - f) / d,
// d = 2 (cx + cy + cz), c_ = 1 / spacing^2.
//
// Layout: the solver works on the two colours stored apart (red and black arrays of
// [nz][ny][w] with w = ceil(nx / 2); cell (i, j, k) lives in its colour's array at i / 2), so a
// sweep reads one whole array of its own colour, the other colour's array and its own half of
// f, and writes its own array - 16 B per cell and iteration, no half-used cache lines. The
// split and the merge back to [nz][ny][nx] are one pass each per solve. A sweep thread owns one
// position of its colour per plane (threads run along the rows of a plane, so they coalesce
// across row ends) and takes 4 planes, all of its loads issued before the first is used (walked one
// after another, 8 planes cost 8 load latencies: a sweep of 300 x 300 x 90 took 13.5 us instead of
// 11.5; its 65 MB take 7.8 us at the rate of a large copy inside the cache). Small grids take both
// colours in one launch (sor_pair_kernel). The residual r = f - L p of
// the state after iteration m is folded without an extra pass: a black cell's neighbours
// are all red, so the black sweep of iteration m knows its residual right after the update;
// a red cell's residual needs the black values of iteration m, which the red sweep of
// iteration m + 1 reads before it overwrites the red cell. One residual-only pass per colour
// covers the initial black cells and the final red cells. One pass per iteration by walking planes
// (new red values of a tile and its ring in LDS) was slower at every size and is gone: 2311 us per
// solve of 300 x 300 x 90 against 1198, 1445 against 278 on 65 x 47 x 33. Workgroup partials (FP64 sum of
// r^2, max |r| as magnitude bits) are added per iteration in a fixed order.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <utility>

#include "sw2d_internal.h"

namespace sw2d {
namespace {

constexpr int kSorThreads = 256;
constexpr int kSorFoldThreads = 256;
enum SorMode { kSorUpdate = 0, kSorResidualOnly = 1 };

struct SorCoef {
    float cx, cy, cz, diag, inv_diag, omega;
};

struct alignas(16) SorPartial {
    double sum_r2;
    unsigned max_bits;
    unsigned pad;
};

struct SorGeometry {
    int nx, ny, nz, w, rows_q, planes, gx, gz, nblocks;  // w = ceil(nx / 2); rows_q = (ny - 2) w
};

// Grids of fewer positions than this take an iteration per launch (sor_pair_kernel), the others two
// sweeps of 4 planes per thread. A small grid costs a launch and one load latency, whatever a thread
// reads beside its own cells; a larger one is bound by the cache's rate and its requests (32 values per
// position against 16), and walking planes reads a z neighbour once for the three cells that use it (us per
// 50-iteration solve, best of 5 back to back, an iteration per launch and the sweeps: 65 x 47 x 33 198 and 379,
// 40 x 300 x 20 222 and 335, 128 x 128 x 64 (500,000 positions) 375 and 385, 160 x 120 x 60 (547,500) 402 and
// 414, 200 x 128 x 64 (781,000) 497 and 472, 300 x 300 x 90 1746 and 1232). 4 planes: fewer read more, more
// leave fewer threads and, but for some sizes, a larger part of the last group unused (sweeps of 2, 4 and 8
// planes: 200 x 128 x 64 498, 470 and 496, 200 x 180 x 70 592, 531 and 571, 201 x 150 x 97 636, 576 and 579,
// 300 x 300 x 50 792, 702 and 755, 300 x 300 x 90 1285, 1169 and 1158, 400 x 300 x 120 2086, 1917 and 1970).
constexpr int64_t kSorPairPositions = 5 << 17;
constexpr int sor_planes(int64_t positions) { return positions < kSorPairPositions ? 1 : 4; }

// Workgroups of one launch: its threads have to stay below 2^32 (the runtime cuts the count off there
// without an error). Long narrow columns (3 x 3 x 17,000,000 cells) take several launches.
constexpr int kSorGroups = 1 << 23;

// Tile b of n in an order that gives each XCD (workgroup b runs on XCD b % 8) a contiguous range.
__device__ __forceinline__ int sor_tile(int b, int n) {
    const int x = b % kXcds;
    return x * (n / kXcds) + min(x, n % kXcds) + b / kXcds;
}


SorGeometry sor_geometry(int nx, int ny, int nz) {
    SorGeometry g;
    g.nx = nx;
    g.ny = ny;
    g.nz = nz;
    g.w = (nx + 1) / 2;
    g.rows_q = (ny - 2) * g.w;
    g.planes = sor_planes((int64_t)g.rows_q * (nz - 2));
    g.gx = (g.rows_q + kSorThreads - 1) / kSorThreads;
    g.gz = (nz - 2 + g.planes - 1) / g.planes;
    g.nblocks = g.gx * g.gz;
    return g;
}

// Sum (FP64) and magnitude maximum over a workgroup of N threads in a fixed order, written by
// thread 0: half waves and 16-lane rows exchanged, four levels within the rows, the waves in order.
// The maximum is of the bits, so a NaN stays the largest.
template <int kCtrl>
__device__ __forceinline__ void sor_row_level(double& sum, unsigned& mx) {
    const unsigned long long b = __double_as_longlong(sum);
    const unsigned lo = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)b, kCtrl, 0xf, 0xf, true);
    const unsigned hi = (unsigned)__builtin_amdgcn_mov_dpp((int)(unsigned)(b >> 32), kCtrl, 0xf, 0xf, true);
    sum += __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
    mx = max(mx, (unsigned)__builtin_amdgcn_mov_dpp((int)mx, kCtrl, 0xf, 0xf, true));
}

template <int N>
__device__ __forceinline__ void sor_fold_group(double sum, unsigned mx, SorPartial* out) {
    __shared__ double s_sum[N / kWave];
    __shared__ unsigned s_max[N / kWave];
    for (int off = kWave / 2; off >= 16; off >>= 1) {
        sum += __shfl_xor(sum, off, kWave);
        mx = max(mx, (unsigned)__shfl_xor((int)mx, off, kWave));
    }
    sor_row_level<0xB1>(sum, mx);   // quad_perm [1, 0, 3, 2]
    sor_row_level<0x4E>(sum, mx);   // quad_perm [2, 3, 0, 1]
    sor_row_level<0x141>(sum, mx);  // row_half_mirror
    sor_row_level<0x140>(sum, mx);  // row_mirror
    __syncthreads();                // an earlier fold's values have been read
    if (threadIdx.x % kWave == 0) {
        s_sum[threadIdx.x / kWave] = sum;
        s_max[threadIdx.x / kWave] = mx;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = s_sum[0];
        unsigned m = s_max[0];
#pragma unroll
        for (int i = 1; i < N / kWave; ++i) {
            t += s_sum[i];
            m = max(m, s_max[i]);
        }
        *out = SorPartial{t, m, 0u};
    }
}

// [nz][ny][nx] -> the two colour arrays, for p (twice where a second pair is given) and f, a
// position (two adjacent cells) per thread.
__global__ __launch_bounds__(256) void sor_split_kernel(const float* __restrict__ p, const float* __restrict__ f,
                                                        float* __restrict__ red, float* __restrict__ black,
                                                        float* __restrict__ f_red, float* __restrict__ f_black,
                                                        float* __restrict__ red2, float* __restrict__ black2,
                                                        SorGeometry g, int first) {
    const int per = (g.ny * g.w + 255) / 256;  // workgroups per plane
    const int b = first + blockIdx.x, k = b / per, q = (b - k * per) * 256 + threadIdx.x;
    if (q >= g.ny * g.w) return;
    const int j = q / g.w, m = q - j * g.w;
    const size_t row = (size_t)k * g.ny + j;
    const size_t o = row * g.w + m, n = row * g.nx + 2 * m;
    const bool both = 2 * m + 1 < g.nx, odd = ((j + k) & 1) != 0;  // odd: the first cell is black
    const float p0 = p[n], p1 = both ? p[n + 1] : 0.f;
    const float f0 = f[n], f1 = both ? f[n + 1] : 0.f;
    if (both || !odd) {
        red[o] = odd ? p1 : p0;
        f_red[o] = odd ? f1 : f0;
        if (red2) red2[o] = odd ? p1 : p0;
    }
    if (both || odd) {
        black[o] = odd ? p0 : p1;
        f_black[o] = odd ? f0 : f1;
        if (black2) black2[o] = odd ? p0 : p1;
    }
}

// The colour arrays back into p.
__global__ __launch_bounds__(256) void sor_merge_kernel(float* __restrict__ p, const float* __restrict__ red,
                                                        const float* __restrict__ black, SorGeometry g, int first) {
    const int per = (g.ny * g.w + 255) / 256;  // workgroups per plane
    const int b = first + blockIdx.x, k = b / per, q = (b - k * per) * 256 + threadIdx.x;
    if (q >= g.ny * g.w) return;
    const int j = q / g.w, m = q - j * g.w;
    const size_t row = (size_t)k * g.ny + j;
    const size_t o = row * g.w + m, n = row * g.nx + 2 * m;
    const bool both = 2 * m + 1 < g.nx, odd = ((j + k) & 1) != 0;
    if (both || !odd) p[n + (odd ? 1 : 0)] = red[o];
    if (both || odd) p[n + (odd ? 0 : 1)] = black[o];
}

// One colour's sweep (or its residual alone). A thread owns position m of a row in P successive
// planes: its z neighbours are the other colour's values at m one plane down and up, and one of
// its x neighbours is the value at m itself, so P planes load P + 2 of those, and the outer x
// neighbour, two y neighbours, p and f of each. Every load is issued before the first is used.
template <int COLOR, int MODE, int P>
__global__ __launch_bounds__(kSorThreads) void sor_sweep_kernel(float* __restrict__ own,
                                                                const float* __restrict__ other,
                                                                const float* __restrict__ f_own, SorGeometry geo,
                                                                SorCoef c, SorPartial* __restrict__ part, int first) {
#pragma clang fp contract(off)
    const int nx = geo.nx, ny = geo.ny, nz = geo.nz, w = geo.w;
    const int tile = sor_tile(first + blockIdx.x, geo.nblocks);
    const int bz = tile / geo.gx, bx = tile - bz * geo.gx;
    const int q = bx * kSorThreads + threadIdx.x;
    const bool row_ok = q < geo.rows_q;
    const int qc = row_ok ? q : 0;
    const int jj = qc / w;
    const int m = qc - jj * w;
    const int j = 1 + jj;
    const int k0 = 1 + bz * P;
    const int planes = min(P, nz - 1 - k0);  // this workgroup's, 1..P
    const size_t plane = (size_t)ny * w;
    const size_t o0 = ((size_t)k0 * ny + j) * w + m;
    float z[P + 2], xo[P], yn[P], ys[P], pc[P], fc[P];
#pragma unroll
    for (int kk = 0; kk < P + 2; ++kk) z[kk] = other[o0 - plane + (size_t)min(kk, planes + 1) * plane];
#pragma unroll
    for (int kk = 0; kk < P; ++kk) {
        const size_t o = o0 + (size_t)min(kk, planes - 1) * plane;
        const int s = (COLOR + j + k0 + kk) & 1;  // i = s + 2 m has the sweep's colour
        xo[kk] = other[s ? o + 1 : o - 1];        // the outer x neighbour
        yn[kk] = other[o + w];
        ys[kk] = other[o - w];
        pc[kk] = own[o];
        fc[kk] = f_own[o];
    }
    double acc = 0.0;
    unsigned mx = 0u;
#pragma unroll
    for (int kk = 0; kk < P; ++kk) {
        const int s = (COLOR + j + k0 + kk) & 1;
        const int i = s + 2 * m;
        const float pE = s ? xo[kk] : z[kk + 1], pW = s ? z[kk + 1] : xo[kk];
        const float sx = pE + pW;
        const float sy = yn[kk] + ys[kk];
        const float sz = z[kk + 2] + z[kk];
        const float nb = fmaf(c.cz, sz, fmaf(c.cy, sy, c.cx * sx));
        const bool live = row_ok && kk < planes && i >= 1 && i <= nx - 2;
        float r = 0.f;
        if constexpr (MODE == kSorResidualOnly || COLOR == 0) r = fc[kk] - fmaf(-c.diag, pc[kk], nb);
        if constexpr (MODE == kSorUpdate) {
            const float g = (nb - fc[kk]) * c.inv_diag;
            const float pn = fmaf(c.omega, g - pc[kk], pc[kk]);
            if (live) own[o0 + (size_t)kk * plane] = pn;
            if constexpr (COLOR == 1) r = fc[kk] - fmaf(-c.diag, pn, nb);
        }
        r = live ? r : 0.f;
        acc += (double)r * (double)r;
        mx = max(mx, __float_as_uint(r) & 0x7fffffffu);
    }
    sor_fold_group<kSorThreads>(acc, mx, part + tile);
}

// One iteration, both colours, in one launch (small grids): a thread updates the red and the black cell of its
// position from the old arrays into the new ones. The black cell's six red neighbours are computed
// from the old black cells around them as their own threads compute them (19 black values, 6 red and 7
// right-hand sides, all loaded before the first is used), so a launch costs one load latency and
// neither waits for another thread nor exchanges anything: the state is bitwise that of the two sweeps.
__global__ __launch_bounds__(kSorThreads) void sor_pair_kernel(const float* __restrict__ R, const float* __restrict__ B,
                                                               const float* __restrict__ FR,
                                                               const float* __restrict__ FB, float* __restrict__ Rn,
                                                               float* __restrict__ Bn, SorGeometry geo, SorCoef c,
                                                               SorPartial* __restrict__ red_part,
                                                               SorPartial* __restrict__ black_part) {
#pragma clang fp contract(off)
    const int nx = geo.nx, ny = geo.ny, nz = geo.nz, w = geo.w;
    const int tile = sor_tile(blockIdx.x, geo.nblocks);
    const int bz = tile / geo.gx, bx = tile - bz * geo.gx;
    const int q = bx * kSorThreads + threadIdx.x;
    const bool row_ok = q < geo.rows_q;
    const int qc = row_ok ? q : 0;
    const int j = 1 + qc / w, m = qc - (j - 1) * w, k = 1 + bz;
    const int s = (j + k) & 1;      // the red cell is i = 2 m + s, the black one 2 m + 1 - s
    const int d = s ? -1 : 1;       // towards the black cell's outer red neighbour
    const int mf = min(max(m + d, 0), w - 1), mb = min(max(m - d, 0), w - 1);
    const size_t plane = (size_t)ny * w;
    const int jn2 = min(j + 2, ny - 1), js2 = max(j - 2, 0), ku2 = min(k + 2, nz - 1), kd2 = max(k - 2, 0);
    const size_t row = (size_t)k * plane + (size_t)j * w, o = row + m, of = row + mf;
    const size_t on = o + w, os = o - w, ou = o + plane, od = o - plane;
    // black: own, the position ahead and behind, the rows and planes around, and around those
    const float b = B[o], bf = B[of], bb = B[row + mb];
    const float bn = B[on], bs = B[os], bu = B[ou], bd = B[od];
    const float bfn = B[of + w], bfs = B[of - w], bfu = B[of + plane], bfd = B[of - plane];
    const float bn2 = B[(size_t)k * plane + (size_t)jn2 * w + m], bs2 = B[(size_t)k * plane + (size_t)js2 * w + m];
    const float bu2 = B[(size_t)ku2 * plane + (size_t)j * w + m], bd2 = B[(size_t)kd2 * plane + (size_t)j * w + m];
    const float bnu = B[on + plane], bnd = B[on - plane], bsu = B[os + plane], bsd = B[os - plane];
    const float r = R[o], rf = R[of], rn = R[on], rs = R[os], ru = R[ou], rd = R[od];
    const float fr = FR[o], ff = FR[of], fn = FR[on], fs = FR[os], fu = FR[ou], fd = FR[od], fb = FB[o];
    auto around = [&](float sx, float sy, float sz) { return fmaf(c.cz, sz, fmaf(c.cy, sy, c.cx * sx)); };
    auto update = [&](float nb, float f, float pc) {
        const float g = (nb - f) * c.inv_diag;
        return fmaf(c.omega, g - pc, pc);
    };
    // new red values; a cell of the boundary layer keeps its own
    const int ir = 2 * m + s, ib = 2 * m + 1 - s, inner = nx - 2;
    const float nb_r = around(b + bb, bn + bs, bu + bd);
    const bool red_in = ir >= 1 && ir <= inner;
    const float r_new = red_in ? update(nb_r, fr, r) : r;
    const int i_f = ir + 2 * d;  // the red cell ahead
    const float f_new = i_f >= 1 && i_f <= inner ? update(around(bf + b, bfn + bfs, bfu + bfd), ff, rf) : rf;
    // the red cells of the rows and planes around lie at the black cell's i
    const bool col = ib >= 1 && ib <= inner;
    const float n_new = col && j + 1 <= ny - 2 ? update(around(bn + bfn, bn2 + b, bnu + bnd), fn, rn) : rn;
    const float s_new = col && j - 1 >= 1 ? update(around(bs + bfs, b + bs2, bsu + bsd), fs, rs) : rs;
    const float u_new = col && k + 1 <= nz - 2 ? update(around(bu + bfu, bnu + bsu, bu2 + b), fu, ru) : ru;
    const float d_new = col && k - 1 >= 1 ? update(around(bd + bfd, bnd + bsd, b + bd2), fd, rd) : rd;
    const float nb_b = around(r_new + f_new, n_new + s_new, u_new + d_new);
    const float b_new = update(nb_b, fb, b);
    const bool live_r = row_ok && red_in, live_b = row_ok && col;
    if (live_r) Rn[o] = r_new;
    if (live_b) Bn[o] = b_new;
    const float res_r = live_r ? fr - fmaf(-c.diag, r, nb_r) : 0.f;       // of the state before
    const float res_b = live_b ? fb - fmaf(-c.diag, b_new, nb_b) : 0.f;   // of the new one
    sor_fold_group<kSorThreads>((double)res_r * (double)res_r, __float_as_uint(res_r) & 0x7fffffffu, red_part + tile);
    sor_fold_group<kSorThreads>((double)res_b * (double)res_b, __float_as_uint(res_b) & 0x7fffffffu, black_part + tile);
}

// Residual of state m = red partials of slot m + black partials of slot m, each added in
// block order by a fixed tree; one workgroup per m.
__global__ __launch_bounds__(kSorFoldThreads) void sor_fold_kernel(const SorPartial* __restrict__ red,
                                                                   const SorPartial* __restrict__ black,
                                                                   int nblocks, sw2d_sor_res* __restrict__ out) {
    __shared__ double s_sum[kSorFoldThreads];
    __shared__ unsigned s_max[kSorFoldThreads];
    const int m = blockIdx.x, t = threadIdx.x;
    const SorPartial* slots[2] = {red + (size_t)m * nblocks, black + (size_t)m * nblocks};
    double acc = 0.0;
    unsigned mx = 0u;
    for (int c = 0; c < 2; ++c)
        for (int b = t; b < nblocks; b += kSorFoldThreads) {
            acc += slots[c][b].sum_r2;
            mx = max(mx, slots[c][b].max_bits);
        }
    s_sum[t] = acc;
    s_max[t] = mx;
    __syncthreads();
    for (int h = kSorFoldThreads / 2; h > 0; h >>= 1) {
        if (t < h) {
            s_sum[t] += s_sum[t + h];
            s_max[t] = max(s_max[t], s_max[t + h]);
        }
        __syncthreads();
    }
    if (t == 0) {
        out[m].iter = m;
        out[m].max_abs_r = __uint_as_float(s_max[0]);
        out[m].sum_r2 = s_sum[0];
    }
}

thread_local char g_sor_msg[256] = "";

int sor_fail(hipError_t e, const char* what) {
    if (e == hipSuccess) return SW2D_OK;
    std::snprintf(g_sor_msg, sizeof g_sor_msg, "%s: %s", what, hipGetErrorString(e));
    detail::set_hip_message(g_sor_msg);
    return SW2D_EHIP;
}

bool sor_params_ok(const sw2d_sor_params* p) {
    if (!p) return false;
    if (p->nx < 3 || p->ny < 3 || p->nz < 3) return false;
    if ((int64_t)p->nx * p->ny * p->nz >= ((int64_t)1 << 31)) return false;
    for (double h : {p->dx, p->dy, p->dz})
        if (!(h > 0.0) || !std::isfinite(h)) return false;
    return p->omega > 0.0 && p->omega < 2.0 && (p->fused == 0 || p->fused == 1);
}

// n workgroups of 256 threads in launches of at most kSorGroups; each gets its first one's number.
template <typename Kernel, typename... Args>
hipError_t launch_groups(Kernel kernel, int n, hipStream_t s, Args... args) {
    for (int first = 0; first < n; first += kSorGroups) {
        const int groups = n - first < kSorGroups ? n - first : kSorGroups;
        hipLaunchKernelGGL(kernel, dim3(groups), dim3(256), 0, s, args..., first);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int COLOR, int MODE>
hipError_t launch_sweep(float* own, const float* other, const float* f_own, const SorGeometry& g, const SorCoef& c,
                        SorPartial* part, hipStream_t s) {
    static_assert(kSorThreads == 256, "launch_groups");
    if (g.planes == 4) return launch_groups(sor_sweep_kernel<COLOR, MODE, 4>, g.nblocks, s, own, other, f_own, g, c, part);
    if constexpr (MODE == kSorResidualOnly)  // small grids update both colours in one launch
        return launch_groups(sor_sweep_kernel<COLOR, MODE, 1>, g.nblocks, s, own, other, f_own, g, c, part);
    return hipErrorInvalidValue;
}

int split_groups(const SorGeometry& g) { return (g.ny * g.w + 255) / 256 * g.nz; }

hipError_t launch_split(const float* p, const float* f, float* red, float* black, float* f_red, float* f_black,
                        float* red2, float* black2, const SorGeometry& g, hipStream_t s) {
    return launch_groups(sor_split_kernel, split_groups(g), s, p, f, red, black, f_red, f_black, red2, black2, g);
}

hipError_t launch_merge(float* p, const float* red, const float* black, const SorGeometry& g, hipStream_t s) {
    return launch_groups(sor_merge_kernel, split_groups(g), s, p, red, black, g);
}

size_t colour_floats(const SorGeometry& g) { return (size_t)g.nz * g.ny * g.w; }

}  // namespace
}  // namespace sw2d

using namespace sw2d;

extern "C" {

size_t sw2d_sor_workspace_bytes(const sw2d_sor_params* p, int32_t iters) {
    if (!sor_params_ok(p) || iters < 0) return 0;
    const SorGeometry g = sor_geometry(p->nx, p->ny, p->nz);
    // red, black, f red, f black (and a second red and black where an iteration is one launch; 256 B aligned
    // each), then the residual partials: iters + 1 slots per colour
    const size_t arr = (colour_floats(g) * sizeof(float) + 255) / 256 * 256;
    return (g.planes == 1 ? 6 : 4) * arr + 2 * (size_t)(iters + 1) * g.nblocks * sizeof(SorPartial);
}

int sw2d_sor_run(const sw2d_sor_params* p, float* d_p, const float* d_f, int32_t iters, sw2d_sor_res* d_res,
                 void* d_work, size_t work_bytes, void* stream) {
    if (!sor_params_ok(p) || !d_p || !d_f || iters < 0 || !d_work) return SW2D_EINVAL;
    if (work_bytes < sw2d_sor_workspace_bytes(p, iters)) return SW2D_ENOSPC;
    const SorGeometry g = sor_geometry(p->nx, p->ny, p->nz);
    SorCoef c;
    const double cx = 1.0 / (p->dx * p->dx), cy = 1.0 / (p->dy * p->dy), cz = 1.0 / (p->dz * p->dz);
    c.cx = (float)cx;
    c.cy = (float)cy;
    c.cz = (float)cz;
    c.diag = (float)(2.0 * (cx + cy + cz));
    c.inv_diag = (float)(1.0 / (2.0 * (cx + cy + cz)));
    c.omega = (float)p->omega;
    const size_t arr = (colour_floats(g) * sizeof(float) + 255) / 256 * 256;
    char* base = static_cast<char*>(d_work);
    float* R = reinterpret_cast<float*>(base);
    float* B = reinterpret_cast<float*>(base + arr);
    float* FR = reinterpret_cast<float*>(base + 2 * arr);
    float* FB = reinterpret_cast<float*>(base + 3 * arr);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const bool pairs = g.planes == 1;
    float* R2 = pairs ? reinterpret_cast<float*>(base + 4 * arr) : nullptr;
    float* B2 = pairs ? reinterpret_cast<float*>(base + 5 * arr) : nullptr;
    auto* red = reinterpret_cast<SorPartial*>(base + (pairs ? 6 : 4) * arr);
    SorPartial* black = red + (size_t)(iters + 1) * g.nblocks;
    // both pairs start as the split state: the boundary layer is never written again
    hipError_t e = launch_split(d_p, d_f, R, B, FR, FB, R2, B2, g, s);
    if (e == hipSuccess) e = launch_sweep<1, kSorResidualOnly>(B, R, FB, g, c, black, s);  // black part of state 0
    for (int32_t n = 0; n < iters && e == hipSuccess; ++n) {
        if (pairs) {
            hipLaunchKernelGGL(sor_pair_kernel, dim3(g.nblocks), dim3(kSorThreads), 0, s, R, B, FR, FB, R2, B2, g, c,
                               red + (size_t)n * g.nblocks, black + (size_t)(n + 1) * g.nblocks);
            e = hipGetLastError();
            std::swap(R, R2);
            std::swap(B, B2);
            continue;
        }
        e = launch_sweep<0, kSorUpdate>(R, B, FR, g, c, red + (size_t)n * g.nblocks, s);
        if (e == hipSuccess) e = launch_sweep<1, kSorUpdate>(B, R, FB, g, c, black + (size_t)(n + 1) * g.nblocks, s);
    }
    if (e == hipSuccess) e = launch_sweep<0, kSorResidualOnly>(R, B, FR, g, c, red + (size_t)iters * g.nblocks, s);
    if (e == hipSuccess) e = launch_merge(d_p, R, B, g, s);
    if (e == hipSuccess && d_res) {
        hipLaunchKernelGGL(sor_fold_kernel, dim3(iters + 1), dim3(kSorFoldThreads), 0, s, red, black, g.nblocks,
                           d_res);
        e = hipGetLastError();
    }
    return sor_fail(e, "sw2d_sor_run");
}

}  // extern "C"
