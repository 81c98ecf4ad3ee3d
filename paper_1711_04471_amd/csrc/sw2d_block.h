// sw2d_block.h - K time steps of one register tile (plain model).
//
// A workgroup of W waves holds a tile of W * R rows x 128 columns in registers: wave w the R
// rows from w R on, lane l the columns 2l and 2l + 1 of the tile ("a" and "b"). The tile is read once, stepped K times in place and its owned cells written
// once. East/west neighbours are the lane's other column and one lane exchange; the rows
// beyond a wave's own go through LDS, two rows of one field per wave and exchange: the surface
// (and v of the row below) before the predictor, the predicted surface before the filter. A
// step spoils two cells on each open side of the tile, so 2K columns and rows next to a
// neighbouring tile are not owned; sides on the grid's edge lose nothing (off-grid cells read
// 0, which is land).
//
// Against the row pipelines this needs no lagged rows: the activity masks of a cell's faces
// are taken once per pass and kept as lane masks, each flux and each surface difference of the
// filter is formed once per face, and all rows of a tile advance at once, so a pass costs one
// load latency instead of one per row. The formulas and the order of every sum are those of
// sw2d_tile.h: the filter adds (es_E - es) + (es_W - es) + (es_N - es) + (es_S - es) in that
// order, here as ((dE - dW) + dN) - dS with dW, dS the neighbours' dE, dN (an exact negation),
// so the state is bitwise that of the row pipelines.
//
// What bounds a pass: the vector issue of a CU's tiles (33 vector instructions per cell and step
// against the two-column row pipeline's 49; a tile of 40 rows takes about 1.4 us per step
// wherever it runs) plus 4 us for the launch, the loads and the stores. Measured per step, the
// default handle's streamed single step before and the tiles now: 66^2 7.0 and 2.1 us (200
// steps a call), 2048^2 22.8 and 10.8 us (50 a call: 388,000 Mcell-steps/s; 117 MB from the
// cache take 14.5 us at a large copy's rate there, so several steps per pass are what beats it).
#pragma once

#include "sw2d_tile.h"

namespace sw2d {

constexpr int kBlockCols = 2 * kWave;

// Rows exchanged between the waves of a tile: row w + 1 of an array is wave w's, rows 0 and
// W + 1 stay 0 (beyond the tile: land).
template <int W>
struct BlockShared {
    float2 top_e[W + 2][kWave], top_v[W + 2][kWave], bot_e[W + 2][kWave];
    float2 top_s[W + 2][kWave], bot_s[W + 2][kWave];
};

// Row accesses of a column pair, 8 bytes whatever the row's alignment (multi-dword buffer accesses
// need dword alignment only). An odd nx leaves the last pair astride the row end: its load takes
// the first cell of the next row as column b, which is land (depth 0) as every border cell is,
// and its store writes column a alone. In the grid's last row that pair may read zeros: land too.
struct BlockIO {
    int nx, ny;
    unsigned off;   // byte offset of column a
    unsigned row_bytes;
    bool odd;

    __device__ __forceinline__ BlockIO(int nx_, int ny_, int c0)
        : nx(nx_), ny(ny_), off((unsigned)c0 * 4u), row_bytes((unsigned)nx_ * 4u), odd((nx_ & 1) != 0) {}

    __device__ __forceinline__ void load(const float* __restrict__ p, int r, float (&x)[2]) const {
        const bool in = r >= 0 && r < ny;
        const unsigned bytes = in ? row_bytes + (odd && r + 1 < ny ? 4u : 0u) : 0u;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<float*>(p + (ptrdiff_t)(in ? r : 0) * nx), 0, (int)bytes, kRsrcWord3);
        const auto q = __builtin_amdgcn_raw_buffer_load_b64(rs, (int)off, 0, 0);
        x[0] = __uint_as_float(q[0]);
        x[1] = __uint_as_float(q[1]);
    }
    // r: a row of the grid; owned: this lane's pair is written
    __device__ __forceinline__ void store(float* __restrict__ p, int r, bool owned, const float (&x)[2]) const {
        const __amdgpu_buffer_rsrc_t rs =
            __builtin_amdgcn_make_buffer_rsrc(p + (ptrdiff_t)r * nx, 0, (int)row_bytes, kRsrcWord3);
        __attribute__((ext_vector_type(2))) unsigned q;
        q[0] = __float_as_uint(x[0]);
        q[1] = __float_as_uint(x[1]);
        __builtin_amdgcn_raw_buffer_store_b64(q, rs, (int)(owned && off + 4u < row_bytes ? off : kNoLane), 0, 0);
        if (odd)  // wave-uniform
            __builtin_amdgcn_raw_buffer_store_b32(q[0], rs, (int)(owned && off + 4u == row_bytes ? off : kNoLane), 0, 0);
    }
};

// This lane's bit of a lane mask held in scalar registers.
__device__ __forceinline__ bool lane_bit(uint64_t mask) { return __builtin_amdgcn_inverse_ballot_w64(mask); }

struct BlockFolds {
    double disp = 0.0;
    float max_u = 0.f, max_v = 0.f;
};

template <int K, int R, int W>
__device__ __forceinline__ void block_pass(const float* __restrict__ eta, const float* __restrict__ u_i,
                                           const float* __restrict__ v_i, const float* __restrict__ hp_i,
                                           float* __restrict__ eta_o, float* __restrict__ u_o,
                                           float* __restrict__ v_o, int nx, int ny, int rbase, int wave, int lane,
                                           int c0, bool owned, int j0, int j1, const StepCoef& k,
                                           BlockShared<W>& sh, BlockFolds (&F)[K]) {
#pragma clang fp contract(off)
    const BlockIO io(nx, ny, c0);
    float e[R][2], u[R][2], v[R][2], hp[R][2];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        io.load(eta, rbase + r, e[r]);
        io.load(hp_i, rbase + r, hp[r]);
        io.load(u_i, rbase + r, u[r]);
        io.load(v_i, rbase + r, v[r]);
    }
    if (wave == 0) {
        const float2 z = make_float2(0.f, 0.f);
        sh.top_e[0][lane] = z;
        sh.top_v[0][lane] = z;
        sh.top_s[0][lane] = z;
        sh.bot_e[W + 1][lane] = z;
        sh.bot_s[W + 1][lane] = z;
    }
    // water masks of the tile's rows (w[r + 1]: row r) and of the rows beyond the wave's own, one
    // bit per lane
    uint64_t w[R + 2][2];
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            w[r + 1][c] = __ballot(hp[r][c] > 0.f);
            e[r][c] = lane_bit(w[r + 1][c]) ? e[r][c] : 0.f;  // the surface of a land cell is never used
        }
    }
    auto publish = [&]() {
        sh.top_e[wave + 1][lane] = make_float2(e[R - 1][0], e[R - 1][1]);
        sh.top_v[wave + 1][lane] = make_float2(v[R - 1][0], v[R - 1][1]);
        sh.bot_e[wave + 1][lane] = make_float2(e[0][0], e[0][1]);
    };
    sh.top_s[wave + 1][lane] = make_float2(hp[R - 1][0], hp[R - 1][1]);
    sh.bot_s[wave + 1][lane] = make_float2(hp[0][0], hp[0][1]);
    publish();
    __syncthreads();
    const float2 hpS2 = sh.top_s[wave][lane], hpN2 = sh.bot_s[wave + 2][lane];
    const float hpS[2] = {hpS2.x, hpS2.y}, hpN[2] = {hpN2.x, hpN2.y};
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        w[0][c] = __ballot(hpS[c] > 0.f);
        w[R + 1][c] = __ballot(hpN[c] > 0.f);
    }
    // Activity of a face = both its cells are water: formed from the water masks by scalar
    // operations wherever it is used (the scalar unit idles otherwise). Kept for the whole pass, the
    // faces' masks would not fit the scalar registers; forget() keeps the compiler from trying.
    auto forget = [&]() {
#pragma unroll
        for (int r = 0; r < R + 2; ++r) asm volatile("" : "+s"(w[r][0]), "+s"(w[r][1]));
    };
    auto east_a = [&](int r) { return lane_bit(w[r + 1][0] & w[r + 1][1]); };
    auto east_b = [&](int r) { return lane_bit(w[r + 1][1] & (w[r + 1][0] >> 1)); };
    auto north = [&](int r, int c) { return lane_bit(w[r + 1][c] & w[r + 2][c]); };  // face between r and r + 1
#pragma unroll
    for (int s = 0; s < K; ++s) {
        if (s > 0) publish();
        __syncthreads();
        forget();
        const float2 eS2 = sh.top_e[wave][lane], vS2 = sh.top_v[wave][lane], eN2 = sh.bot_e[wave + 2][lane];
        const float eS[2] = {eS2.x, eS2.y}, vS[2] = {vS2.x, vS2.y}, eN[2] = {eN2.x, eN2.y};
        float es[R][2], sx[R][2];
        float fyS[2], h[2];  // flux through the face below row r, total depth of row r
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            h[c] = hp[0][c] + e[0][c];
            fyS[c] = upwind_flux(y_pred(eS[c], e[0][c], vS[c], north(-1, c), k), hpS[c] + eS[c], h[c]);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            // x faces of the row (lane exchanges are taken by every lane)
            const float eEb = from_east(e[r][0]), hEb = from_east(h[0]);
            const float usa = x_pred(e[r][0], e[r][1], u[r][0], east_a(r), k);
            const float usb = x_pred(e[r][1], eEb, u[r][1], east_b(r), k);
            const float fxa = upwind_flux(usa, h[0], h[1]);
            const float fxb = upwind_flux(usb, h[1], hEb);
            const float pe[2] = {x_update(e[r][0], fxa, from_west(fxb), k), x_update(e[r][1], fxb, fxa, k)};
            u[r][0] = usa;
            u[r][1] = usb;
            // y face above the row, then the predicted surface (0 on land: its fluxes are 0)
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const float eU = r + 1 < R ? e[r + 1 < R ? r + 1 : r][c] : eN[c];
                const float hU = (r + 1 < R ? hp[r + 1 < R ? r + 1 : r][c] : hpN[c]) + eU;
                const float vs = y_pred(e[r][c], eU, v[r][c], north(r, c), k);
                const float fyN = upwind_flux(vs, h[c], hU);
                es[r][c] = fmaf(-k.ry, fyN - fyS[c], pe[c]);
                v[r][c] = vs;
                fyS[c] = fyN;
                h[c] = hU;
            }
            const float esEb = from_east(es[r][0]);
            const float da = east_a(r) ? es[r][1] - es[r][0] : 0.f;
            const float db = east_b(r) ? esEb - es[r][1] : 0.f;
            sx[r][0] = da - from_west(db);
            sx[r][1] = db - da;
        }
        sh.top_s[wave + 1][lane] = make_float2(es[R - 1][0], es[R - 1][1]);
        sh.bot_s[wave + 1][lane] = make_float2(es[0][0], es[0][1]);
        __syncthreads();
        forget();
        const float2 sS2 = sh.top_s[wave][lane], sN2 = sh.bot_s[wave + 2][lane];
        const float sS[2] = {sS2.x, sS2.y}, sN[2] = {sN2.x, sN2.y};
        float dS[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) dS[c] = north(-1, c) ? es[0][c] - sS[c] : 0.f;
#pragma unroll
        for (int r = 0; r < R; ++r) {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const float esU = r + 1 < R ? es[r + 1 < R ? r + 1 : r][c] : sN[c];
                const float dN = north(r, c) ? esU - es[r][c] : 0.f;
                const float sum = (sx[r][c] + dN) - dS[c];
                e[r][c] = lane_bit(w[r + 1][c]) ? fmaf(k.e4, sum, es[r][c]) : 0.f;
                dS[c] = dN;
            }
            if (rbase + r >= j0 && rbase + r < j1 && owned) {
                F[s].disp += (double)e[r][0] + (double)e[r][1];
                F[s].max_u = fmaxf(F[s].max_u, fmaxf(fabsf(u[r][0]), fabsf(u[r][1])));
                F[s].max_v = fmaxf(F[s].max_v, fmaxf(fabsf(v[r][0]), fabsf(v[r][1])));
            }
        }
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int row = rbase + r;
        if (row >= j0 && row < j1) {
            io.store(eta_o, row, owned, e[r]);
            io.store(u_o, row, owned, u[r]);
            io.store(v_o, row, owned, v[r]);
        }
    }
}

// Sums of the surface and maxima of the velocities of K <= 4 steps over a wave. Swapping half
// waves of two steps' values and then adding reduces both at once, so the four steps end up in
// the wave's four rows of 16 lanes (row s: step s, complete in every lane of the row) after one
// two-step exchange per pair, one four-step exchange and four levels within the rows: 41 vector
// instructions against 24 LDS exchanges per step for a plain butterfly. The order is fixed.
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

template <bool kHalves>  // kHalves: 32-lane halves, otherwise 16-lane rows
__device__ __forceinline__ void swap_lanes(unsigned& a, unsigned& b) {
    u32x2 r;
    if constexpr (kHalves)
        r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    else
        r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}

template <bool kHalves>
__device__ __forceinline__ float swap_max(float a, float b) {
    unsigned x = __float_as_uint(a), y = __float_as_uint(b);
    swap_lanes<kHalves>(x, y);
    return fmaxf(__uint_as_float(x), __uint_as_float(y));
}

template <bool kHalves>
__device__ __forceinline__ double swap_add(double a, double b) {
    const unsigned long long p = __double_as_longlong(a), q = __double_as_longlong(b);
    unsigned xl = (unsigned)p, xh = (unsigned)(p >> 32), yl = (unsigned)q, yh = (unsigned)(q >> 32);
    swap_lanes<kHalves>(xl, yl);
    swap_lanes<kHalves>(xh, yh);
    return __longlong_as_double((long long)(((unsigned long long)xh << 32) | xl)) +
           __longlong_as_double((long long)(((unsigned long long)yh << 32) | yl));
}

template <int kCtrl>
__device__ __forceinline__ unsigned dpp(unsigned x) {
    return (unsigned)__builtin_amdgcn_mov_dpp((int)x, kCtrl, 0xf, 0xf, true);
}

template <int kCtrl>
__device__ __forceinline__ void row_level(BlockFolds& f) {
    const unsigned long long p = __double_as_longlong(f.disp);
    const unsigned lo = dpp<kCtrl>((unsigned)p), hi = dpp<kCtrl>((unsigned)(p >> 32));
    f.disp += __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
    f.max_u = fmaxf(f.max_u, __uint_as_float(dpp<kCtrl>(__float_as_uint(f.max_u))));
    f.max_v = fmaxf(f.max_v, __uint_as_float(dpp<kCtrl>(__float_as_uint(f.max_v))));
}

template <bool kHalves>
__device__ __forceinline__ BlockFolds swap_fold(const BlockFolds& a, const BlockFolds& b) {
    BlockFolds r;
    r.disp = swap_add<kHalves>(a.disp, b.disp);
    r.max_u = swap_max<kHalves>(a.max_u, b.max_u);
    r.max_v = swap_max<kHalves>(a.max_v, b.max_v);
    return r;
}

template <int K>
__device__ __forceinline__ BlockFolds wave_folds(const BlockFolds (&F)[K]) {
    static_assert(K <= 4, "one row of lanes per step");
    const BlockFolds none;
    const BlockFolds even = swap_fold<true>(F[0], K > 2 ? F[K > 2 ? 2 : 0] : none);
    const BlockFolds odd = swap_fold<true>(K > 1 ? F[K > 1 ? 1 : 0] : none, K > 3 ? F[K > 3 ? 3 : 0] : none);
    BlockFolds r = swap_fold<false>(even, odd);
    row_level<0xB1>(r);   // quad_perm [1, 0, 3, 2]
    row_level<0x4E>(r);   // quad_perm [2, 3, 0, 1]
    row_level<0x141>(r);  // row_half_mirror
    row_level<0x140>(r);  // row_mirror
    return r;
}

// A tile's folds of K steps: the waves' sums added in wave order, one partial per step at
// part[s * stride]. Every wave has passed its last read of the tile's exchange rows when this
// returns, so the next tile may use them.
template <int W>
struct BlockFoldShared {
    double disp[4][W];
    float mu[4][W], mv[4][W];
};

template <int K, int W>
__device__ __forceinline__ void block_fold(const BlockFolds (&F)[K], int wave, int lane, BlockFoldShared<W>& sh,
                                           FoldPartial* __restrict__ part, size_t stride) {
    const BlockFolds f = wave_folds<K>(F);
    const int s = lane / 16;
    if (lane % 16 == 0) {
        sh.disp[s][wave] = f.disp;
        sh.mu[s][wave] = f.max_u;
        sh.mv[s][wave] = f.max_v;
    }
    __syncthreads();
    if (wave == 0 && lane < K) {
        double d = 0.0;
        float mu = 0.f, mv = 0.f;
#pragma unroll
        for (int i = 0; i < W; ++i) {
            d += sh.disp[lane][i];
            mu = fmaxf(mu, sh.mu[lane][i]);
            mv = fmaxf(mv, sh.mv[lane][i]);
        }
        FoldPartial* o = part + (size_t)lane * stride;
        o->disp = d;
        o->mu = mu;
        o->mv = mv;
    }
}

}  // namespace sw2d
