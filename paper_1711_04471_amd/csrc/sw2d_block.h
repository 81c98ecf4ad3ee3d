// sw2d_block.h - K time steps of one register tile.
//
// A workgroup of W waves holds a tile of W * R rows x 128 columns in registers: wave w the R
// rows from w R on, lane l the columns 2l and 2l + 1 of the tile ("a" and "b"). The tile is read
// once, stepped K times in place and its owned cells written once. East/west neighbours are the lane's other column and one lane exchange; the rows
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
// The variants add their terms to the same faces: friction and advection to the predictors (u and v
// of the rows next to a wave's own come through LDS as well, and v of two rows below), the velocity
// filter a second use of the exchange with the predicted velocities, wetting and drying masks of the
// cells wet now, formed per step.
//
// What bounds a pass: the vector issue of a CU's tiles (33 vector instructions per cell and step
// against the two-column row pipeline's 49; a tile of 40 rows takes about 1.2 us per step
// wherever it runs) plus 4 us for the launch, the loads and the stores. Measured per step, the
// default handle's streamed single step before and the tiles now: 66^2 7.0 and 1.7 us (200
// steps a call), 2048^2 22.8 and 8.7 us (50 a call: 483,000 Mcell-steps/s; 117 MB from the
// cache take 14.5 us at a large copy's rate there, so several steps per pass are what beats it).
// All variants at once, 2047 x 1531: 31.2 and 22.7 us (bound by the issue of friction's four
// divisions per cell), 301 x 221 10.2 and 4.5; friction alone 23.2 and 15.8, the velocity filter
// 21.1 and 9.5, advection 20.9 and 12.7, wetting and drying 19.7 and 9.1.
#pragma once

#include "sw2d_tile.h"

namespace sw2d {

constexpr int kBlockCols = 2 * kWave;

// Rows exchanged between the waves of a tile: row w + 1 of an array is wave w's, rows 0 and
// W + 1 stay 0 (beyond the tile: land). The velocity filter and the advection exchange more rows.
template <int W>
using BlockRow = float2[W + 2][kWave];

struct BlockNoRows {};

template <int W>
struct BlockFilterRows {
    BlockRow<W> top_us, bot_us, bot_vs;  // predicted velocities
};

template <int W>
struct BlockAdvRows {
    BlockRow<W> top_u, bot_u, bot_v, low_v;  // low_v: v of the row below the top one
};

template <int W, int kVar = 0>
struct BlockShared : std::conditional_t<(kVar & kVarFilterUV) != 0, BlockFilterRows<W>, BlockNoRows>,
                     std::conditional_t<(kVar & kVarAdvection) != 0, BlockAdvRows<W>, StageNoFlags> {
    BlockRow<W> top_e, top_v, bot_e;
    BlockRow<W> top_s, bot_s;
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

struct BlockNoFix {};  // the state is stored as the steps leave it

// Fix: what is done to the cells of a row before they are stored, after the folds.
template <int K, int R, int W, int kVar = 0, typename Fix = BlockNoFix>
__device__ __forceinline__ void block_pass(const float* __restrict__ eta, const float* __restrict__ u_i,
                                           const float* __restrict__ v_i, const float* __restrict__ hp_i,
                                           float* __restrict__ eta_o, float* __restrict__ u_o,
                                           float* __restrict__ v_o, int nx, int ny, int rbase, int wave, int lane,
                                           int c0, bool owned, int j0, int j1, const StepCoef& k,
                                           BlockShared<W, kVar>& sh, BlockFolds (&F)[K], const Fix& fix = Fix()) {
#pragma clang fp contract(off)
    constexpr bool kFriction = (kVar & kVarFriction) != 0, kFilterUV = (kVar & kVarFilterUV) != 0;
    constexpr bool kAdv = (kVar & kVarAdvection) != 0, kWetDry = (kVar & kVarWetDry) != 0;
    static_assert(R >= 2 || !kAdv, "the row below the top one is the wave's own");
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
        if constexpr (kFilterUV) {
            sh.top_us[0][lane] = z;
            sh.bot_us[W + 1][lane] = z;
            sh.bot_vs[W + 1][lane] = z;
        }
        if constexpr (kAdv) {
            sh.top_u[0][lane] = z;
            sh.low_v[0][lane] = z;
            sh.bot_u[W + 1][lane] = z;
            sh.bot_v[W + 1][lane] = z;
        }
    }
    // water masks of the tile's rows (w[r + 1]: row r) and of the rows beyond the wave's own, one
    // bit per lane (the velocity filter looks two rows up)
    constexpr int kMasks = R + (kFilterUV ? 3 : 2);
    uint64_t w[kMasks][2];
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            w[r + 1][c] = __ballot(hp[r][c] > 0.f);
            // The surface of a land cell is never used (wetting and drying compares it), but one that is
            // not finite makes the flux through a shut face, 0 times its depth, NaN: it stays so. (The
            // surface as it was loaded gives the same, 0.7 % slower on 2048^2.)
            if constexpr (!kWetDry) e[r][c] = lane_bit(w[r + 1][c]) ? e[r][c] : 0.f * e[r][c];
        }
    }
    auto pack = [](const float (&x)[2]) { return make_float2(x[0], x[1]); };
    auto publish = [&]() {
        sh.top_e[wave + 1][lane] = pack(e[R - 1]);
        sh.top_v[wave + 1][lane] = pack(v[R - 1]);
        sh.bot_e[wave + 1][lane] = pack(e[0]);
        if constexpr (kAdv) {
            sh.top_u[wave + 1][lane] = pack(u[R - 1]);
            sh.low_v[wave + 1][lane] = pack(v[R > 1 ? R - 2 : 0]);
            sh.bot_u[wave + 1][lane] = pack(u[0]);
            sh.bot_v[wave + 1][lane] = pack(v[0]);
        }
    };
    sh.top_s[wave + 1][lane] = pack(hp[R - 1]);
    sh.bot_s[wave + 1][lane] = pack(hp[0]);
    if constexpr (kFilterUV) sh.bot_us[wave + 1][lane] = pack(hp[R > 1 ? 1 : 0]);
    publish();
    __syncthreads();
    auto fetch = [&](const BlockRow<W>& rows, int at, float (&x)[2]) {
        const float2 q = rows[at][lane];
        x[0] = q.x;
        x[1] = q.y;
    };
    float hpS[2], hpN[2];
    fetch(sh.top_s, wave, hpS);
    fetch(sh.bot_s, wave + 2, hpN);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        w[0][c] = __ballot(hpS[c] > 0.f);
        w[R + 1][c] = __ballot(hpN[c] > 0.f);
    }
    if constexpr (kFilterUV) {
        static_assert(R >= 2, "the second row up is the next wave's own");
        float hp2[2];
        fetch(sh.bot_us, wave + 2, hp2);
#pragma unroll
        for (int c = 0; c < 2; ++c) w[kMasks - 1][c] = __ballot(hp2[c] > 0.f);
    }
    // Activity of a face = both its cells are water: formed from the water masks by scalar
    // operations wherever it is used (the scalar unit idles otherwise). Kept for the whole pass, the
    // faces' masks would not fit the scalar registers; forget() keeps the compiler from trying.
    auto forget = [&]() {
#pragma unroll
        for (int r = 0; r < kMasks; ++r) asm volatile("" : "+s"(w[r][0]), "+s"(w[r][1]));
    };
    auto east_a = [&](int r) { return w[r + 1][0] & w[r + 1][1]; };
    auto east_b = [&](int r) { return w[r + 1][1] & (w[r + 1][0] >> 1); };
    auto north = [&](int r, int c) { return w[r + 1][c] & w[r + 2][c]; };  // face between r and r + 1
    // Predictor of an x-face (west cell e, h; east cell eE, hE; uW, uE, uS, uN its neighbours, vb the
    // mean v) and of a y-face: the formulas of row_x, face_y and StageAdv.
    auto x_face = [&](float eC, float eE, float hC, float hE, float uC, float uW, float uE, float uS, float uN,
                      float vb, bool act) {
        float p;
        if constexpr (kWetDry)
            return act && face_open(hC > k.hmin, hE > k.hmin, eC, eE) ? fmaf(-k.cx, eE - eC, uC) : 0.f;
        p = fmaf(-k.cx, eE - eC, uC);
        if constexpr (kAdv) {
            const float tx = uC > 0.f ? uC * (uC - uW) : uC * (uE - uC);
            const float ty = vb > 0.f ? vb * (uC - uS) : vb * (uN - uC);
            p = p - (tx * k.rx + ty * k.ry);
        }
        // (without advection the pipelines select before the friction as well: the same value)
        if constexpr (kFriction) p = friction(p, uC, hC, hE, k);
        return act ? p : 0.f;
    };
    auto y_face = [&](float eC, float eN, float hC, float hN, float vC, float vW, float vE, float vS, float vN,
                      float ub, bool act) {
        float p;
        if constexpr (kWetDry)
            return act && face_open(hC > k.hmin, hN > k.hmin, eC, eN) ? fmaf(-k.cy, eN - eC, vC) : 0.f;
        p = fmaf(-k.cy, eN - eC, vC);
        if constexpr (kAdv) {
            const float tx = ub > 0.f ? ub * (vC - vW) : ub * (vE - vC);
            const float ty = vC > 0.f ? vC * (vC - vS) : vC * (vN - vC);
            p = p - (tx * k.rx + ty * k.ry);
        }
        if constexpr (kFriction) p = friction(p, vC, hC, hN, k);
        return act ? p : 0.f;
    };
    // mean of the four u faces around the y-face between a row and the next: their own and the west one
    auto mean_u = [&](const float (&lo)[2], const float (&hi)[2], float (&ub)[2]) {
        const float loW = from_west(lo[1]), hiW = from_west(hi[1]);
        ub[0] = 0.25f * ((lo[0] + loW) + (hi[0] + hiW));
        ub[1] = 0.25f * ((lo[1] + lo[0]) + (hi[1] + hi[0]));
    };
    float none[2] = {0.f, 0.f};
#pragma unroll
    for (int s = 0; s < K; ++s) {
        if (s > 0) publish();
        __syncthreads();
        forget();
        float eS[2], vS[2], eN[2];
        fetch(sh.top_e, wave, eS);
        fetch(sh.top_v, wave, vS);
        fetch(sh.bot_e, wave + 2, eN);
        float uS[2], uN[2], vN[2], vSS[2];
        if constexpr (kAdv) {
            fetch(sh.top_u, wave, uS);
            fetch(sh.low_v, wave, vSS);
            fetch(sh.bot_u, wave + 2, uN);
            fetch(sh.bot_v, wave + 2, vN);
        }
        float es[R][2], sx[R][2];
        float fyS[2], h[2];  // flux through the face below row r, total depth of row r
        float vsS[2];        // predicted velocity of the face below row 0
        uint64_t d[kWetDry ? R + 2 : 1][2];  // wet now (rows as in w)
        float ub[2] = {0.f, 0.f}, vSw[2] = {0.f, 0.f}, vSe[2] = {0.f, 0.f};
        if constexpr (kAdv) {
            mean_u(uS, u[0], ub);
            vSw[0] = from_west(vS[1]);
            vSw[1] = vS[0];
            vSe[0] = vS[1];
            vSe[1] = from_east(vS[0]);
        }
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            h[c] = hp[0][c] + e[0][c];
            const float hS = hpS[c] + eS[c];
            vsS[c] = y_face(eS[c], e[0][c], hS, h[c], vS[c], vSw[c], vSe[c], kAdv ? vSS[c] : 0.f, v[0][c], ub[c],
                            lane_bit(north(-1, c)));
            fyS[c] = upwind_flux(vsS[c], hS, h[c]);
            if constexpr (kWetDry) {
                d[0][c] = __ballot(hS > k.hmin);
                d[R + 1][c] = __ballot(hpN[c] + eN[c] > k.hmin);
            }
        }
        float uL[2] = {0.f, 0.f}, vL[2] = {0.f, 0.f};  // old u and v of the row below
        if constexpr (kAdv) {
            uL[0] = uS[0];
            uL[1] = uS[1];
            vL[0] = vS[0];
            vL[1] = vS[1];
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            // lane exchanges are taken by every lane before any select
            const float eEb = from_east(e[r][0]), hEb = from_east(h[0]);
            const float(&uU)[2] = !kAdv ? none : r + 1 < R ? u[r + 1 < R ? r + 1 : r] : uN;  // old rows above
            const float(&vU)[2] = !kAdv ? none : r + 1 < R ? v[r + 1 < R ? r + 1 : r] : vN;
            float uWa = 0.f, uEb = 0.f, vWa = 0.f, vEb = 0.f, vb[2] = {0.f, 0.f}, uo[2], vo[2];
            if constexpr (kAdv) {
                uWa = from_west(u[r][1]);
                uEb = from_east(u[r][0]);
                vWa = from_west(v[r][1]);
                vEb = from_east(v[r][0]);
                vb[0] = 0.25f * ((v[r][0] + v[r][1]) + (vL[0] + vL[1]));
                vb[1] = 0.25f * ((v[r][1] + vEb) + (vL[1] + from_east(vL[0])));
                mean_u(u[r], uU, ub);
                uo[0] = u[r][0];
                uo[1] = u[r][1];
                vo[0] = v[r][0];
                vo[1] = v[r][1];
            }
            const float usa = x_face(e[r][0], e[r][1], h[0], h[1], u[r][0], uWa, u[r][1], uL[0], uU[0], vb[0],
                                     lane_bit(east_a(r)));
            const float usb = x_face(e[r][1], eEb, h[1], hEb, u[r][1], u[r][0], uEb, uL[1], uU[1], vb[1],
                                     lane_bit(east_b(r)));
            const float fxa = upwind_flux(usa, h[0], h[1]);
            const float fxb = upwind_flux(usb, h[1], hEb);
            const float pe[2] = {x_update(e[r][0], fxa, from_west(fxb), k), x_update(e[r][1], fxb, fxa, k)};
            u[r][0] = usa;
            u[r][1] = usb;
            // y face above the row, then the predicted surface (0 on land: its fluxes are 0)
            const float vW[2] = {vWa, v[r][0]}, vE[2] = {v[r][1], vEb};
            float vs[2];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const float eU = r + 1 < R ? e[r + 1 < R ? r + 1 : r][c] : eN[c];
                const float hU = (r + 1 < R ? hp[r + 1 < R ? r + 1 : r][c] : hpN[c]) + eU;
                vs[c] = y_face(e[r][c], eU, h[c], hU, v[r][c], vW[c], vE[c], vL[c], vU[c], ub[c],
                               lane_bit(north(r, c)));
                const float fyN = upwind_flux(vs[c], h[c], hU);
                es[r][c] = fmaf(-k.ry, fyN - fyS[c], pe[c]);
                if constexpr (kWetDry) {
                    d[r + 1][c] = __ballot(h[c] > k.hmin);
                    es[r][c] = lane_bit(w[r + 1][c]) ? es[r][c] : 0.f;
                }
                fyS[c] = fyN;
                h[c] = hU;
            }
            if constexpr (kAdv) {
                uL[0] = uo[0];
                uL[1] = uo[1];
                vL[0] = vo[0];
                vL[1] = vo[1];
            }
            v[r][0] = vs[0];
            v[r][1] = vs[1];
            const float esEb = from_east(es[r][0]);
            uint64_t ma, mb;
            if constexpr (kWetDry) {
                ma = d[r + 1][0] & d[r + 1][1];
                mb = d[r + 1][1] & (d[r + 1][0] >> 1);
            } else {
                ma = east_a(r);
                mb = east_b(r);
            }
            const float da = lane_bit(ma) ? es[r][1] - es[r][0] : 0.f;
            const float db = lane_bit(mb) ? esEb - es[r][1] : 0.f;
            sx[r][0] = da - from_west(db);
            sx[r][1] = db - da;
        }
        sh.top_s[wave + 1][lane] = pack(es[R - 1]);
        sh.bot_s[wave + 1][lane] = pack(es[0]);
        if constexpr (kFilterUV) {
            sh.top_us[wave + 1][lane] = pack(u[R - 1]);
            sh.bot_us[wave + 1][lane] = pack(u[0]);
            sh.bot_vs[wave + 1][lane] = pack(v[0]);
        }
        __syncthreads();
        forget();
        float sS[2], sN[2];
        fetch(sh.top_s, wave, sS);
        fetch(sh.bot_s, wave + 2, sN);
        auto pair_mask = [&](int r, int c) {  // the filter's exchange between rows r and r + 1
            if constexpr (kWetDry) return d[r + 1][c] & d[r + 2][c];
            else return north(r, c);
        };
        float dS[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) dS[c] = lane_bit(pair_mask(-1, c)) ? es[0][c] - sS[c] : 0.f;
        // differences of the predicted velocities across the lower side of the row (filter)
        float usN[2], vsN[2], duS[2], dvS[2];
        if constexpr (kFilterUV) {
            float usS[2];
            fetch(sh.top_us, wave, usS);
            fetch(sh.bot_us, wave + 2, usN);
            fetch(sh.bot_vs, wave + 2, vsN);
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const uint64_t below = c ? east_b(-1) : east_a(-1), here = c ? east_b(0) : east_a(0);
                duS[c] = lane_bit(below & here) ? u[0][c] - usS[c] : 0.f;
                dvS[c] = lane_bit(north(-1, c) & north(0, c)) ? v[0][c] - vsS[c] : 0.f;
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const float esU = r + 1 < R ? es[r + 1 < R ? r + 1 : r][c] : sN[c];
                const float dN = lane_bit(pair_mask(r, c)) ? esU - es[r][c] : 0.f;
                const float sum = (sx[r][c] + dN) - dS[c];
                const float f = fmaf(k.e4, sum, es[r][c]);
                if constexpr (kWetDry)
                    e[r][c] = lane_bit(d[r + 1][c]) ? f : es[r][c];
                else
                    e[r][c] = lane_bit(w[r + 1][c]) ? f : 0.f;
                dS[c] = dN;
            }
            if constexpr (kFilterUV) {
                // the same filter on the faces: each difference once, masked by both faces
                const uint64_t ua = east_a(r), ubm = east_b(r), va = north(r, 0), vbm = north(r, 1);
                const float uEb = from_east(u[r][0]), vEb = from_east(v[r][0]);
                const float uda = lane_bit(ua & ubm) ? u[r][1] - u[r][0] : 0.f;
                const float udb = lane_bit(ubm & (ua >> 1)) ? uEb - u[r][1] : 0.f;
                const float vda = lane_bit(va & vbm) ? v[r][1] - v[r][0] : 0.f;
                const float vdb = lane_bit(vbm & (va >> 1)) ? vEb - v[r][1] : 0.f;
                const float ux[2] = {uda - from_west(udb), udb - uda}, vx[2] = {vda - from_west(vdb), vdb - vda};
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const uint64_t um = c ? ubm : ua, vm = c ? vbm : va;
                    const float uUp = r + 1 < R ? u[r + 1 < R ? r + 1 : r][c] : usN[c];
                    const float vUp = r + 1 < R ? v[r + 1 < R ? r + 1 : r][c] : vsN[c];
                    const float duN = lane_bit(um & (c ? east_b(r + 1) : east_a(r + 1))) ? uUp - u[r][c] : 0.f;
                    const float dvN = lane_bit(vm & north(r + 1, c)) ? vUp - v[r][c] : 0.f;
                    const float un = fmaf(k.e4, (ux[c] + duN) - duS[c], u[r][c]);
                    const float vn = fmaf(k.e4, (vx[c] + dvN) - dvS[c], v[r][c]);
                    duS[c] = duN;
                    dvS[c] = dvN;
                    u[r][c] = lane_bit(um) ? un : 0.f;
                    v[r][c] = lane_bit(vm) ? vn : 0.f;
                }
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
            if constexpr (!std::is_same_v<Fix, BlockNoFix>) fix(io, row, e[r], u[r], v[r]);
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
