// sw2d_block.h - K time steps of one register tile (plain model).
//
// A workgroup of W waves holds a tile of W * R rows x 128 columns in registers: wave w the R
// rows from w R on, lane l the columns 2l and 2l + 1 of the tile ("a" and "b", as in
// sw2d_pair.h). The tile is read once, stepped K times in place and its owned cells written
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

#include "sw2d_pair.h"

namespace sw2d {

constexpr int kBlockCols = 2 * kWave;

// Rows exchanged between the waves of a tile: row w + 1 of an array is wave w's, rows 0 and
// W + 1 stay 0 (beyond the tile: land).
template <int W>
struct BlockShared {
    float2 top_e[W + 2][kWave], top_v[W + 2][kWave], bot_e[W + 2][kWave];
    float2 top_s[W + 2][kWave], bot_s[W + 2][kWave];
};

struct BlockFolds {
    double disp = 0.0;
    float max_u = 0.f, max_v = 0.f;
};

template <int K, int R, int W, bool kWide>
__device__ __forceinline__ void block_pass(const float* __restrict__ eta, const float* __restrict__ u_i,
                                           const float* __restrict__ v_i, const float* __restrict__ hp_i,
                                           float* __restrict__ eta_o, float* __restrict__ u_o,
                                           float* __restrict__ v_o, int nx, int ny, int rbase, int wave, int lane,
                                           int c0, bool owned, int j0, int j1, const StepCoef& k,
                                           BlockShared<W>& sh, BlockFolds (&F)[K]) {
#pragma clang fp contract(off)
    const PairIO<kWide> io{nx, ny, (unsigned)c0 * 4u};
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
    bool w[R][2], au[R][2], av[R + 1][2];
#pragma unroll
    for (int r = 0; r < R; ++r) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            w[r][c] = hp[r][c] > 0.f;
            e[r][c] = w[r][c] ? e[r][c] : 0.f;  // the surface of a land cell is never used
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
    for (int r = 0; r < R; ++r) {
        const bool wEb = from_east(hp[r][0]) > 0.f;
        au[r][0] = w[r][0] && w[r][1];
        au[r][1] = w[r][1] && wEb;
    }
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        av[0][c] = hpS[c] > 0.f && w[0][c];
#pragma unroll
        for (int r = 1; r < R; ++r) av[r][c] = w[r - 1][c] && w[r][c];
        av[R][c] = w[R - 1][c] && hpN[c] > 0.f;
    }
#pragma unroll
    for (int s = 0; s < K; ++s) {
        if (s > 0) publish();
        __syncthreads();
        const float2 eS2 = sh.top_e[wave][lane], vS2 = sh.top_v[wave][lane], eN2 = sh.bot_e[wave + 2][lane];
        const float eS[2] = {eS2.x, eS2.y}, vS[2] = {vS2.x, vS2.y}, eN[2] = {eN2.x, eN2.y};
        float es[R][2], sx[R][2];
        float fyS[2], h[2];  // flux through the face below row r, total depth of row r
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            h[c] = hp[0][c] + e[0][c];
            fyS[c] = upwind_flux(y_pred(eS[c], e[0][c], vS[c], av[0][c], k), hpS[c] + eS[c], h[c]);
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            // x faces of the row (lane exchanges are taken by every lane)
            const float eEb = from_east(e[r][0]), hEb = from_east(h[0]);
            const float usa = x_pred(e[r][0], e[r][1], u[r][0], au[r][0], k);
            const float usb = x_pred(e[r][1], eEb, u[r][1], au[r][1], k);
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
                const float vs = y_pred(e[r][c], eU, v[r][c], av[r + 1][c], k);
                const float fyN = upwind_flux(vs, h[c], hU);
                es[r][c] = fmaf(-k.ry, fyN - fyS[c], pe[c]);
                v[r][c] = vs;
                fyS[c] = fyN;
                h[c] = hU;
            }
            const float esEb = from_east(es[r][0]);
            const float da = au[r][0] ? es[r][1] - es[r][0] : 0.f;
            const float db = au[r][1] ? esEb - es[r][1] : 0.f;
            sx[r][0] = da - from_west(db);
            sx[r][1] = db - da;
        }
        sh.top_s[wave + 1][lane] = make_float2(es[R - 1][0], es[R - 1][1]);
        sh.bot_s[wave + 1][lane] = make_float2(es[0][0], es[0][1]);
        __syncthreads();
        const float2 sS2 = sh.top_s[wave][lane], sN2 = sh.bot_s[wave + 2][lane];
        const float sS[2] = {sS2.x, sS2.y}, sN[2] = {sN2.x, sN2.y};
        float dS[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) dS[c] = av[0][c] ? es[0][c] - sS[c] : 0.f;
#pragma unroll
        for (int r = 0; r < R; ++r) {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                const float esU = r + 1 < R ? es[r + 1 < R ? r + 1 : r][c] : sN[c];
                const float dN = av[r + 1][c] ? esU - es[r][c] : 0.f;
                const float sum = (sx[r][c] + dN) - dS[c];
                e[r][c] = w[r][c] ? fmaf(k.e4, sum, es[r][c]) : 0.f;
                dS[c] = dN;
            }
            if (rbase + r >= j0 && rbase + r < j1 && owned) {
                F[s].disp += (double)e[r][0] + (double)e[r][1];
                F[s].max_u = fmaxf(F[s].max_u, fmaxf(fabsf(u[r][0]), fabsf(u[r][1])));
                F[s].max_v = fmaxf(F[s].max_v, fmaxf(fabsf(v[r][0]), fabsf(v[r][1])));
            }
        }
    }
    const unsigned so = owned ? (unsigned)c0 * 4u : kNoLane;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int row = rbase + r;
        if (row >= j0 && row < j1) {
            io.store(eta_o, row, so, e[r]);
            io.store(u_o, row, so, u[r]);
            io.store(v_o, row, so, v[r]);
        }
    }
}

}  // namespace sw2d
