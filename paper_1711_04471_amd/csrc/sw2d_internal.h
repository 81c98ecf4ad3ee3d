// sw2d_internal.h - types shared by the 2DSW kernels and the C ABI host code.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sw2d.h"

namespace sw2d {

constexpr int kWave = 64;                            // CDNA wavefront width
constexpr int kHalo = 2;                             // stencil radius of the fused step
constexpr int kStripOut = kWave - 2 * kHalo;         // output columns per wave strip (60)
constexpr int kMaxStepsPerPass = 4;                 // temporal blocking depth (K steps per pass)
// Owned columns of a strip at K steps per pass: the plain model at K >= 2 takes two adjacent
// columns per lane (120, 116, 112), one step per pass one column (60).
constexpr int strip_out_for(int K) { return (K >= 2 ? 2 * kWave : kWave) - 4 * K; }
constexpr int kWavesPerGroup = 4;                    // strips per workgroup
constexpr int kGroupThreads = kWave * kWavesPerGroup;
constexpr int kGroupCols = kStripOut * kWavesPerGroup;  // 240 output columns per workgroup
constexpr int kFoldThreads = 256;
constexpr int kCus = 256;                            // MI355X
constexpr int kXcds = 8;                             // MI355X: 8 XCDs, one L2 each
constexpr int kMinRows = 8;                          // smallest band height a handle may use
constexpr int kFoldChunk = 16;                       // steps whose partials are buffered at least
constexpr size_t kMinPartBytes = 64 << 10;           // fold partials of the smallest grids
constexpr int kRingCap = 4096;                       // steps of folds kept for sw2d_reduce

// Per-workgroup fold partial of one step (16 B).
struct alignas(16) FoldPartial {
    double disp;  // sum over water cells of eta
    float mu;     // max |u|
    float mv;     // max |v|
};

struct StepGeometry {
    int nx, ny;
    int strips;    // ceil(nx / kStripOut)
    int groups_x;  // ceil(strips / kWavesPerGroup)
    int rows;      // rows per band
    int bands;     // ceil(ny / rows)
    int nblocks;   // groups_x * bands
};

// Step coefficients, computed in double on the host and rounded once to float.
struct StepCoef {
    float cx, cy;  // g dt / dx, g dt / dy
    float rx, ry;  // dt / dx, dt / dy
    float e4;      // eps / 4
    float kf;      // dt cd (bottom friction; 0 without it)
    float hmin;    // wet threshold on the total depth (wetting and drying; 0 without it)
};

// Model variants of the step (the flags of sw2d_params), as template arguments.
enum : int {
    kVarFriction = 1,
    kVarFilterUV = 2,
    kVarAdvection = 4,
    kVarAll = kVarFriction | kVarFilterUV | kVarAdvection,
    kVarWetDry = 8  // alone
};
// With advection the single-step strip keeps a 3-lane halo on its west side (the x-face
// predictor reads u one face further west) and 2 on its east side: 59 owned columns.
constexpr int kAdvHaloW = 3;
constexpr int kAdvStripOut = kWave - kAdvHaloW - kHalo;
constexpr int single_strip_out(uint32_t flags) { return (flags & kVarAdvection) ? kAdvStripOut : kStripOut; }
// Owned columns of a strip for K >= 2 steps per pass: the two-column pass for the plain
// model, the one-column pass for the variants that have one (all but advection).
constexpr int kstep_strip_out(int K, uint32_t flags) { return flags ? kWave - 4 * K : strip_out_for(K); }
// Variants that may advance several steps per pass: those whose step reaches no further than
// the plain step's two cells (advection reads one more face upstream).
constexpr bool kstep_variant_ok(uint32_t flags) { return (flags & kVarAdvection) == 0; }

enum : uint32_t {
    kWetBorder = 1u,
    kBadDepth = 2u,
    kBadState = 4u,
    kDryCell = 8u,
};

struct PrepFlags {
    uint32_t bad;        // OR of the k* bits above
    uint32_t hmax_bits;  // bit pattern of the largest water depth (positive float)
    double h_sum;        // sum over water cells of H (static part of the total volume)
};

constexpr int kHsumBlocks = 256;  // partials of the one-off sum_wet H

inline StepGeometry make_geometry(int nx, int ny, int rows, int strip_out = kStripOut) {
    StepGeometry g;
    g.nx = nx;
    g.ny = ny;
    g.strips = (nx + strip_out - 1) / strip_out;
    g.groups_x = (g.strips + kWavesPerGroup - 1) / kWavesPerGroup;
    g.rows = rows;
    g.bands = (ny + rows - 1) / rows;
    g.nblocks = g.groups_x * g.bands;
    return g;
}

// Register tiles (sw2d_block.h): kBlockWaves waves of R rows x 128 columns, K steps per pass.
// 8 waves: at 12 or 16 the barriers of a tile cost more than they share (us per step at K = 4,
// tiles of 40-48 rows: 2048^2 basin 8.4 with 8 waves, 8.6 with 12, 16.4 with 16; 66^2 basin 2.2,
// 2.4 and 3.3); 4 waves are no faster.
constexpr int kBlockWaves = 8;
constexpr int kBlockRows[] = {3, 5, 7, 8};  // tiles of 24, 40, 56 and 64 rows
constexpr int kBlockMaxK = 4;
// Grids of at most 2^23 cells, whose state and depth (28 B per cell and step, 235 MB) the 256 MB
// Infinity Cache holds, take several steps per pass whatever the caller's steps per pass: there is
// no HBM pass to choose. Larger grids take the caller's, if one was chosen, and else kBlockMaxK:
// the plain model over tiles at 4 steps per pass only (us per step on 8192 x 4096, tiles against the
// row pipelines: K = 1 197 and 192, K = 2 103 and 101, K = 3 71 and 71, K = 4 51.7 and 54.3:
// overlapping tiles re-read and recompute more, which the fewer instructions per cell outweigh at
// K = 4 alone), the variants at any, wetting and drying from 2 steps per pass on (K = 1 199 and
// 195).
constexpr int64_t kBlockMaxCells = (int64_t)1 << 23;
// Friction divides four times per cell and step, so that a pass of 4 steps, which recomputes a third
// of a tile or more, is bound by its vector issue: beyond 2^21 cells two steps per pass are faster (all
// variants, us per step at K = 2 and 4: 2047 x 1531 22.7 and 23.7, 8192 x 4096 164 and 200); below,
// where a launch has few tiles per CU, four are (1024^2 11.4 and 9.8).
constexpr int64_t kBlockFrictionCells = (int64_t)1 << 21;

// The order of the tiles of a larger grid: runs of this many, XCD by XCD, so that what runs at once lies
// close together in HBM (8192^2, K = 4, us per step at runs of 1, 2, 4, 9 and 16: 114, 106.8, 103.3,
// 101.1, 101.5; one contiguous range per XCD 104.0, vertical blocks of 8 bands 111). In the cache the
// rows shared within an XCD's L2 count for more: 2048^2 8.8 contiguous, 9.3 in runs of 16.
constexpr int kBlockRun = 16;

struct BlockGeometry {
    int nx, ny;
    int rows;  // R, rows per wave
    int strips, bands, nblocks;
    bool contiguous;  // an XCD's tiles lie together (see kBlockRun)
};

// Rows a step of a tile spoils on an open south side (2 on the others, and as many columns west):
// the advection's upwind differences reach one face further.
constexpr int block_south(int kVar) { return (kVar & kVarAdvection) ? 3 : 2; }
constexpr int block_west_lanes(int K, int kVar) { return (block_south(kVar) * K + 1) / 2; }

inline BlockGeometry make_block_geometry(int nx, int ny, int K, int R, int kvar = 0) {
    // neighbouring tiles overlap by what K steps spoil on their sides
    const int cols = 2 * kWave, rows = kBlockWaves * R;
    const int own_cols = cols - 2 * (block_west_lanes(K, kvar) + K), own_rows = rows - (block_south(kvar) + 2) * K;
    BlockGeometry g;
    g.nx = nx;
    g.ny = ny;
    g.rows = R;
    g.strips = nx <= cols ? 1 : 1 + (nx - cols + own_cols - 1) / own_cols;
    g.bands = ny <= rows ? 1 : 1 + (ny - rows + own_rows - 1) / own_rows;
    g.nblocks = g.strips * g.bands;
    g.contiguous = (int64_t)nx * ny <= kBlockMaxCells;
    return g;
}

// The tile heights for K steps of a model (kvar: its variants). The plain step at K <= 2 loads with the
// most waves on low tiles and overlaps little (2048^2, K = 2: 10.5, 10.9 and 12.1 us per step at 3, 5
// and 8 rows); wetting and drying, as cheap as the plain step but with more registers, is no faster on
// 64 rows (4096 x 2048 21.8 us against 20.0 on 40).
constexpr bool block_shape(int K, int R, int kvar) {
    if (R == 3) return true;
    if (R == 5) return kvar != 0 || K >= 3;
    if (R == 7) return kvar == 0 && K == 4;
    return kvar == 0 ? K == 4 : kvar != kVarWetDry && K >= 2;
}

// The tile height for K steps: the one whose tiles take the fewest rows on the CU with the most of
// them. A step of a tile alone takes 0.8 us at 3 rows per wave, 1.2 at 5 and 1.8 at 8, CUs with several
// tiles take about as long as their rows together, and a tile owns 4K (with advection 5K) rows less
// than it steps, so low tiles win while every CU has one, higher ones as the recomputed overlap counts,
// and between sizes the round that is left nearly empty decides. Plain model, passes of 4 steps alone (a
// call adds its remainder and its folds), us per step at 3, 5, 7 and 8 rows: 300 x 221 1.8, 2.3, 2.8, 3.1; 693 x 700 3.2, 2.55, 3.0, 3.35; 1024^2 4.7, 3.6, 3.2,
// 3.4; 2048^2 13.8, 8.7, 8.1, 8.8; 2300 x 2200 15.7, 9.4, 9.4, 9.1; 6000 x 5000 79, 52, 48, 47. All
// variants, K = 4, at 3, 5 and 8 rows: 693 x 700 16.0, 6.5, 9.5; 1024^2 30.5, 11.1, 9.8.
inline BlockGeometry block_geometry(int nx, int ny, int K, int kvar = 0) {
    BlockGeometry best{};
    int64_t least = 0;
    for (int R : kBlockRows) {
        if (!block_shape(K, R, kvar)) continue;
        const BlockGeometry g = make_block_geometry(nx, ny, K, R, kvar);
        const int64_t rows = (int64_t)((g.nblocks + kCus - 1) / kCus) * R;
        if (least == 0 || rows < least) {
            least = rows;
            best = g;
        }
    }
    return best;
}

// Whether the caller is capturing the stream (the null stream cannot be captured).
inline bool captured(hipStream_t s) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (!s) return false;
    if (hipStreamIsCapturing(s, &st) == hipSuccess) return st == hipStreamCaptureStatusActive;
    (void)hipGetLastError();
    return false;
}

// Each pass swaps a state's two buffers. A replayed capture starts from the buffer that it was recorded
// with, so it goes on from its own result only if it holds an even number of passes. The number of
// steps that a pass takes is the library's choice; for the caller, passes are of the steps per pass that
// the handle reports, and a captured call keeps their parity: single_steps steps are taken one at a time
// first, and the n steps then make an odd (or an even) number of passes of at most k steps.
inline int single_steps(int n, int k, bool odd) {
    if ((((n - 1) / k + 1) % 2 != 0) == odd) return 0;
    return n % k == 1 ? 2 : 1;  // one pass more
}

// K = 1..4 steps of the model (kvar: its variants, 0 for the plain step) in one pass over register
// tiles (geometry from block_geometry); the partials of step s of the pass go to
// part[s * geo.nblocks + 0..nblocks).
hipError_t launch_block(int K, int kvar, const float* eta, const float* u, const float* v, const float* hp,
                        float* eta_o, float* u_o, float* v_o, FoldPartial* part, const BlockGeometry& geo,
                        const StepCoef& k, hipStream_t s);

// A correction added to the state that a step leaves: scale times delta's three planes [3][ny][nx], on
// the water cells of mask and the faces between two of them.
struct StepCorrection {
    const float* delta;
    const uint8_t* mask;
    float scale[3];
};
// One step of the plain model over tiles (geometry for K = 1) with the correction added as the new state
// is stored; the folds are of the state before it.
hipError_t launch_block_corrected(const float* eta, const float* u, const float* v, const float* hp, float* eta_o,
                                  float* u_o, float* v_o, FoldPartial* part, const BlockGeometry& geo,
                                  const StepCoef& k, const StepCorrection& fix, hipStream_t s);

// kvar: the model variants (0 for the plain step).
hipError_t launch_step(int kvar, const float* eta, const float* u, const float* v, const float* hp,
                       float* eta_o, float* u_o, float* v_o, FoldPartial* part,
                       const StepGeometry& geo, const StepCoef& k, hipStream_t s);
// K = 2..4 steps in one pass (geometry from make_geometry(..., kstep_strip_out(K, flags))),
// kvar 0 or a variant without advection; the partials of step s of the pass go to
// part[s * stride + 0..nblocks).
hipError_t launch_stepk(int K, int kvar, const float* eta, const float* u, const float* v, const float* hp,
                        float* eta_o, float* u_o, float* v_o, FoldPartial* part, int stride,
                        const StepGeometry& geo, const StepCoef& k, hipStream_t s);
// Runs of steps whose partials wait to be folded: step i of a run has its parts at
// part + offset + i * stride. Several runs, as a call of 4 + 1 steps leaves, go into one launch.
struct FoldRuns {
    static constexpr int kMax = 4;
    int n;
    struct {
        int64_t offset;
        int nparts, stride, first;  // first: its first step among the steps of all runs
    } run[kMax];
};
hipError_t launch_fold(const FoldPartial* part, const FoldRuns& runs, int nsteps, int64_t first_step, sw2d_red* ring,
                       int ring_cap, double cell_area, double h_sum, hipStream_t s);
// Validation + packing, then sum_wet H; scratch holds kHsumBlocks doubles.
// The paper-shaped split: dyn, shapiro, velocity update, then a fold over the new state
// into part[0..nparts). scratch holds 3 nx ny floats.
hipError_t launch_unfused_step(const float* eta, const float* u, const float* v, const float* hp, float* eta_o,
                               float* u_o, float* v_o, float* scratch, int nx, int ny, const StepCoef& k,
                               FoldPartial* part, int nparts, hipStream_t s);
hipError_t launch_prep(const float* H, const uint8_t* mask, const float* eta, const float* u,
                       const float* v, int nx, int ny, float* hp, PrepFlags* flags,
                       double* scratch, hipStream_t s, bool allow_dry = false);

namespace detail {
// Shared by the single-grid and batched C ABI (defined in sw2d_api.hip).
bool params_valid(const sw2d_params* p);
StepCoef make_coef(const sw2d_params* p);
void set_hip_message(const char* msg);
}  // namespace detail

}  // namespace sw2d
