// sw2d_batch.hip - ensembles of independent 2DSW basins of uneven sizes advanced together.
//
// A pass advances every member K <= 4 steps over register tiles (sw2d_block.h: the tile routine
// of the single-grid step, so each instance is bitwise equal to the same basin stepped alone).
// The tiles of all members, member by member and band by band, form one list; all cost the same,
// whatever part of the grid they cover. Each writes one fold partial per step; one wave per
// member and step adds a pass's partials in a fixed order and writes the ring entry while the
// next pass runs.
//
// One launch per pass (sw2d_batch_pass_kernel, a workgroup per tile): the hardware hands tiles out
// as workgroups end and the stream order is the barrier. The launches of a call are recorded as a
// HIP graph and replayed.
//
// One persistent launch per chunk of steps (sw2d_batch_kernel) where the caller asks for it:
// workgroup g of G takes the g-th of G equal runs of the list and meets the others at a grid
// barrier after each pass. Measured slower at either end: 12 members of 64-256 cells a side, 50 steps,
// 189 us (the barrier takes longer than a launch) against 135; 256 members of 128-1024, 48 steps, 10.4 ms
// (equal runs end up to a quarter apart, and the loop's state spills scalar registers) against 6.6.
//
// The barrier uses no contended atomics: every workgroup publishes the epoch it has
// reached in its own flag (after an agent-scope release), workgroup 0 waits for all
// flags in parallel and publishes the epoch in one "go" word, which the others poll.
// Epochs are the global step counts, so they only grow and no flag is ever reset. Every
// wait has a wall-clock deadline: on expiry it raises an error flag and the kernel
// returns, so no wave can wait forever even if the grid were not co-resident.
//
// The steps done so far live in device memory and are advanced by the kernel itself, so
// a captured graph of launches can be replayed without host-side parameters.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <new>
#include <utility>
#include <vector>

#include "sw2d_block.h"
#include "sw2d_internal.h"

namespace sw2d {

// Tiles of a member at K steps per pass: bands of strips, tile_begin the first in the list.
struct BatchTiles {
    int strips, bands, tile_begin;
};

struct BatchInst {
    const float* hp;
    float* state[2][3];
    int nx, ny;
    StepCoef k;
    double cell_area;
    double h_sum;
    BatchTiles t[kBlockMaxK];  // [K - 1]
};

constexpr int kFlagStride = 16;  // 64-bit words between flags: one 128 B line each

struct BatchControl {
    unsigned error;         // 1: a barrier wait ran past its deadline
    unsigned pad0;
    long long steps_done;   // advanced by the kernel at the end of every launch
    long long passes_done;  // passes over the state so far: its parity picks the current buffer
    long long pad1[kFlagStride - 3];
    unsigned long long go;  // last epoch every workgroup has reached (own line)
    unsigned long long pad2[kFlagStride - 1];
    // followed by one flag line per workgroup
};

constexpr int kBatchThreads = kWave * kBlockWaves;
constexpr int kMaxBatchK = 3;  // steps per pass a caller may ask for: 1..3
constexpr int kBatchRing = 64;  // steps of per-instance folds kept

struct BatchArgs {
    const BatchInst* inst;
    FoldPartial* part;  // [2][K][n_tiles]
    sw2d_red* ring;     // [kBatchRing][n_inst]
    BatchControl* ctl;
    unsigned long long* flags;  // [grid][kFlagStride]
    int n_inst, n_tiles, steps;
    unsigned long long timeout_ticks;
};

__device__ __forceinline__ bool spin_until(const unsigned long long* word, unsigned long long epoch,
                                           unsigned long long deadline, BatchControl* ctl) {
    while (__hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < epoch) {
        __builtin_amdgcn_s_sleep(2);
        if (wall_clock64() > deadline) {
            __hip_atomic_fetch_or(&ctl->error, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return false;
        }
    }
    return true;
}

// Returns false (for the whole workgroup) if a wait ran past the deadline.
__device__ bool grid_barrier(const BatchArgs& a, unsigned long long epoch) {
    __shared__ int s_ok;
    const unsigned long long deadline = wall_clock64() + a.timeout_ticks;
    if (threadIdx.x == 0) s_ok = 1;
    __syncthreads();  // every wave's stores of this step precede thread 0's release
    if (threadIdx.x == 0) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        __hip_atomic_store(a.flags + (size_t)blockIdx.x * kFlagStride, epoch, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
    if (blockIdx.x == 0) {
        for (int w = threadIdx.x; w < (int)gridDim.x; w += kBatchThreads)
            if (!spin_until(a.flags + (size_t)w * kFlagStride, epoch, deadline, a.ctl)) s_ok = 0;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        __syncthreads();
        if (threadIdx.x == 0 && s_ok) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
            __hip_atomic_store(&a.ctl->go, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    if (threadIdx.x == 0 && s_ok) {
        if (!spin_until(&a.ctl->go, epoch, deadline, a.ctl)) s_ok = 0;
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
    return s_ok != 0;
}

// Folds of one pass: wave q of the grid adds the tile partials of (member, step) pairs q, q + the
// grid's waves, ... (a lane every 64th partial, then the lanes) and writes their ring entries. The
// order does not depend on the grid.
template <int K>
__device__ __forceinline__ void fold_pass(const BatchArgs& a, int first_wave, int nwaves, int lane,
                                          const FoldPartial* __restrict__ part, long long first_step) {
    for (int q = first_wave; q < a.n_inst * K; q += nwaves) {
        const int i = q / K, s = q - i * K;
        const BatchInst& in = a.inst[i];
        const int t0 = in.t[K - 1].tile_begin, t1 = t0 + in.t[K - 1].strips * in.t[K - 1].bands;
        const FoldPartial* p = part + (size_t)s * a.n_tiles;
        BlockFolds F[1];
        for (int it = t0 + lane; it < t1; it += kWave) {
            F[0].disp += p[it].disp;
            F[0].max_u = fmaxf(F[0].max_u, p[it].mu);
            F[0].max_v = fmaxf(F[0].max_v, p[it].mv);
        }
        const BlockFolds f = wave_folds<1>(F);  // complete in lanes 0..15
        if (lane == 0) {
            const long long step = first_step + s;
            sw2d_red* o = a.ring + (size_t)((step - 1) % kBatchRing) * a.n_inst + i;
            o->step = step;
            o->vol_total = in.cell_area * (in.h_sum + f.disp);
            o->vol_disp = in.cell_area * f.disp;
            o->max_abs_u = f.max_u;
            o->max_abs_v = f.max_v;
        }
    }
}

__device__ __forceinline__ int logical_block(int b, int n) {
    const int q = n / kXcds, r = n % kXcds;
    const int x = b % kXcds, k = b / kXcds;
    return x * q + min(x, r) + k;
}

__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

template <typename T>
__device__ __forceinline__ T* uniform_ptr(T* p) {
    const uintptr_t v = reinterpret_cast<uintptr_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return reinterpret_cast<T*>(((uintptr_t)hi << 32) | lo);
}

__device__ __forceinline__ float uniform_f(float x) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}

// K steps per pass over tiles of R rows per wave; a.steps is a multiple of K.
template <int K, int R>
__global__ __launch_bounds__(kBatchThreads) void sw2d_batch_kernel(BatchArgs a) {
    constexpr int W = kBlockWaves, T = W * R;
    __shared__ BlockShared<W> sh;
    __shared__ BlockFoldShared<W> fsh;
    const int nwg = gridDim.x;
    const int lwg = logical_block(blockIdx.x, nwg);
    const int wave = uniform(threadIdx.x / kWave), lane = threadIdx.x % kWave;
    const long long base = a.ctl->steps_done;
    const long long pbase = a.ctl->passes_done;
    const int passes = a.steps / K;
    // this workgroup's run of tiles (none beyond the first n_tiles workgroups)
    const int workers = min(nwg, a.n_tiles);
    const int t0 = lwg < workers ? (int)((long long)lwg * a.n_tiles / workers) : 0;
    const int t1 = lwg < workers ? (int)((long long)(lwg + 1) * a.n_tiles / workers) : 0;
    int m0 = 0;  // the member of tile t0
    for (int lo = 0, hi = a.n_inst; hi - lo > 1;) {
        const int mid = (lo + hi) / 2;
        if (uniform(a.inst[mid].t[K - 1].tile_begin) <= t0) lo = m0 = mid;
        else hi = mid;
    }
    // the folds start from the last workgroups, which a small ensemble leaves without tiles
    const int fold_wave = (nwg - 1 - lwg) * W + wave, fold_waves = nwg * W;

    for (int ps = 0; ps < passes; ++ps) {
        const long long step0 = base + (long long)ps * K;  // steps made before this pass
        const int cur = (int)((pbase + ps) & 1);
        FoldPartial* part = a.part + (size_t)(ps & 1) * K * a.n_tiles;
        int m = m0;
        for (int t = t0; t < t1; ++t) {
            int local = t - uniform(a.inst[m].t[K - 1].tile_begin);
            int strips = uniform(a.inst[m].t[K - 1].strips), bands = uniform(a.inst[m].t[K - 1].bands);
            if (local >= strips * bands) {
                ++m;
                local = 0;
                strips = uniform(a.inst[m].t[K - 1].strips);
                bands = uniform(a.inst[m].t[K - 1].bands);
            }
            const BatchInst& in = a.inst[m];
            const int nx = uniform(in.nx), ny = uniform(in.ny);
            StepCoef k;
            k.cx = uniform_f(in.k.cx);
            k.cy = uniform_f(in.k.cy);
            k.rx = uniform_f(in.k.rx);
            k.ry = uniform_f(in.k.ry);
            k.e4 = uniform_f(in.k.e4);
            k.kf = 0.f;
            k.hmin = 0.f;
            const int band = local / strips, strip = local - band * strips;
            const int r0 = band * (T - 4 * K), c0 = strip * (kBlockCols - 4 * K) + 2 * lane;
            const int j0 = band > 0 ? r0 + 2 * K : 0, j1 = band + 1 < bands ? r0 + T - 2 * K : ny;
            const bool owned = (strip == 0 || lane >= K) && (strip + 1 == strips ? c0 < nx : lane < kWave - K);
            BlockFolds F[K];
            block_pass<K, R, W>(uniform_ptr(in.state[cur][0]), uniform_ptr(in.state[cur][1]),
                                uniform_ptr(in.state[cur][2]), uniform_ptr(in.hp), uniform_ptr(in.state[cur ^ 1][0]),
                                uniform_ptr(in.state[cur ^ 1][1]), uniform_ptr(in.state[cur ^ 1][2]), nx, ny,
                                r0 + wave * R, wave, lane, c0, owned, j0, j1, k, sh, F);
            block_fold<K, W>(F, wave, lane, fsh, part + t, a.n_tiles);
        }
        if (ps > 0)
            fold_pass<K>(a, fold_wave, fold_waves, lane, a.part + (size_t)((ps - 1) & 1) * K * a.n_tiles, step0 - K + 1);
        if (!grid_barrier(a, (unsigned long long)(step0 + K))) return;
    }
    fold_pass<K>(a, fold_wave, fold_waves, lane, a.part + (size_t)((passes - 1) & 1) * K * a.n_tiles,
                 base + (long long)(passes - 1) * K + 1);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.ctl->steps_done = base + a.steps;
        a.ctl->passes_done = pbase + passes;
    }
}

// One pass of one launch: workgroup b takes tile b (XCD-contiguous); the workgroups beyond the
// tiles add the previous pass's partials (fold_steps of them, none before the first pass of a
// call). pass, step: passes and steps of this call made before this pass.
struct BatchPass {
    const BatchInst* inst;
    const int* member;  // of each tile
    FoldPartial *part, *prev_part;
    sw2d_red* ring;
    const BatchControl* ctl;
    int n_inst, n_tiles, pass, step;
    int fold_steps, prev_tiles;
};

// Folds of a pass of K steps in `part`, K any of 1..kBlockMaxK.
__device__ __forceinline__ void fold_any(int K, BatchArgs a, int first_wave, int nwaves, int lane,
                                         const FoldPartial* __restrict__ part, long long first_step) {
    switch (K) {
        case 1: fold_pass<1>(a, first_wave, nwaves, lane, part, first_step); break;
        case 2: fold_pass<2>(a, first_wave, nwaves, lane, part, first_step); break;
        case 3: fold_pass<3>(a, first_wave, nwaves, lane, part, first_step); break;
        case 4: fold_pass<4>(a, first_wave, nwaves, lane, part, first_step); break;
    }
}

__device__ __forceinline__ void fold_prev(const BatchPass& a, int block, int nblocks) {
    BatchArgs f{};
    f.inst = a.inst;
    f.ring = a.ring;
    f.n_inst = a.n_inst;
    f.n_tiles = a.prev_tiles;
    const int wave = uniform(threadIdx.x / kWave), lane = threadIdx.x % kWave;
    fold_any(a.fold_steps, f, block * kBlockWaves + wave, nblocks * kBlockWaves, lane, a.prev_part,
             a.ctl->steps_done + a.step - a.fold_steps + 1);
}

template <int K, int R>
__global__ __launch_bounds__(kBatchThreads) void sw2d_batch_pass_kernel(const BatchInst* __restrict__ inst,
                                                                        const int* __restrict__ member, BatchPass a) {
    constexpr int W = kBlockWaves, T = W * R;
    __shared__ BlockShared<W> sh;
    __shared__ BlockFoldShared<W> fsh;
    if ((int)blockIdx.x >= a.n_tiles) {
        fold_prev(a, blockIdx.x - a.n_tiles, gridDim.x - a.n_tiles);
        return;
    }
    const int t = logical_block(blockIdx.x, a.n_tiles);
    const BatchInst& in = inst[member[t]];
    const int cur = (int)((a.ctl->passes_done + a.pass) & 1);
    const int wave = uniform(threadIdx.x / kWave), lane = threadIdx.x % kWave;
    const int strips = in.t[K - 1].strips, bands = in.t[K - 1].bands;
    const int local = t - in.t[K - 1].tile_begin;
    const int band = local / strips, strip = local - band * strips;
    const int r0 = band * (T - 4 * K), c0 = strip * (kBlockCols - 4 * K) + 2 * lane;
    const int j0 = band > 0 ? r0 + 2 * K : 0, j1 = band + 1 < bands ? r0 + T - 2 * K : in.ny;
    const bool owned = (strip == 0 || lane >= K) && (strip + 1 == strips ? c0 < in.nx : lane < kWave - K);
    BlockFolds F[K];
    block_pass<K, R, W>(in.state[cur][0], in.state[cur][1], in.state[cur][2], in.hp, in.state[cur ^ 1][0],
                        in.state[cur ^ 1][1], in.state[cur ^ 1][2], in.nx, in.ny, r0 + wave * R, wave, lane, c0, owned,
                        j0, j1, in.k, sh, F);
    block_fold<K, W>(F, wave, lane, fsh, a.part + t, a.n_tiles);
}

// After the last pass of a call: its folds, then the step and pass counts.
__global__ __launch_bounds__(kBatchThreads) void sw2d_batch_fold_kernel(BatchPass a) {
    fold_prev(a, blockIdx.x, gridDim.x);
}

__global__ void sw2d_batch_advance_kernel(BatchControl* ctl, int steps, int passes) {
    ctl->steps_done += steps;
    ctl->passes_done += passes;
}

}  // namespace sw2d

// ---------------------------------------------------------------------------------------
// C ABI of the batched form

using namespace sw2d;

struct sw2d_bctx {
    int n;
    std::vector<sw2d_params> p;
    std::vector<float*> state;  // [n][6]
    hipStream_t stream;         // the caller's
    hipStream_t capture;        // private stream used only to record graphs
    BatchInst* d_inst;
    int* d_member[kBlockMaxK];  // member of each tile at K = 1.. steps per pass
    FoldPartial* d_part;
    sw2d_red* d_ring;
    BatchControl* d_ctl;
    unsigned long long* d_flags;
    int n_tiles[kBlockMaxK];  // tiles of all members at K = 1.. steps per pass
    int tile_rows;            // R, rows per wave
    int cus;
    int resident;             // workgroups of the persistent launch that the device holds at once
    int grid;                 // the caller's, or the most it may ask for
    bool persistent;          // persistent launches: chosen by the caller, or too many tiles
    bool many_tiles;          // more than a launch per pass holds
    int steps_per_launch;
    int steps_per_pass;       // the caller's K, 1..kMaxBatchK: step counts are multiples of it
    bool use_graph;
    int64_t steps_done;
    int64_t passes_done;
    hipGraph_t graph;
    hipGraphExec_t exec;
    int graph_n;
    unsigned long long timeout_ticks;
};

namespace {

thread_local char g_batch_msg[256] = "";

int batch_hip_fail(hipError_t e, const char* what) {
    std::snprintf(g_batch_msg, sizeof g_batch_msg, "%s: %s", what, hipGetErrorString(e));
    sw2d::detail::set_hip_message(g_batch_msg);
    return SW2D_EHIP;
}

#define SW2D_BHIP(call)                                          \
    do {                                                         \
        hipError_t e_ = (call);                                  \
        if (e_ != hipSuccess) return batch_hip_fail(e_, #call);  \
    } while (0)

constexpr size_t kAlign = 256;
size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

struct BatchLayout {
    std::vector<size_t> hp;  // per instance
    size_t flags, scratch, inst, member, part, ring, ctl, gflags, total;
    int tile_rows;
    size_t map_tiles;  // tiles at every K together
    int n_tiles[kBlockMaxK];
};

constexpr int kMaxBatchGrid = 256 * 8;  // flag lines reserved: 8 workgroups on each of 256 CUs
// Resident workgroups per CU that the grid may count on. The occupancy query counts vector
// registers and LDS, but a SIMD of this family also holds at most 800 scalar registers, so a
// kernel near 100 SGPRs fits 7 waves per SIMD even when its vector registers would allow 8 (3
// workgroups of 8 waves per CU, not 4); a grid barrier that waits for a workgroup that never
// became resident would only end at its deadline.
constexpr int kBatchWgPerCu = 3;
// Workgroups per CU that a caller may ask for at K = 1, 2 and 3 steps per pass; a launch takes no more of
// them than are resident.
constexpr int kBatchGridPerCu[kMaxBatchK] = {6, 5, 4};
constexpr int kBatchRowsLow = 3, kBatchRowsMid = 5, kBatchRowsHigh = 8;  // rows per wave: tiles of 24, 40 and 64
constexpr int kBatchRows[3] = {kBatchRowsLow, kBatchRowsMid, kBatchRowsHigh};
constexpr int kBatchLowTiles = 320;    // most tiles of 24 rows chosen without the caller's word
constexpr int kBatchHighTiles = 2048;  // fewest tiles of 64 rows chosen without the caller's word

bool batch_layout(int n, const sw2d_params* p, const int32_t* band_rows, BatchLayout& L) {
    if (n < 1) return false;
    size_t off = 0;
    L.hp.resize(n);
    int64_t tiles[3][kBlockMaxK] = {};
    int64_t sum_rows = 0;
    for (int i = 0; i < n; ++i) {
        if (!sw2d::detail::params_valid(&p[i]) || p[i].flags != 0) return false;  // plain model only
        const int rows = band_rows ? band_rows[i] : 16;
        if (rows < kMinRows) return false;
        sum_rows += rows;
        L.hp[i] = off;
        off = align_up(off + (size_t)p[i].nx * p[i].ny * sizeof(float));
        for (int K = 1; K <= kBlockMaxK; ++K) {
            for (int r = 0; r < 3; ++r)
                tiles[r][K - 1] += make_block_geometry(p[i].nx, p[i].ny, K, kBatchRows[r]).nblocks;
            if (tiles[0][K - 1] > (1 << 28)) return false;
        }
    }
    // The tile height follows the band height: tiles of 24 rows for bands below 16 rows on average,
    // of 40 rows below 48, of 64 rows from there (they own 8, 24 and 48 rows at 4 steps per pass).
    // Without the caller's choice: the lowest while they all run at once, the highest where even those
    // take several rounds (their overlap is the least), 40 rows between. Us per step at 24, 40 and 64
    // rows: 12 members of 64-256 cells a side (391 low tiles) 3.1, 2.9, 3.8; 48 of them (1642 low, 306
    // high) 6.8, 5.4, 6.0; 4 of 701 x 523 (308 high) 6.9, 5.5, 6.1; 64 of 256^2 (960 high) 17.3, 10.9,
    // 10.3; 32 of 128-1024 (2581 high) 45.1, 28.4, 25.5; 256 of those 256, 165, 141. Below 320 low tiles
    // 12 smaller members took 145 us a call at 24 rows and 163 at 40. Between 960 and 2048 high tiles
    // the highest are up to 5 % faster than the 40 rows taken (16 of 128-1024, 1503 high: 15.5 and
    // 14.7); the line leaves a margin above the crossing, which moves with the members' sizes.
    int r = 1;
    if (band_rows)
        r = sum_rows < 16 * (int64_t)n ? 0 : sum_rows < 48 * (int64_t)n ? 1 : 2;
    else if (tiles[0][kBlockMaxK - 1] <= kBatchLowTiles)
        r = 0;
    else if (tiles[2][kBlockMaxK - 1] >= kBatchHighTiles)
        r = 2;
    L.tile_rows = kBatchRows[r];
    int most = 0;
    for (int K = 1; K <= kBlockMaxK; ++K) {
        L.n_tiles[K - 1] = (int)tiles[r][K - 1];
        most = std::max(most, K * L.n_tiles[K - 1]);
    }
    L.flags = off;
    off = align_up(off + (size_t)n * sizeof(PrepFlags));
    L.scratch = off;
    off = align_up(off + kHsumBlocks * sizeof(double));
    L.inst = off;
    off = align_up(off + (size_t)n * sizeof(BatchInst));
    L.member = off;
    L.map_tiles = 0;
    for (int K = 1; K <= kBlockMaxK; ++K) L.map_tiles += (size_t)L.n_tiles[K - 1];
    off = align_up(off + L.map_tiles * sizeof(int));
    L.part = off;
    off = align_up(off + 2 * (size_t)most * sizeof(FoldPartial));
    L.ring = off;
    off = align_up(off + (size_t)kBatchRing * n * sizeof(sw2d_red));
    L.ctl = off;
    off = align_up(off + sizeof(BatchControl));
    L.gflags = off;
    off = align_up(off + (size_t)kMaxBatchGrid * kFlagStride * sizeof(unsigned long long));
    L.total = off;
    return true;
}

// The batched kernel for K steps per pass and R rows per wave.
typedef void (*BatchKernel)(BatchArgs);

template <int R>
BatchKernel batch_kernel_of(int K) {
    switch (K) {
        case 1: return sw2d_batch_kernel<1, R>;
        case 2: return sw2d_batch_kernel<2, R>;
        case 3: return sw2d_batch_kernel<3, R>;
        default: return sw2d_batch_kernel<4, R>;
    }
}

BatchKernel batch_kernel(int K, int R) {
    return R == kBatchRowsLow   ? batch_kernel_of<kBatchRowsLow>(K)
           : R == kBatchRowsMid ? batch_kernel_of<kBatchRowsMid>(K)
                                : batch_kernel_of<kBatchRowsHigh>(K);
}

typedef void (*BatchPassKernel)(const BatchInst*, const int*, BatchPass);

template <int R>
BatchPassKernel batch_pass_kernel_of(int K) {
    switch (K) {
        case 1: return sw2d_batch_pass_kernel<1, R>;
        case 2: return sw2d_batch_pass_kernel<2, R>;
        case 3: return sw2d_batch_pass_kernel<3, R>;
        default: return sw2d_batch_pass_kernel<4, R>;
    }
}

BatchPassKernel batch_pass_kernel(int K, int R) {
    return R == kBatchRowsLow   ? batch_pass_kernel_of<kBatchRowsLow>(K)
           : R == kBatchRowsMid ? batch_pass_kernel_of<kBatchRowsMid>(K)
                                : batch_pass_kernel_of<kBatchRowsHigh>(K);
}

// Passes of a chunk of steps: as many of kBlockMaxK steps as it holds, one for the rest.
int chunk_passes(int32_t steps) { return steps / kBlockMaxK + (steps % kBlockMaxK != 0); }

// Steps per launch chunk: the caller's, rounded down to whole passes of its own K (all of a call's
// steps where every pass is a launch).
int32_t chunk_steps(const sw2d_bctx* b, int32_t nsteps) {
    if (!b->persistent) return nsteps;
    const int K = b->steps_per_pass;
    return b->steps_per_launch >= K ? b->steps_per_launch / K * K : K;
}

// nsteps steps, a launch per pass; the first `singles` of them one at a time.
int enqueue_passes(sw2d_bctx* b, int32_t nsteps, int singles, hipStream_t s) {
    BatchPass a{};
    a.inst = b->d_inst;
    a.ring = b->d_ring;
    a.ctl = b->d_ctl;
    a.n_inst = b->n;
    size_t most = 0;
    for (int K = 1; K <= kBlockMaxK; ++K) most = std::max(most, (size_t)K * b->n_tiles[K - 1]);
    auto fold_blocks = [&]() { return (b->n * a.fold_steps + kBlockWaves - 1) / kBlockWaves; };
    while (a.step < nsteps) {
        const int K = a.step < singles ? 1 : nsteps - a.step < kBlockMaxK ? nsteps - a.step : kBlockMaxK;
        a.member = b->d_member[K - 1];
        a.n_tiles = b->n_tiles[K - 1];
        a.part = b->d_part + (a.pass & 1) * most;
        hipLaunchKernelGGL(batch_pass_kernel(K, b->tile_rows), dim3(a.n_tiles + fold_blocks()), dim3(kBatchThreads), 0, s,
                           b->d_inst, a.member, a);
        SW2D_BHIP(hipGetLastError());
        a.prev_part = a.part;
        a.prev_tiles = a.n_tiles;
        a.fold_steps = K;
        a.step += K;
        a.pass += 1;
    }
    hipLaunchKernelGGL(sw2d_batch_fold_kernel, dim3(fold_blocks()), dim3(kBatchThreads), 0, s, a);
    SW2D_BHIP(hipGetLastError());
    hipLaunchKernelGGL(sw2d_batch_advance_kernel, dim3(1), dim3(1), 0, s, b->d_ctl, (int)nsteps, a.pass);
    SW2D_BHIP(hipGetLastError());
    return SW2D_OK;
}

// nsteps steps in chunks; the first `singles` (of the first chunk) one at a time.
int enqueue_chunks(sw2d_bctx* b, int32_t nsteps, int singles, hipStream_t s) {
    if (!b->persistent) return enqueue_passes(b, nsteps, singles, s);
    BatchArgs a;
    a.inst = b->d_inst;
    a.part = b->d_part;
    a.ring = b->d_ring;
    a.ctl = b->d_ctl;
    a.flags = b->d_flags;
    a.n_inst = b->n;
    a.timeout_ticks = b->timeout_ticks;
    auto launch = [&](int K, int32_t steps) -> int {  // in passes of K
        if (steps == 0) return SW2D_OK;
        a.steps = steps;
        a.n_tiles = b->n_tiles[K - 1];
        // no more workgroups than have tiles, or folds beside them, to do
        const int64_t useful = (int64_t)a.n_tiles + ((int64_t)b->n * K + kBlockWaves - 1) / kBlockWaves;
        const int grid = (int)std::min<int64_t>(useful, std::min(b->grid, b->resident));
        hipLaunchKernelGGL(batch_kernel(K, b->tile_rows), dim3(grid), dim3(kBatchThreads), 0, s, a);
        SW2D_BHIP(hipGetLastError());
        return SW2D_OK;
    };
    const int32_t per_launch = chunk_steps(b, nsteps);
    for (int32_t done = 0; done < nsteps;) {
        const int32_t chunk = nsteps - done < per_launch ? nsteps - done : per_launch;
        const int32_t rest = (chunk - singles) % kBlockMaxK;
        int rc = launch(1, singles);
        if (rc == SW2D_OK) rc = launch(kBlockMaxK, chunk - singles - rest);
        if (rc == SW2D_OK && rest > 0) rc = launch(rest, rest);
        if (rc) return rc;
        done += chunk;
        singles = 0;
    }
    return SW2D_OK;
}

// Workgroups of the tile kernels the device holds at once (capped, see kBatchWgPerCu): the least
// of the passes of every length.
int resident_grid(int R, int cus, int* out) {
    int least = kBatchWgPerCu;
    for (int K = 1; K <= kBlockMaxK; ++K) {
        int per_cu = 0;
        SW2D_BHIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(
            &per_cu, reinterpret_cast<const void*>(batch_kernel(K, R)), kBatchThreads, 0));
        if (per_cu < least) least = per_cu;
    }
    if (least < 1 || cus < 1) return SW2D_EINVAL;
    const int g = cus * least;
    *out = g < kMaxBatchGrid ? g : kMaxBatchGrid;
    return SW2D_OK;
}

// The largest grid that a caller may ask for.
int max_grid(const sw2d_bctx* b) { return std::min(b->cus * kBatchGridPerCu[b->steps_per_pass - 1], kMaxBatchGrid); }

void drop_graph(sw2d_bctx* b) {
    if (b->exec) (void)hipGraphExecDestroy(b->exec);
    if (b->graph) (void)hipGraphDestroy(b->graph);
    b->exec = nullptr;
    b->graph = nullptr;
    b->graph_n = -1;
}

}  // namespace

extern "C" {

size_t sw2d_batch_workspace_bytes(int32_t n, const sw2d_params* p, const int32_t* band_rows) {
    BatchLayout L;
    if (!p || !batch_layout(n, p, band_rows, L)) return 0;
    return L.total;
}

int sw2d_batch_create(int32_t n, const sw2d_params* p, const float* const* d_H,
                      const uint8_t* const* d_mask, float* const* d_state, const int32_t* band_rows,
                      void* d_work, size_t work_bytes, void* hip_stream, sw2d_batch_t* out) {
    if (!out) return SW2D_ESTATE;
    *out = nullptr;
    BatchLayout L;
    if (!p || !d_H || !d_mask || !d_state || !d_work || !batch_layout(n, p, band_rows, L))
        return SW2D_EINVAL;
    if (work_bytes < L.total) return SW2D_ENOSPC;
    if (reinterpret_cast<uintptr_t>(d_work) % kAlign != 0) return SW2D_EINVAL;
    for (int i = 0; i < n; ++i)
        if (!d_H[i] || !d_mask[i] || !d_state[i]) return SW2D_EINVAL;

    sw2d_bctx* b = new (std::nothrow) sw2d_bctx();
    if (!b) return SW2D_ESTATE;
    b->n = n;
    b->p.assign(p, p + n);
    b->stream = static_cast<hipStream_t>(hip_stream);
    b->capture = nullptr;
    b->graph = nullptr;
    b->exec = nullptr;
    b->graph_n = -1;
    // a launch holds fewer than 2^32 threads
    b->many_tiles = false;
    for (int K = 1; K <= kBlockMaxK; ++K)
        if ((int64_t)L.n_tiles[K - 1] + ((int64_t)n * kBlockMaxK + kBlockWaves - 1) / kBlockWaves >= (1 << 23))
            b->many_tiles = true;
    b->persistent = b->many_tiles;
    b->steps_per_launch = 50;
    b->use_graph = true;
    b->steps_done = 0;
    std::copy(L.n_tiles, L.n_tiles + kBlockMaxK, b->n_tiles);
    b->tile_rows = L.tile_rows;
    char* w = static_cast<char*>(d_work);
    b->d_inst = reinterpret_cast<BatchInst*>(w + L.inst);
    int* map = reinterpret_cast<int*>(w + L.member);
    for (int K = 1; K <= kBlockMaxK; ++K) {
        b->d_member[K - 1] = map;
        map += L.n_tiles[K - 1];
    }
    b->d_flags = reinterpret_cast<unsigned long long*>(w + L.gflags);
    b->d_part = reinterpret_cast<FoldPartial*>(w + L.part);
    b->d_ring = reinterpret_cast<sw2d_red*>(w + L.ring);
    b->d_ctl = reinterpret_cast<BatchControl*>(w + L.ctl);
    PrepFlags* d_flags = reinterpret_cast<PrepFlags*>(w + L.flags);
    double* d_scratch = reinterpret_cast<double*>(w + L.scratch);

    auto fail = [&](int rc) {
        if (b->capture) (void)hipStreamDestroy(b->capture);
        delete b;
        return rc;
    };

    std::vector<PrepFlags> flags(n, PrepFlags{0u, 0u, 0.0});
    hipError_t e = hipMemcpyAsync(d_flags, flags.data(), n * sizeof(PrepFlags), hipMemcpyHostToDevice,
                                  b->stream);
    b->state.resize((size_t)n * 6);
    for (int i = 0; i < n && e == hipSuccess; ++i) {
        const size_t cells = (size_t)p[i].nx * p[i].ny;
        for (int f = 0; f < 6; ++f) b->state[(size_t)i * 6 + f] = d_state[i] + f * cells;
        e = launch_prep(d_H[i], d_mask[i], d_state[i], d_state[i] + cells, d_state[i] + 2 * cells,
                        p[i].nx, p[i].ny, reinterpret_cast<float*>(w + L.hp[i]), d_flags + i, d_scratch,
                        b->stream);
    }
    if (e == hipSuccess)
        e = hipMemcpyAsync(flags.data(), d_flags, n * sizeof(PrepFlags), hipMemcpyDeviceToHost, b->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(b->stream);
    if (e != hipSuccess) return fail(batch_hip_fail(e, "sw2d_batch_create"));

    std::vector<BatchInst> inst(n);
    int tile_begin[kBlockMaxK] = {};
    for (int i = 0; i < n; ++i) {
        if (flags[i].bad != 0 || flags[i].hmax_bits == 0) return fail(SW2D_EINVAL);
        float hmax;
        std::memcpy(&hmax, &flags[i].hmax_bits, sizeof hmax);
        const sw2d_params& q = p[i];
        const double courant =
            q.dt * std::sqrt(q.g * (double)hmax) * std::sqrt(1.0 / (q.dx * q.dx) + 1.0 / (q.dy * q.dy));
        if (!(courant <= 1.0)) return fail(SW2D_EINVAL);
        BatchInst& in = inst[i];
        in.hp = reinterpret_cast<const float*>(w + L.hp[i]);
        const size_t cells = (size_t)q.nx * q.ny;
        for (int buf = 0; buf < 2; ++buf)
            for (int f = 0; f < 3; ++f) in.state[buf][f] = d_state[i] + (size_t)(3 * buf + f) * cells;
        in.nx = q.nx;
        in.ny = q.ny;
        in.k = sw2d::detail::make_coef(&q);
        in.cell_area = q.dx * q.dy;
        in.h_sum = flags[i].h_sum;
        for (int K = 1; K <= kBlockMaxK; ++K) {
            const BlockGeometry g = make_block_geometry(q.nx, q.ny, K, b->tile_rows);
            in.t[K - 1] = BatchTiles{g.strips, g.bands, tile_begin[K - 1]};
            tile_begin[K - 1] += g.nblocks;
        }
    }
    std::vector<int> member;
    member.reserve(L.map_tiles);
    for (int K = 1; K <= kBlockMaxK; ++K)
        for (int i = 0; i < n; ++i) member.insert(member.end(), (size_t)inst[i].t[K - 1].strips * inst[i].t[K - 1].bands, i);
    b->steps_per_pass = 1;
    b->passes_done = 0;
    BatchControl ctl;
    std::memset(&ctl, 0, sizeof ctl);
    std::vector<unsigned long long> zero_flags((size_t)kMaxBatchGrid * kFlagStride, 0ull);
    e = hipMemcpyAsync(b->d_inst, inst.data(), n * sizeof(BatchInst), hipMemcpyHostToDevice, b->stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync(b->d_member[0], member.data(), member.size() * sizeof(int), hipMemcpyHostToDevice, b->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(b->d_ctl, &ctl, sizeof ctl, hipMemcpyHostToDevice, b->stream);
    if (e == hipSuccess)
        e = hipMemcpyAsync(b->d_flags, zero_flags.data(), zero_flags.size() * sizeof(unsigned long long),
                           hipMemcpyHostToDevice, b->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(b->stream);
    if (e != hipSuccess) return fail(batch_hip_fail(e, "sw2d_batch_create upload"));

    // persistent grid: no more workgroups than the device can hold at once
    int dev = 0, clock_khz = 0;
    e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&clock_khz, hipDeviceAttributeWallClockRate, dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&b->cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return fail(batch_hip_fail(e, "device query"));
    const int rc = resident_grid(b->tile_rows, b->cus, &b->resident);
    if (rc) return fail(rc);
    b->grid = max_grid(b);
    if (clock_khz <= 0) clock_khz = 100000;
    b->timeout_ticks = (unsigned long long)clock_khz * 1000ull * 2ull;  // 2 s per barrier
    e = hipStreamCreateWithFlags(&b->capture, hipStreamNonBlocking);
    if (e != hipSuccess) return fail(batch_hip_fail(e, "hipStreamCreateWithFlags"));
    *out = b;
    return SW2D_OK;
}

int sw2d_batch_set_time_blocking(sw2d_batch_t b, int32_t steps_per_pass) {
    if (!b) return SW2D_ESTATE;
    if (steps_per_pass < 1 || steps_per_pass > kMaxBatchK) return SW2D_EINVAL;
    if (steps_per_pass == b->steps_per_pass) return SW2D_OK;
    b->steps_per_pass = steps_per_pass;
    b->grid = std::min(b->grid, max_grid(b));
    drop_graph(b);
    return SW2D_OK;
}

int32_t sw2d_batch_time_blocking(sw2d_batch_t b) { return b ? b->steps_per_pass : -1; }

int sw2d_batch_set_launch(sw2d_batch_t b, int32_t steps_per_launch, int32_t use_graph, int32_t grid) {
    if (!b) return SW2D_ESTATE;
    if (steps_per_launch < 1 || grid < 0) return SW2D_EINVAL;
    if (grid > max_grid(b)) return SW2D_EINVAL;
    b->grid = grid > 0 ? grid : max_grid(b);
    b->persistent = grid > 0 || b->many_tiles;
    b->steps_per_launch = steps_per_launch;
    b->use_graph = use_graph != 0;
    drop_graph(b);
    return SW2D_OK;
}

int sw2d_batch_step(sw2d_batch_t b, int32_t nsteps) {
    if (!b || nsteps < 0) return SW2D_ESTATE;
    if (nsteps == 0) return SW2D_OK;
    if (nsteps % b->steps_per_pass != 0) return SW2D_EINVAL;
    const int32_t per_launch = chunk_steps(b, nsteps);
    int64_t passes = (int64_t)(nsteps / per_launch) * chunk_passes(per_launch) + chunk_passes(nsteps % per_launch);
    if (!b->use_graph) {
        // under the caller's capture the passes keep the parity of passes of the caller's K, so that the
        // buffer of sw2d_batch_state stays the current one over replays
        int singles = 0;
        if ((passes - nsteps / b->steps_per_pass) % 2 != 0 && captured(b->stream)) {
            const int32_t first = nsteps < per_launch ? nsteps : per_launch;
            singles = single_steps(first, kBlockMaxK, chunk_passes(first) % 2 == 0);
            ++passes;
        }
        int rc = enqueue_chunks(b, nsteps, singles, b->stream);
        if (rc) return rc;
    } else {
        if (b->graph_n != nsteps) {
            drop_graph(b);
            SW2D_BHIP(hipStreamBeginCapture(b->capture, hipStreamCaptureModeThreadLocal));
            int rc = enqueue_chunks(b, nsteps, 0, b->capture);
            hipGraph_t g = nullptr;
            hipError_t e = hipStreamEndCapture(b->capture, &g);
            if (rc) {
                if (g) (void)hipGraphDestroy(g);
                return rc;
            }
            if (e != hipSuccess) return batch_hip_fail(e, "hipStreamEndCapture");
            b->graph = g;
            e = hipGraphInstantiate(&b->exec, g, nullptr, nullptr, 0);
            if (e != hipSuccess) {
                drop_graph(b);
                return batch_hip_fail(e, "hipGraphInstantiate");
            }
            b->graph_n = nsteps;
        }
        SW2D_BHIP(hipGraphLaunch(b->exec, b->stream));
    }
    b->steps_done += nsteps;
    b->passes_done += passes;
    return SW2D_OK;
}

int sw2d_batch_step_timed(sw2d_batch_t b, int32_t nsteps, double* ms_per_step) {
    if (!b || nsteps < 1 || !ms_per_step) return SW2D_ESTATE;
    hipEvent_t e0, e1;
    SW2D_BHIP(hipEventCreate(&e0));
    hipError_t e = hipEventCreate(&e1);
    if (e != hipSuccess) {
        (void)hipEventDestroy(e0);
        return batch_hip_fail(e, "hipEventCreate");
    }
    int rc = SW2D_OK;
    e = hipEventRecord(e0, b->stream);
    if (e == hipSuccess) rc = sw2d_batch_step(b, nsteps);
    if (e == hipSuccess && rc == SW2D_OK) e = hipEventRecord(e1, b->stream);
    if (e == hipSuccess && rc == SW2D_OK) e = hipEventSynchronize(e1);
    float ms = 0.f;
    if (e == hipSuccess && rc == SW2D_OK) e = hipEventElapsedTime(&ms, e0, e1);
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (rc) return rc;
    if (e != hipSuccess) return batch_hip_fail(e, "sw2d_batch_step_timed");
    *ms_per_step = (double)ms / nsteps;
    return SW2D_OK;
}

int sw2d_batch_reduce(sw2d_batch_t b, sw2d_red* host_out) {
    if (!b || !host_out) return SW2D_ESTATE;
    if (b->steps_done < 1) return SW2D_ESTATE;
    BatchControl ctl;
    SW2D_BHIP(hipMemcpyAsync(&ctl, b->d_ctl, sizeof ctl, hipMemcpyDeviceToHost, b->stream));
    const size_t slot = (size_t)((b->steps_done - 1) % kBatchRing);
    SW2D_BHIP(hipMemcpyAsync(host_out, b->d_ring + slot * b->n, (size_t)b->n * sizeof(sw2d_red),
                             hipMemcpyDeviceToHost, b->stream));
    SW2D_BHIP(hipStreamSynchronize(b->stream));
    if (ctl.error != 0) {
        std::snprintf(g_batch_msg, sizeof g_batch_msg, "grid barrier wait ran past its deadline");
        sw2d::detail::set_hip_message(g_batch_msg);
        return SW2D_EHIP;
    }
    if (ctl.steps_done != b->steps_done) return SW2D_ESTATE;
    (void)kBatchRing;
    for (int i = 0; i < b->n; ++i) {
        const sw2d_red& r = host_out[i];
        if (!std::isfinite(r.vol_total) || !std::isfinite(r.vol_disp) || !std::isfinite(r.max_abs_u) ||
            !std::isfinite(r.max_abs_v))
            return SW2D_EUNSTABLE;
    }
    return SW2D_OK;
}

int sw2d_batch_state(sw2d_batch_t b, int32_t k, float** d_eta, float** d_u, float** d_v) {
    if (!b || k < 0 || k >= b->n) return SW2D_ESTATE;
    const int cur = (int)(b->passes_done & 1);
    float* const* s = &b->state[(size_t)k * 6 + 3 * cur];
    if (d_eta) *d_eta = s[0];
    if (d_u) *d_u = s[1];
    if (d_v) *d_v = s[2];
    return SW2D_OK;
}

int64_t sw2d_batch_steps_done(sw2d_batch_t b) { return b ? b->steps_done : -1; }

int sw2d_batch_set_barrier_timeout(sw2d_batch_t b, double seconds) {
    if (!b || !(seconds >= 0.0) || seconds > 60.0) return SW2D_EINVAL;
    int dev = 0, clock_khz = 0;
    SW2D_BHIP(hipGetDevice(&dev));
    SW2D_BHIP(hipDeviceGetAttribute(&clock_khz, hipDeviceAttributeWallClockRate, dev));
    if (clock_khz <= 0) clock_khz = 100000;
    b->timeout_ticks = (unsigned long long)(seconds * clock_khz * 1000.0);
    b->persistent = true;  // only a persistent launch has a barrier to wait at
    drop_graph(b);
    return SW2D_OK;
}

int32_t sw2d_batch_grid(sw2d_batch_t b) { return b ? b->grid : -1; }

int sw2d_batch_destroy(sw2d_batch_t b) {
    if (!b) return SW2D_OK;
    drop_graph(b);
    if (b->capture) (void)hipStreamDestroy(b->capture);
    delete b;
    return SW2D_OK;
}

}  // extern "C"
