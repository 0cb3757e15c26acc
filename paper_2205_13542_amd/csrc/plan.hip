// Plan building for BEV pooling: the camera-fixed point-to-cell association
// (BEVFusion, arXiv 2205.13542, Sec. III-B, "Precomputation" paragraph:
// compute each frustum point's 3-D coordinate and grid index once, sort the
// points by grid index and record their ranks).
//
// Kernels, in launch order:
//   k_project      one thread per point: camera ray -> ego frame -> cell id
//   k_radix_hist   } stable LSD radix sort of (cell, point id), digits of
//                  } at most 9 bits; the first pass reads the cells themselves,
//   k_scan...      } in id order, so ties stay in id order (scans: one
//   k_radix_scatter} workgroup for a short array, else chunk sums and
//                    per-chunk scans from the sums before)
//   k_cell_start   interval table from the sorted keys
//   k_cell_stats   non-empty cells and the largest interval
//   k_combo_walk ... k_generic_runs   work partition of the forward pass:
//                  clean combos, the column table, empty cells, the
//                  partial-sum slots of multi-combo cells, generic cells and
//                  their runs
//
// The geometry is evaluated in IEEE double with the file built without
// floating-point contraction, in one fixed expression order, so the cell ids
// equal those of any plain CPU evaluation of the same expressions.
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <mutex>
#include <utility>

#include "internal.h"

#pragma clang fp contract(off)

namespace bevpool {
namespace {

constexpr int kSortItems = 8;                       // keys per thread per tile
constexpr int kSortTile = kBlock * kSortItems;      // 2048 keys per workgroup
constexpr int kWaveItems = kWaveSize * kSortItems;  // 512 keys per wave
constexpr int kRadixBits = 9;                       // digit bits per pass, at most
constexpr int kRadixBins = 1 << kRadixBits;         // 512 digits, at most two per thread

// A sort on `bits` key bits takes the fewest passes of at most kRadixBits
// bits, with the bits split evenly over them (17-bit cell ids: two passes of
// 9; 19 bits: three of 7, whose 128-digit histograms are cheaper than 512).
constexpr int radix_passes(int bits) { return (bits + kRadixBits - 1) / kRadixBits; }
constexpr int radix_digit_bits(int bits) {
    return (bits + radix_passes(bits) - 1) / radix_passes(bits);
}
constexpr int kScanBlock = 1024;
constexpr int kScanItems = 4;
constexpr int kScanChunk = kScanBlock * kScanItems;  // elements per workgroup of a multi-block scan
constexpr int kScanOneBlockChunks = 2;               // scans of up to 2 chunks take one workgroup
constexpr int kScanBlocks = 1024;                    // workgroups of a multi-block scan, at most
static_assert(kBlock == 256, "a sort tile is four waves of 512 keys");

constexpr int kArgCams = 16;   // cameras whose calibration travels in the kernel arguments

struct ProjectArgs {
    const double *intr;  // [N][4] in device memory, or null: the calibration is in cal
    const double *extr;  // [N][12]
    double cal[kArgCams * 16];   // [N][4] intrinsics, then [N][12] extrinsics (intr null)
    bevpool_geometry g;
    FastDiv div_w, div_h, div_b;   // div_b: blocks of kProjectBins depth bins
    int32_t n_threads, n_blocks, nz;
    int32_t *cell_of_point;
};
constexpr int kProjectBins = 4;

// Sec. III-B, first paragraph: the pixel's ray at depth bin d, in the ego
// frame, quantised at the cell size, z like x and y; points outside the grid
// or the nz stacked z slabs are dropped. Cell id (iy * nx + ix) * nz + iz.
// One thread per pixel and kProjectBins depth bins, whose points share the
// pixel's two quotients: the fp64 divisions are what the kernel spends its time
// on, five for each point otherwise, here three (16.0 -> 12.6 us for 2 M points,
// with the sort's keys and ids no longer written here).
__global__ __launch_bounds__(kBlock) void k_project(ProjectArgs a) {
    const int32_t x = blockIdx.x * kBlock + threadIdx.x;
    if (x >= a.n_threads) return;
    const bevpool_geometry &g = a.g;
    const uint32_t q_w = fdiv(uint32_t(x), a.div_w);
    const int w = x - int(q_w) * g.feat_w;
    const uint32_t q_h = fdiv(q_w, a.div_h);
    const int h = int(q_w) - int(q_h) * g.feat_h;
    const int n = int(fdiv(q_h, a.div_b));
    const int d0 = (int(q_h) - n * a.n_blocks) * kProjectBins;

    const double *I = a.intr ? a.intr + 4 * n : a.cal + 4 * n;
    const double *E = a.intr ? a.extr + 12 * n : a.cal + 4 * g.n_cams + 12 * n;
    const double fx = I[0], fy = I[1], cx = I[2], cy = I[3];
    const double u = double(w) + g.pixel_offset;
    const double v = double(h) + g.pixel_offset;
    const double ru = (u - cx) / fx;
    const double rv = (v - cy) / fy;
#pragma unroll
    for (int k = 0; k < kProjectBins; ++k) {
        const int d = d0 + k;
        if (d >= g.n_depth) break;
        const double depth = g.depth_min + double(d) * g.depth_step;
        const double xc = depth * ru;
        const double yc = depth * rv;
        const double zc = depth;
        const double X = ((E[0] * xc + E[1] * yc) + E[2] * zc) + E[3];
        const double Y = ((E[4] * xc + E[5] * yc) + E[6] * zc) + E[7];
        const double Z = ((E[8] * xc + E[9] * yc) + E[10] * zc) + E[11];
        const double qx = floor((X - g.x_min) / g.cell_x);
        const double qy = floor((Y - g.y_min) / g.cell_y);
        const double qz = floor((Z - g.z_min) / g.z_cell);
        int32_t cell = -1;
        if (qx >= 0.0 && qx < double(g.nx) && qy >= 0.0 && qy < double(g.ny) && qz >= 0.0 &&
            qz < double(a.nz))
            cell = (int32_t(qy) * g.nx + int32_t(qx)) * a.nz + int32_t(qz);
        a.cell_of_point[((int64_t(n) * g.n_depth + d) * g.feat_h + h) * g.feat_w + w] = cell;
    }
}

// ---------------------------------------------------------------- scan

// Exclusive scan of one value per thread across the block; *total gets the
// block sum. Uses wave shuffles, then one LDS slot per wave.
template <int BLOCK>
__device__ __forceinline__ int block_exclusive_scan(int v, int *lds, int *total) {
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int wave = threadIdx.x / kWaveSize;
    int x = v;
#pragma unroll
    for (int off = 1; off < kWaveSize; off <<= 1) {
        const int y = __shfl_up(x, off, kWaveSize);
        if (lane >= off) x += y;
    }
    if (lane == kWaveSize - 1) lds[wave] = x;
    __syncthreads();
    int before = 0, sum = 0;
#pragma unroll
    for (int w = 0; w < BLOCK / kWaveSize; ++w) {
        const int s = lds[w];
        before += (w < wave) ? s : 0;
        sum += s;
    }
    __syncthreads();
    *total = sum;
    return before + x - v;
}

// In-place exclusive scan of data[0..n) by a single workgroup (plan-time
// only; sizes are at most a few million). *total receives the sum.
__global__ __launch_bounds__(kScanBlock) void k_scan(int32_t *data, int64_t n, int32_t *total) {
    __shared__ int lds[kScanBlock / kWaveSize];
    int carry = 0;
    for (int64_t base = 0; base < n; base += int64_t(kScanBlock) * kScanItems) {
        const int64_t i0 = base + int64_t(threadIdx.x) * kScanItems;
        int v[kScanItems];
        int local = 0;
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            v[k] = (i0 + k < n) ? data[i0 + k] : 0;
            local += v[k];
        }
        int blocksum;
        int run = carry + block_exclusive_scan<kScanBlock>(local, lds, &blocksum);
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            if (i0 + k < n) data[i0 + k] = run;
            run += v[k];
        }
        carry += blocksum;
    }
    if (threadIdx.x == 0 && total) *total = carry;
}

// Multi-block exclusive scan, for arrays longer than a few chunks: each
// workgroup sums its chunks, then each adds up the sums before its own (few,
// and in cache) and scans its chunks from there. Up to kScanJobs arrays are
// scanned by one pair of launches (grid y): the three scans of a classification
// took nine launches, each 2 to 5 us.
constexpr int kScanJobs = 3;
struct ScanJob {
    int32_t *data;
    int64_t n;
    int32_t *total;     // receives the sum; may be null
    int32_t *sums;      // kScanBlocks ints
    int32_t blocks;     // workgroups
    int32_t chunks;     // chunks of each
};
struct ScanArgs {
    ScanJob job[kScanJobs];
};

__global__ __launch_bounds__(kScanBlock) void k_scan_sums(ScanArgs args) {
    __shared__ int lds[kScanBlock / kWaveSize];
    const ScanJob a = args.job[blockIdx.y];
    if (int(blockIdx.x) >= a.blocks) return;
    int local = 0;
    for (int c = 0; c < a.chunks; ++c) {
        const int64_t i0 = (int64_t(blockIdx.x) * a.chunks + c) * kScanChunk + int64_t(threadIdx.x) * kScanItems;
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) local += (i0 + k < a.n) ? a.data[i0 + k] : 0;
    }
    int total;
    (void)block_exclusive_scan<kScanBlock>(local, lds, &total);
    if (threadIdx.x == 0) a.sums[blockIdx.x] = total;
}

__global__ __launch_bounds__(kScanBlock) void k_scan_apply(ScanArgs args) {
    __shared__ int lds[kScanBlock / kWaveSize];
    const ScanJob a = args.job[blockIdx.y];
    if (int(blockIdx.x) >= a.blocks) return;
    static_assert(kScanBlocks <= kScanBlock, "a thread per sum");
    int carry;
    (void)block_exclusive_scan<kScanBlock>(threadIdx.x < blockIdx.x ? a.sums[threadIdx.x] : 0, lds, &carry);
    for (int c = 0; c < a.chunks; ++c) {
        const int64_t i0 = (int64_t(blockIdx.x) * a.chunks + c) * kScanChunk + int64_t(threadIdx.x) * kScanItems;
        int v[kScanItems];
        int local = 0;
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            v[k] = (i0 + k < a.n) ? a.data[i0 + k] : 0;
            local += v[k];
        }
        int total;
        int run = carry + block_exclusive_scan<kScanBlock>(local, lds, &total);
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            if (i0 + k < a.n) a.data[i0 + k] = run;
            run += v[k];
        }
        carry += total;
    }
    if (a.total && threadIdx.x == 0 && int(blockIdx.x) == a.blocks - 1) *a.total = carry;
}

// ---------------------------------------------------------------- radix sort

// Digit histogram of each tile, stored digit-major:
// hist[digit * n_tiles + tile], so an exclusive scan of the whole array
// gives every (digit, tile) its first output slot in stable order.
// Digit counts of one tile: hist[digit * tiles + tile], digits of dbits
// bits (dbits <= kRadixBits) from bit `shift` on.
// With CELLS the keys are the points' cells as projected (the sort's first
// pass): a dropped point's -1 counts as n_cells, which comes last, and the
// values are the positions themselves, so neither is written beforehand.
template <bool CELLS>
__device__ __forceinline__ uint32_t sort_key(const uint32_t *keys, int64_t i, int32_t n_cells) {
    const uint32_t k = keys[i];
    return CELLS ? min(k, uint32_t(n_cells)) : k;
}

template <bool CELLS>
__global__ __launch_bounds__(kBlock) void k_radix_hist(const uint32_t *keys, int32_t n, int32_t n_cells,
                                                       int shift, int dbits, int32_t *hist) {
    __shared__ int cnt[kRadixBins];
    const int bins = 1 << dbits;
    const uint32_t mask = uint32_t(bins) - 1u;
    for (int d = threadIdx.x; d < bins; d += kBlock) cnt[d] = 0;
    __syncthreads();
    const int64_t base = int64_t(blockIdx.x) * kSortTile;
#pragma unroll
    for (int k = 0; k < kSortItems; ++k) {
        const int64_t i = base + int64_t(k) * kBlock + threadIdx.x;
        if (i < n) atomicAdd(&cnt[(sort_key<CELLS>(keys, i, n_cells) >> shift) & mask], 1);
    }
    __syncthreads();
    for (int d = threadIdx.x; d < bins; d += kBlock)
        hist[int64_t(d) * gridDim.x + blockIdx.x] = cnt[d];
}

// Stable scatter. Wave w of a tile owns keys [w, w + 1) * kWaveItems of the tile
// and walks them 64 at a time in order. Within a step, a key's rank among
// equal digits comes from one ballot per digit bit: lanes whose ballots
// agree on every bit hold the same digit. A per-wave LDS counter per
// digit carries ranks across steps. Per-wave counts are then prefixed across
// the waves and added to the scanned global offsets.
template <bool CELLS>
__global__ __launch_bounds__(kBlock) void k_radix_scatter(const uint32_t *keys_in,
                                                          const int32_t *vals_in, int32_t n,
                                                          int32_t n_cells, int shift, int dbits,
                                                          const int32_t *hist_scan,
                                                          uint32_t *keys_out, int32_t *vals_out) {
    __shared__ int wcount[kWaves][kRadixBins];
    __shared__ int gbase[kRadixBins];
    const int bins = 1 << dbits;
    const uint32_t mask = uint32_t(bins) - 1u;
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int wave = threadIdx.x / kWaveSize;
    for (int d = threadIdx.x; d < bins; d += kBlock) {
#pragma unroll
        for (int w = 0; w < kWaves; ++w) wcount[w][d] = 0;
        gbase[d] = hist_scan[int64_t(d) * gridDim.x + blockIdx.x];
    }
    __syncthreads();

    const int64_t base = int64_t(blockIdx.x) * kSortTile + int64_t(wave) * kWaveItems;
    const uint64_t lanes_below = (uint64_t(1) << lane) - 1;
    uint32_t key[kSortItems];
    int32_t val[kSortItems];
    int rank[kSortItems];
#pragma unroll
    for (int k = 0; k < kSortItems; ++k) {
        const int64_t i = base + int64_t(k) * kWaveSize + lane;
        const bool valid = i < n;
        key[k] = valid ? sort_key<CELLS>(keys_in, i, n_cells) : 0u;
        val[k] = CELLS ? int32_t(i) : valid ? vals_in[i] : 0;
        const uint32_t digit = (key[k] >> shift) & mask;
        uint64_t same = __ballot(valid);
#pragma unroll
        for (int b = 0; b < kRadixBits; ++b) {
            if (b < dbits) {   // uniform over the workgroup
                const bool bit = (digit >> b) & 1u;
                const uint64_t ones = __ballot(bit);
                same &= bit ? ones : ~ones;
            }
        }
        const int before = __popcll(same & lanes_below);
        const int prior = wcount[wave][digit];
        rank[k] = prior + before;
        __builtin_amdgcn_wave_barrier();
        // the highest lane of each digit group advances the wave's counter
        if (valid && (same >> lane) == 1u) wcount[wave][digit] = prior + __popcll(same);
        __builtin_amdgcn_wave_barrier();
    }
    __syncthreads();
    for (int d = threadIdx.x; d < bins; d += kBlock) {
        int run = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const int c = wcount[w][d];
            wcount[w][d] = run;
            run += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kSortItems; ++k) {
        const int64_t i = base + int64_t(k) * kWaveSize + lane;
        if (i < n) {
            const uint32_t digit = (key[k] >> shift) & mask;
            const int64_t pos = int64_t(gbase[digit]) + wcount[wave][digit] + rank[k];
            keys_out[pos] = key[k];
            vals_out[pos] = val[k];
        }
    }
}

// ---------------------------------------------------------------- interval table

// cell_start[c] = number of kept points with cell < c, for c in [0, n_cells].
// Sorted keys are the kept cells, then n_cells for every dropped point. Slot
// i (0..n) fills the cells in (key[i-1], key[i]] with i; each entry of
// cell_start is written by exactly one slot.
// A thread takes kStartItems slots, whose keys it reads as one piece (skeys is
// 16-byte aligned). Runs of more than kStartRun empty cells (rows of the grid
// that no camera sees) are filled by the whole wave: by one thread they were
// what the kernel waited for (9.1 us of a nuScenes-shaped build, now 4.0).
constexpr int kStartItems = 4;
constexpr int kStartRun = 16;
__global__ __launch_bounds__(kBlock) void k_cell_start(const uint32_t *skeys, int32_t n,
                                                       int32_t n_cells, int32_t *cell_start) {
    const int64_t i0 = (int64_t(blockIdx.x) * kBlock + threadIdx.x) * kStartItems;
    uint32_t key[kStartItems];
    if (i0 + kStartItems <= n) {
        const uint4 v = *reinterpret_cast<const uint4 *>(skeys + i0);
        key[0] = v.x;
        key[1] = v.y;
        key[2] = v.z;
        key[3] = v.w;
    } else {
#pragma unroll
        for (int k = 0; k < kStartItems; ++k) key[k] = i0 + k < n ? skeys[i0 + k] : uint32_t(n_cells);
    }
    int32_t prev = i0 == 0 ? -1 : i0 <= n ? int32_t(skeys[i0 - 1]) : n_cells;
    // long runs of empty cells (whole rows of the grid) are filled by the wave
    const int lane = threadIdx.x & (kWaveSize - 1);
#pragma unroll
    for (int k = 0; k < kStartItems; ++k) {
        const bool in = i0 + k <= n;
        const int32_t last = in ? int32_t(key[k]) : prev;
        const bool wide = last - prev > kStartRun;
        if (!wide)
            for (int32_t c = prev + 1; c <= last; ++c) cell_start[c] = int32_t(i0 + k);
        for (uint64_t rest = __ballot(wide); rest != 0; rest &= rest - 1) {
            const int from = __builtin_ctzll(rest);
            const int32_t hi = __shfl(last, from), v = __shfl(int32_t(i0 + k), from);
            for (int32_t c = __shfl(prev, from) + 1 + lane; c <= hi; c += kWaveSize) cell_start[c] = v;
        }
        prev = last;
    }
}

// Counters shared by the whole grid (counts, maxima) are reduced in the
// workgroup first and updated by one atomic per workgroup, and the kernels
// that update them run a capped grid over their elements: atomics on one
// address are performed one after another, about 11 ns each, so one per wave
// (what the compiler makes of per-thread updates) would cost tens of
// microseconds. Each counter is kept in kShards words on cache lines of their
// own, which workgroups update in turn; the host adds them up (or takes the
// largest).
constexpr int kReduceBlocks = 256;
constexpr int kShards = 8;
constexpr int kCounters = 16;      // counters of a shard: 64 bytes

__device__ __forceinline__ int32_t *shard(int32_t *counters, int id) {
    return counters + (blockIdx.x % kShards) * kCounters + id;
}

// Counters [first, first + 2) of every shard to zero (2 * kShards threads).
__device__ __forceinline__ void clear_pair(int32_t *counters, int first, int t) {
    if (t < 2 * kShards) counters[t / 2 * kCounters + first + t % 2] = 0;
}

__global__ void k_clear_pair(int32_t *counters, int first) { clear_pair(counters, first, int(threadIdx.x)); }

// Workgroup sum (MAX: maximum) of one value per thread; every thread of the
// workgroup calls it, the result is valid in thread 0. s_red holds kWaves
// words and is not reused by another call before a barrier.
template <bool MAX>
__device__ __forceinline__ int32_t block_reduce(int32_t v, int32_t *s_red) {
#pragma unroll
    for (int o = kWaveSize / 2; o > 0; o >>= 1) {
        const int32_t u = __shfl_xor(v, o, kWaveSize);
        v = MAX ? max(v, u) : v + u;
    }
    if ((threadIdx.x & (kWaveSize - 1)) == 0) s_red[threadIdx.x / kWaveSize] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 1; w < kWaves; ++w) v = MAX ? max(v, s_red[w]) : v + s_red[w];
    }
    return v;
}

// Non-empty cells and the largest interval into counters 0 and 1, the kept
// count (cell_start[n_cells]) into counter 10; clears two per-cell arrays
// (the combo walk's counters) on the way.
__global__ __launch_bounds__(kBlock) void k_cell_stats(const int32_t *cell_start, int32_t n_cells,
                                                       int32_t *stats,
                                                       int32_t *clear_a, int32_t *clear_b) {
    __shared__ int32_t s_n[kWaves], s_m[kWaves];
    if (blockIdx.x == 0 && threadIdx.x == 0) stats[10] = cell_start[n_cells];
    int32_t nonempty = 0, most = 0;
    for (int32_t c = blockIdx.x * kBlock + threadIdx.x; c < n_cells; c += gridDim.x * kBlock) {
        clear_a[c] = 0;
        clear_b[c] = 0;
        const int32_t cnt = cell_start[c + 1] - cell_start[c];
        nonempty += cnt > 0 ? 1 : 0;
        most = max(most, cnt);
    }
    nonempty = block_reduce<false>(nonempty, s_n);
    most = block_reduce<true>(most, s_m);
    if (threadIdx.x == 0) {
        if (nonempty > 0) atomicAdd(shard(stats, 0), nonempty);
        if (most > 0) atomicMax(shard(stats, 1), most);
    }
}


// ---------------------------------------------------------------- work partition
//
// Combos, items and cell classes as described in internal.h. Every kernel
// below is a plain per-element pass; ordering comes from scans and the
// stable radix sort only, so the partition is deterministic.

__global__ __launch_bounds__(kBlock) void k_fill(int32_t *p, int64_t n, int32_t v) {
    const int64_t i = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (i < n) p[i] = v;
}

struct ComboArgs {
    const int32_t *cell_of_point;
    int32_t N, D, H, W;
    int32_t allow_clean;        // 0 when rows do not fit the packed row range
    int32_t *combo_cell;        // [N*D*W]: cell of a clean combo, -1 none kept, -2 not clean
    int32_t *cell_generic;      // [n_cells]: 1 if a combo that is not clean touches the cell
    int32_t *cell_ncombo;       // [n_cells]: row segments of column-served combos in the cell
    int32_t planes;             // segments a combo may have and stay column-served
    int32_t *seg_cell;          // [planes][N*D*W]: cell of segment s of the combo, or -1
    int32_t *seg_range;         // [planes][N*D*W]: its rows h_lo | h_hi << 16
    int32_t *counters;          // 6: most segments of a column-served combo, 7: kept points of such
                                // combos; 4 and 5, k_cell_class's, are cleared here for it
};

// One thread per combo walks its H rows and splits the kept ones into
// segments: maximal runs of consecutive kept rows in one cell. A combo with
// at most `planes` segments is served by the column items, one segment per
// pass (a level camera gives every combo one segment: a clean combo);
// otherwise its cells are generic. The rows are loaded kWalkRows at a time
// before they are walked (rows past H read row H - 1 and count as dropped),
// so one round trip serves kWalkRows rows.
constexpr int kWalkRows = 16;

__device__ __forceinline__ void walk_rows(const ComboArgs &a, int64_t base, int32_t h0,
                                          int32_t (&cc)[kWalkRows]) {
#pragma unroll
    for (int u = 0; u < kWalkRows; ++u)
        cc[u] = a.cell_of_point[base + int64_t(min(h0 + u, a.H - 1)) * a.W];
}

__device__ __forceinline__ void combo_walk_one(const ComboArgs &a, int32_t X, int64_t n_combo,
                                               int32_t &max_seg, int32_t &served_pts) {
    const int32_t w = X % a.W, nd = X / a.W;
    const int64_t base = int64_t(nd) * a.H * a.W + w;
    int32_t cell[kMaxSeg], lo[kMaxSeg], hi[kMaxSeg];
    int32_t n_seg = 0, cur = -1, first = -1, last = -1, kept = 0;
    for (int32_t h0 = 0; h0 < a.H; h0 += kWalkRows) {
        int32_t cc[kWalkRows];
        walk_rows(a, base, h0, cc);
#pragma unroll
        for (int u = 0; u < kWalkRows; ++u) {
            const int32_t h = h0 + u;
            const int32_t c = h < a.H ? cc[u] : -1;
            if (c < 0) {
                cur = -1;
            } else {
                ++kept;
                if (first < 0) first = h;
                last = h;
                if (c != cur) {
                    if (n_seg < a.planes) {
                        cell[n_seg] = c;
                        lo[n_seg] = h;
                    }
                    ++n_seg;
                    cur = c;
                }
                if (n_seg <= a.planes) hi[n_seg - 1] = h + 1;
            }
        }
    }
    for (int s = 0; s < a.planes; ++s) a.seg_cell[int64_t(s) * n_combo + X] = -1;
    if (n_seg == 0) {
        a.combo_cell[X] = -1;
        return;
    }
    if (a.allow_clean && n_seg <= a.planes) {
        for (int s = 0; s < n_seg; ++s) {
            a.seg_cell[int64_t(s) * n_combo + X] = cell[s];
            a.seg_range[int64_t(s) * n_combo + X] = lo[s] | (hi[s] << 16);
            atomicAdd(&a.cell_ncombo[cell[s]], 1);
        }
        max_seg = max(max_seg, n_seg);
        served_pts += kept;
        a.combo_cell[X] = n_seg == 1 ? cell[0] : -2;
    } else {
        a.combo_cell[X] = -2;
        for (int32_t h0 = first; h0 <= last; h0 += kWalkRows) {
            int32_t cc[kWalkRows];
            walk_rows(a, base, h0, cc);
#pragma unroll
            for (int u = 0; u < kWalkRows; ++u)
                if (h0 + u <= last && cc[u] >= 0) atomicOr(&a.cell_generic[cc[u]], 1);
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_combo_walk(ComboArgs a) {
    __shared__ int32_t s_m[kWaves], s_p[kWaves];
    if (blockIdx.x == 0) clear_pair(a.counters, 4, int(threadIdx.x));
    const int64_t n_combo = int64_t(a.N) * a.D * a.W;
    int32_t max_seg = 0, served_pts = 0;
    for (int64_t x = int64_t(blockIdx.x) * kBlock + threadIdx.x; x < n_combo;
         x += int64_t(gridDim.x) * kBlock)
        combo_walk_one(a, int32_t(x), n_combo, max_seg, served_pts);
    max_seg = block_reduce<true>(max_seg, s_m);
    served_pts = block_reduce<false>(served_pts, s_p);
    if (threadIdx.x == 0) {
        if (max_seg > 0) atomicMax(shard(a.counters, 6), max_seg);
        if (served_pts > 0) atomicAdd(shard(a.counters, 7), served_pts);
    }
}

// Per cell: generic flag, empty flag (both arrays n_cells + 1 long, the
// last entry 0); counter 4 += column-served cells, counter 5 += heavy
// generic cells.
__global__ __launch_bounds__(kBlock) void k_cell_class(ComboArgs a, const int32_t *cell_start,
                                                       int32_t n_cells, int32_t *generic_flag,
                                                       int32_t *empty_flag) {
    __shared__ int32_t s_s[kWaves], s_h[kWaves];
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        generic_flag[n_cells] = 0;   // the flags are scanned over n_cells + 1 entries
        empty_flag[n_cells] = 0;
    }
    int32_t n_served = 0, n_heavy = 0;
    for (int32_t c = blockIdx.x * kBlock + threadIdx.x; c < n_cells; c += gridDim.x * kBlock) {
        const int32_t cnt = cell_start[c + 1] - cell_start[c];
        const bool served = cnt > 0 && a.cell_generic[c] == 0;
        generic_flag[c] = (cnt > 0 && !served) ? 1 : 0;
        empty_flag[c] = cnt == 0 ? 1 : 0;
        n_served += served ? 1 : 0;
        n_heavy += (cnt > kGenHeavy && !served) ? 1 : 0;
    }
    n_served = block_reduce<false>(n_served, s_s);
    n_heavy = block_reduce<false>(n_heavy, s_h);
    if (threadIdx.x == 0) {
        if (n_served > 0) atomicAdd(shard(a.counters, 4), n_served);
        if (n_heavy > 0) atomicAdd(shard(a.counters, 5), n_heavy);
    }
}

// Column table entries, one plane per segment index, and a flag on each
// segment of a cell fed by several segments (one more entry, 0, ends the
// flags).
__global__ __launch_bounds__(kBlock) void k_combo_table(ComboArgs a, int2 *table, int32_t *multi_flag) {
    const int64_t t = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    const int64_t n = int64_t(a.planes) * a.N * a.D * a.W;
    if (t == 0) multi_flag[n] = 0;   // scanned over n + 1 entries
    if (t >= n) return;
    const int32_t c = a.seg_cell[t];
    int2 e = make_int2(-1, 0);
    bool multi = false;
    if (c >= 0 && a.cell_generic[c] == 0) {
        multi = a.cell_ncombo[c] > 1;
        e = make_int2(c, a.seg_range[t] | int32_t(multi ? kComboMulti : 0u));
    }
    table[t] = e;
    multi_flag[t] = multi ? 1 : 0;
}

// Every entry of the column table empty ({-1, 0}): planes that the final
// partition does not use hold no stale entries.
__global__ __launch_bounds__(kBlock) void k_clear_table(int2 *table, int64_t n) {
    const int64_t t = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (t < n) table[t] = make_int2(-1, 0);
}

// Planes in use (counter 2): one past the highest plane of the column table
// that holds an entry.
__global__ __launch_bounds__(kBlock) void k_planes_used(const int2 *table, int64_t n,
                                                        int32_t n_combo, int32_t *counters) {
    __shared__ int32_t s_m[kWaves];
    int32_t most = 0;
    for (int64_t t = int64_t(blockIdx.x) * kBlock + threadIdx.x; t < n; t += int64_t(gridDim.x) * kBlock)
        if (table[t].x >= 0) most = max(most, int32_t(t / n_combo) + 1);
    most = block_reduce<true>(most, s_m);
    if (threadIdx.x == 0 && most > 0) atomicMax(shard(counters, 2), most);
}

// Backward lists (internal.h). One thread per (camera, depth bin, row block,
// column block) looks at its kBwdRows x kBwdCols cells; threads with
// adjacent column blocks read adjacent pieces. A column's kept rows are cut
// where the cell changes (dropped rows in between do not cut), and slot s of
// the depth bin takes piece s of every column; slot 0 also writes the zeros
// of the dropped rows. Every depth bin has a slot.
struct BwdListArgs {
    const int32_t *cell_of_point;
    int32_t N, D, H, W, quads_w, blocks_h;
    FastDiv div_q, div_b, div_d;
    int32_t total;              // N * D * blocks_h * quads_w threads
    int32_t n_lists;
    int32_t *counts;            // [N][quads_w][blocks_h][D] slots of the bins, then their places in the list
    int32_t *offs;              // [n_lists + 1] slots of the lists, then their first slots
    int4 *cells, *masks;
    int32_t *bins;
};

struct BwdTile {
    int32_t c[kBwdCols][kBwdRows];   // cells, -1 for a dropped point or one past the map
    int32_t rows;                    // rows of the block inside the map
    int32_t cols;                    // columns inside the map
    int32_t d;
    int64_t at;                      // entry of counts
};

__device__ __forceinline__ void load_bwd_tile(const BwdListArgs &a, int32_t x, BwdTile &t) {
    const uint32_t xq = fdiv(uint32_t(x), a.div_q), xb = fdiv(xq, a.div_b), n = fdiv(xb, a.div_d);
    const int32_t cq = x - int32_t(xq) * a.quads_w, rb = int32_t(xq) - int32_t(xb) * a.blocks_h;
    t.d = int32_t(xb) - int32_t(n) * a.D;
    t.at = ((int64_t(n) * a.quads_w + cq) * a.blocks_h + rb) * a.D + t.d;
    const int32_t h0 = rb * kBwdRows, w0 = cq * kBwdCols;
    t.rows = min(kBwdRows, a.H - h0);
    t.cols = min(kBwdCols, a.W - w0);
    const int32_t *src = a.cell_of_point + (int64_t(xb) * a.H + h0) * a.W + w0;
    // rows and columns past the map read clamped, so that all loads are
    // issued together; a row's piece is one 16-byte load where the rows keep
    // the alignment (cell_of_point begins at a multiple of 256 bytes)
    if (a.W % kBwdCols == 0) {
#pragma unroll
        for (int r = 0; r < kBwdRows; ++r) {
            const int4 v = *reinterpret_cast<const int4 *>(src + int64_t(min(r, t.rows - 1)) * a.W);
            t.c[0][r] = r < t.rows ? v.x : -1;
            t.c[1][r] = r < t.rows ? v.y : -1;
            t.c[2][r] = r < t.rows ? v.z : -1;
            t.c[3][r] = r < t.rows ? v.w : -1;
        }
    } else {
#pragma unroll
        for (int r = 0; r < kBwdRows; ++r)
#pragma unroll
            for (int i = 0; i < kBwdCols; ++i) {
                const int32_t v = src[int64_t(min(r, t.rows - 1)) * a.W + min(i, t.cols - 1)];
                t.c[i][r] = r < t.rows && i < t.cols ? v : -1;
            }
    }
}

__global__ __launch_bounds__(kBlock) void k_bwd_counts(BwdListArgs a) {
    const int32_t x = blockIdx.x * kBlock + threadIdx.x;
    if (x >= a.total) return;
    BwdTile t;
    load_bwd_tile(a, x, t);
    int32_t most = 1;
#pragma unroll
    for (int i = 0; i < kBwdCols; ++i) {
        int32_t last = -1, n = 0;
#pragma unroll
        for (int r = 0; r < kBwdRows; ++r) {
            const bool cut = t.c[i][r] >= 0 && t.c[i][r] != last;
            n += cut ? 1 : 0;
            last = t.c[i][r] >= 0 ? t.c[i][r] : last;
        }
        most = max(most, n);
    }
    a.counts[t.at] = most;
}

// One workgroup per list: the bins' places in it. A bin's slots stay within
// kBwdStep slots of the list (the step of the kernel that runs it), which puts
// empty slots before a bin that would cross. That order is serial, but what a
// run of bins adds depends on where it starts only through the place within a
// step: the bins are cut into kBwdStep runs, thread (c, o) walks run c from
// offset o of a step, the runs' true starts follow from their 16 advances
// each, and the thread that started where run c starts writes its places.
constexpr int kPlaceBins = 1024;   // bins in LDS at a time

__device__ __forceinline__ int32_t bwd_place(int32_t at, int32_t n) {
    return (at & (kBwdStep - 1)) + n > kBwdStep ? (at | (kBwdStep - 1)) + 1 : at;
}

__global__ __launch_bounds__(kBlock) void k_bwd_places(BwdListArgs a) {
    static_assert(kBlock == kBwdStep * kBwdStep, "a thread per run and offset");
    __shared__ int32_t s_n[kPlaceBins];
    __shared__ int32_t s_add[kBwdStep][kBwdStep];
    int32_t *counts = a.counts + int64_t(blockIdx.x) * a.D;
    const int c = threadIdx.x / kBwdStep, o = threadIdx.x % kBwdStep;
    int32_t at = 0;
    for (int32_t d0 = 0; d0 < a.D; d0 += kPlaceBins) {
        const int32_t nd = min(kPlaceBins, a.D - d0), run = (nd + kBwdStep - 1) / kBwdStep;
        for (int32_t d = threadIdx.x; d < nd; d += kBlock) s_n[d] = counts[d0 + d];
        __syncthreads();
        const int32_t lo = min(nd, c * run), hi = min(nd, lo + run);
        int32_t end = o;
        for (int32_t d = lo; d < hi; ++d) end = bwd_place(end, s_n[d]) + s_n[d];
        s_add[c][o] = end - o;
        __syncthreads();
        int32_t start = at;
        for (int u = 0; u < kBwdStep; ++u) {
            if (u == c) start = at;
            at += s_add[u][at & (kBwdStep - 1)];
        }
        if ((start & (kBwdStep - 1)) == o)
            for (int32_t d = lo; d < hi; ++d) {
                start = bwd_place(start, s_n[d]);
                counts[d0 + d] = start;
                start += s_n[d];
            }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        a.offs[blockIdx.x] = at;
        if (blockIdx.x == 0) a.offs[a.n_lists] = 0;   // scanned over n_lists + 1 entries
    }
}

__global__ __launch_bounds__(kBlock) void k_bwd_lists(BwdListArgs a) {
    const int32_t x = blockIdx.x * kBlock + threadIdx.x;
    if (x >= a.total) return;
    BwdTile t;
    load_bwd_tile(a, x, t);
    const int32_t list = int32_t(t.at / a.D);
    const int32_t base = a.offs[list], first = base + a.counts[t.at];
    const int32_t end = t.d + 1 < a.D ? base + a.counts[t.at + 1] : a.offs[list + 1];
    const uint32_t in_rows = (1u << t.rows) - 1u;
    // slots past the bin's last piece fill the step: no cells, no rows
    for (int32_t s = 0; s < end - first; ++s) {
        int32_t cell[kBwdCols];
        uint32_t keep[kBwdCols], write[kBwdCols];
#pragma unroll
        for (int i = 0; i < kBwdCols; ++i) {
            int32_t last = -1, piece = -1;
            uint32_t kept = 0u, any = 0u;
            cell[i] = -1;
#pragma unroll
            for (int r = 0; r < kBwdRows; ++r) {
                const int32_t c = t.c[i][r];
                piece += c >= 0 && c != last ? 1 : 0;
                last = c >= 0 ? c : last;
                const bool mine = c >= 0 && piece == s;
                cell[i] = mine ? c : cell[i];
                kept |= mine ? 1u << r : 0u;
                any |= c >= 0 ? 1u << r : 0u;
            }
            keep[i] = kept;
            write[i] = i < t.cols ? kept | (s == 0 ? in_rows & ~any : 0u) : 0u;
        }
        a.cells[first + s] = make_int4(cell[0], cell[1], cell[2], cell[3]);
        a.masks[first + s] = make_int4(int32_t(keep[0] | keep[1] << 16), int32_t(keep[2] | keep[3] << 16),
                                       int32_t(write[0] | write[1] << 16), int32_t(write[2] | write[3] << 16));
        a.bins[first + s] = t.d;
    }
}

// Not enough empty rows to hold the partial sums: cells fed by several
// combos become generic.
__global__ __launch_bounds__(kBlock) void k_demote_multi(ComboArgs a, int32_t n_cells) {
    const int32_t c = blockIdx.x * kBlock + threadIdx.x;
    clear_pair(a.counters, 4, c);
    if (c < n_cells && a.cell_generic[c] == 0 && a.cell_ncombo[c] > 1) a.cell_generic[c] = 1;
}

__global__ __launch_bounds__(kBlock) void k_empty_list(const int32_t *empty_pos, int32_t n_cells,
                                                       int32_t *empty_cells) {
    const int32_t c = blockIdx.x * kBlock + threadIdx.x;
    if (c < n_cells && empty_pos[c + 1] != empty_pos[c]) empty_cells[empty_pos[c]] = c;
}

// Segments of multi-segment cells as (cell, segment) pairs in segment order.
__global__ __launch_bounds__(kBlock) void k_multi_compact(const int32_t *seg_cell,
                                                          const int32_t *multi_pos, int32_t n_seg,
                                                          uint32_t *key, int32_t *val) {
    const int32_t X = blockIdx.x * kBlock + threadIdx.x;
    if (X >= n_seg || multi_pos[X + 1] == multi_pos[X]) return;
    key[multi_pos[X]] = uint32_t(seg_cell[X]);
    val[multi_pos[X]] = X;
}

// After the stable sort by cell, position i is the partial-sum slot of combo
// val[i]: a cell's slots are contiguous and in combo order. Slot i is kept in
// the BEV row of empty cell i (the output has a row for every cell, and the
// rows of empty cells are free until they are zeroed), so the table entry of
// the combo names that row; cell heads are flagged.
__global__ __launch_bounds__(kBlock) void k_multi_slots(const uint32_t *key, const int32_t *val,
                                                        int32_t n, const int32_t *empty_cells,
                                                        int2 *table, int32_t *head_flag) {
    const int32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i == 0) head_flag[n] = 0;   // scanned over n + 1 entries
    if (i >= n) return;
    table[val[i]].x = empty_cells[i];
    head_flag[i] = (i == 0 || key[i] != key[i - 1]) ? 1 : 0;
}

__global__ __launch_bounds__(kBlock) void k_multi_cells(const uint32_t *key, const int32_t *head_scan,
                                                        int32_t n, int32_t *multi_begin,
                                                        int32_t *multi_cell) {
    const int32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i > n) return;
    if (i == n) {
        multi_begin[head_scan[n]] = n;
        return;
    }
    if (head_scan[i + 1] != head_scan[i]) {
        multi_begin[head_scan[i]] = i;
        multi_cell[head_scan[i]] = int32_t(key[i]);
    }
}

// The borrowed rows of the first kCombineInline slots of each multi-combo
// cell, next to each other, so that the combine kernel finds them with one
// access; -1 past the cell's last slot. One thread per entry, launched for the
// most cells there can be (their number stays on the device until the end).
__global__ __launch_bounds__(kBlock) void k_multi_rows(const int32_t *multi_begin, const int32_t *n_multi,
                                                       const int32_t *empty_cells,
                                                       int32_t *multi_rows) {
    const int64_t x = int64_t(blockIdx.x) * kBlock + threadIdx.x;
    if (x >= int64_t(*n_multi) * kCombineInline) return;
    const int32_t k = int32_t(x / kCombineInline), u = int32_t(x % kCombineInline);
    const int32_t s = multi_begin[k] + u;
    multi_rows[x] = s < multi_begin[k + 1] ? empty_cells[s] : -1;
}

// Generic cells keyed for a descending sort by point count.
__global__ __launch_bounds__(kBlock) void k_compact_generic(const int32_t *cell_start, int32_t n_cells,
                                                            const int32_t *generic_pos,
                                                            int32_t max_per_cell, uint32_t *gen_key,
                                                            int32_t *gen_cell) {
    const int32_t c = blockIdx.x * kBlock + threadIdx.x;
    if (c >= n_cells || generic_pos[c + 1] == generic_pos[c]) return;
    gen_key[generic_pos[c]] = uint32_t(max_per_cell - (cell_start[c + 1] - cell_start[c]));
    gen_cell[generic_pos[c]] = c;
}

// 1 where a kept point of a generic cell starts a run: its previous depth
// bin (same pixel) is not a point of the same cell (one more entry, 0, ends
// the flags).
__global__ __launch_bounds__(kBlock) void k_run_flags(const int32_t *sorted_point, int32_t n_kept,
                                                      const int32_t *cell_of_point,
                                                      const int32_t *generic_pos, int32_t HW,
                                                      FastDiv div_hw, FastDiv div_d, int32_t D,
                                                      int32_t *flag) {
    const int32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i == 0) flag[n_kept] = 0;   // scanned over n_kept + 1 entries
    if (i >= n_kept) return;
    const int32_t p = sorted_point[i];
    const int32_t c = cell_of_point[p];
    const bool generic = generic_pos[c + 1] != generic_pos[c];
    const uint32_t q = fdiv(uint32_t(p), div_hw);
    const int32_t d = int32_t(q) - int32_t(fdiv(q, div_d)) * D;
    flag[i] = (generic && (d == 0 || cell_of_point[p - HW] != c)) ? 1 : 0;
}

// Runs per listed generic cell (one more entry, 0, for the scan), and each
// cell's list position.
__global__ __launch_bounds__(kBlock) void k_generic_counts(const int32_t *gen_cell, int32_t n_gen,
                                                           const int32_t *cell_start,
                                                           const int32_t *run_scan,
                                                           int32_t *runs_of, int32_t *pos_of_cell) {
    const int32_t k = blockIdx.x * kBlock + threadIdx.x;
    if (k == 0) runs_of[n_gen] = 0;   // scanned over n_gen + 1 entries
    if (k >= n_gen) return;
    const int32_t c = gen_cell[k];
    runs_of[k] = run_scan[cell_start[c + 1]] - run_scan[cell_start[c]];
    pos_of_cell[c] = k;
}

__global__ __launch_bounds__(kBlock) void k_generic_hdr(const int32_t *gen_cell, int32_t n_gen,
                                                        const int32_t *cell_start,
                                                        const int32_t *run_begin, int4 *hdr) {
    const int32_t k = blockIdx.x * kBlock + threadIdx.x;
    if (k >= n_gen) return;
    const int32_t c = gen_cell[k];
    hdr[k] = make_int4(c, run_begin[k], run_begin[k + 1] - run_begin[k],
                       cell_start[c + 1] - cell_start[c]);
}

// One thread per run start: the run's record, at its place in list order.
__global__ __launch_bounds__(kBlock) void k_generic_runs(const int32_t *sorted_point, int32_t n_kept,
                                                         const int32_t *cell_of_point,
                                                         const int32_t *cell_start,
                                                         const int32_t *run_scan,
                                                         const int32_t *pos_of_cell,
                                                         const int32_t *run_begin, int32_t HW,
                                                         int32_t D, FastDiv div_hw, FastDiv div_d,
                                                         int4 *runs) {
    const int32_t i = blockIdx.x * kBlock + threadIdx.x;
    if (i >= n_kept || run_scan[i + 1] == run_scan[i]) return;
    const int32_t p = sorted_point[i];
    const int32_t c = cell_of_point[p];
    const uint32_t q = fdiv(uint32_t(p), div_hw);           // n * D + d
    const int32_t n = int32_t(fdiv(q, div_d));
    const int32_t d = int32_t(q) - n * D;
    const int32_t pixel = n * HW + (p - int32_t(q) * HW);
    int32_t len = 1;
    while (d + len < D && cell_of_point[p + len * HW] == c) ++len;
    const int32_t r = run_begin[pos_of_cell[c]] + (run_scan[i] - run_scan[cell_start[c]]);
    runs[r] = make_int4(p, pixel, len, 0);
}

int blocks_for(int64_t n) { return int((n + kBlock - 1) / kBlock); }
// Grid of a kernel that reduces into shared counters (at least one workgroup).
int reduce_blocks(int64_t n) { return std::max(1, std::min(blocks_for(n), kReduceBlocks)); }

template <typename T>
int dev_alloc(T **p, size_t count, const char *what) {
    *p = nullptr;
    const size_t bytes = (count ? count : 1) * sizeof(T);
    hipError_t e = hipMalloc(reinterpret_cast<void **>(p), bytes);
    if (e == hipErrorOutOfMemory || e == hipErrorMemoryAllocation) {
        int dev = -1;
        size_t cap = 0;
        char *kept = hipGetDevice(&dev) == hipSuccess ? bevpool_workspace_out(dev, &cap) : nullptr;
        if (kept) {
            (void)hipGetLastError();
            (void)hipFree(kept);
            e = hipMalloc(reinterpret_cast<void **>(p), bytes);
        }
    }
    if (e == hipErrorOutOfMemory || e == hipErrorMemoryAllocation) {
        (void)hipGetLastError();
        return bevpool_fail(BEVPOOL_ERR_OOM, "out of device memory allocating %s (%zu bytes)", what,
                            count * sizeof(T));
    }
    if (e != hipSuccess) return bevpool_hip_fail(e, what);
    return BEVPOOL_OK;
}

// One device allocation carved into arrays: each piece is rounded to 256
// bytes, and the total is reserved beforehand, so that a plan build makes one
// allocation for its temporaries (from upper bounds that the geometry fixes)
// and two or three for the plan, instead of one per array (each hipMalloc
// and hipFree costs about 10 us of host time).
struct Arena {
    char *base = nullptr;
    size_t cap = 0, used = 0;
    static size_t piece(size_t bytes) { return ((bytes ? bytes : 1) + 255) & ~size_t(255); }
    template <typename T>
    int take(T **p, size_t count, const char *what) {
        const size_t b = piece(count * sizeof(T));
        if (used + b > cap) {
            *p = nullptr;
            return bevpool_fail(BEVPOOL_ERR_HIP, "plan arrays: %s does not fit the reserved %zu bytes", what, cap);
        }
        *p = reinterpret_cast<T *>(base + used);
        used += b;
        return BEVPOOL_OK;
    }
};

// Exclusive scans in place of up to kScanJobs arrays, in one pair of launches
// (or one launch where a single short array is left to one workgroup).
struct Scan {
    int32_t *data;
    int64_t n;
    int32_t *total;   // receives the sum; may be null
};
constexpr int64_t kScanSums = int64_t(kScanJobs) * kScanBlocks;   // scratch ints

template <int N>
void device_scan(const Scan (&scans)[N], int32_t *sums, hipStream_t stream) {
    static_assert(N <= kScanJobs, "jobs of one launch");
    if (N == 1 && scans[0].n <= int64_t(kScanOneBlockChunks) * kScanChunk) {
        hipLaunchKernelGGL(k_scan, dim3(1), dim3(kScanBlock), 0, stream, scans[0].data, scans[0].n, scans[0].total);
        return;
    }
    ScanArgs a = {};
    int blocks = 1;
    for (int i = 0; i < N; ++i) {
        const int64_t chunks = std::max<int64_t>(1, (scans[i].n + kScanChunk - 1) / kScanChunk);
        ScanJob &b = a.job[i];
        b.data = scans[i].data;
        b.n = scans[i].n;
        b.total = scans[i].total;
        b.sums = sums + i * kScanBlocks;
        b.chunks = int32_t((chunks + kScanBlocks - 1) / kScanBlocks);
        b.blocks = int32_t((chunks + b.chunks - 1) / b.chunks);
        blocks = std::max(blocks, b.blocks);
    }
    hipLaunchKernelGGL(k_scan_sums, dim3(blocks, N), dim3(kScanBlock), 0, stream, a);
    hipLaunchKernelGGL(k_scan_apply, dim3(blocks, N), dim3(kScanBlock), 0, stream, a);
}

void device_scan(int32_t *data, int64_t n, int32_t *total, int32_t *sums, hipStream_t stream) {
    const Scan one[1] = {{data, n, total}};
    device_scan(one, sums, stream);
}

// Stable LSD radix sort of n (key, value) pairs on the keys' low `bits` bits
// (radix_passes passes of radix_digit_bits bits), ping-ponging between keys /
// kalt and vals / valt; keys and vals are left pointing at the buffers that
// hold the result. With cells, the first pass takes the points' cells as keys
// and their positions as values, and writes to keys and valt.
int radix_sort(const int32_t *cells, int32_t n_cells, uint32_t *&keys, uint32_t *kalt, int32_t *&vals, int32_t *valt,
               int32_t n, int bits, int32_t *hist, int32_t *sums, hipStream_t stream) {
    if (n <= 0) return BEVPOOL_OK;
    const int tiles = int((int64_t(n) + kSortTile - 1) / kSortTile);
    const int passes = radix_passes(bits), dbits = radix_digit_bits(bits);
    uint32_t *kin = keys, *kout = kalt;
    int32_t *vin = vals, *vout = valt;
    if (cells) std::swap(kin, kout);
    for (int pass = 0; pass < passes; ++pass) {
        const int shift = dbits * pass;
        const bool first = cells && pass == 0;
        const uint32_t *src = first ? reinterpret_cast<const uint32_t *>(cells) : kin;
        if (first) hipLaunchKernelGGL(k_radix_hist<true>, dim3(tiles), dim3(kBlock), 0, stream, src, n, n_cells, shift, dbits, hist);
        else hipLaunchKernelGGL(k_radix_hist<false>, dim3(tiles), dim3(kBlock), 0, stream, src, n, n_cells, shift, dbits, hist);
        device_scan(hist, int64_t(tiles) << dbits, nullptr, sums, stream);
        if (first) hipLaunchKernelGGL(k_radix_scatter<true>, dim3(tiles), dim3(kBlock), 0, stream, src, vin, n, n_cells, shift, dbits, hist, kout, vout);
        else hipLaunchKernelGGL(k_radix_scatter<false>, dim3(tiles), dim3(kBlock), 0, stream, src, vin, n, n_cells, shift, dbits, hist, kout, vout);
        BEVPOOL_HIP(hipGetLastError());
        std::swap(kin, kout);
        std::swap(vin, vout);
    }
    keys = kin;
    vals = vin;
    return BEVPOOL_OK;
}

// Projection arguments common to both entry points.
void project_args(ProjectArgs &pa, const bevpool_geometry &g, int32_t nz, int32_t *cell_of_point) {
    pa.g = g;
    pa.n_blocks = (g.n_depth + kProjectBins - 1) / kProjectBins;
    pa.div_w = make_fastdiv(uint32_t(g.feat_w));
    pa.div_h = make_fastdiv(uint32_t(g.feat_h));
    pa.div_b = make_fastdiv(uint32_t(pa.n_blocks));
    pa.n_threads = g.n_cams * pa.n_blocks * g.feat_h * g.feat_w;   // at most the points
    pa.nz = nz;
    pa.cell_of_point = cell_of_point;
}

}  // namespace
}  // namespace bevpool

using namespace bevpool;

int bevpool_build_plan(const double *intrinsics, const double *extrinsics,
                       const int32_t *host_cells, const bevpool_geometry &g, int32_t nz,
                       hipStream_t stream, bevpool_plan_s *plan) {
    const int64_t np64 = int64_t(g.n_cams) * g.n_depth * g.feat_h * g.feat_w;
    const int32_t np = int32_t(np64);
    const int32_t n_cells = g.nx * g.ny * nz;
    const int32_t N = g.n_cams, D = g.n_depth, H = g.feat_h, W = g.feat_w;
    const int32_t HW = H * W;
    const int64_t n_combo = int64_t(N) * D * W;
    // column-table planes: segment indices a combo may use (a segment has a
    // row of its own, so never more than H)
    const int32_t planes = H < kMaxSeg ? H : kMaxSeg;
    const int64_t n_seg = int64_t(planes) * n_combo;   // table entries reserved
    int64_t n_seg_act = n_seg;                          // entries of the planes in use
    const int32_t quads_w = (W + kBwdCols - 1) / kBwdCols, blocks_h = (H + kBwdRows - 1) / kBwdRows;
    const int32_t n_lists = N * quads_w * blocks_h;     // backward lists, n_bwd (list, depth bin) pairs:
    const int32_t n_bwd = n_lists * D;                  // at most one for each point
    // No lists (the backward then takes the per-row kernel) where a launch of one
    // workgroup for each list, or two, would not fit a grid's 2^32 threads, or
    // where the slots might not fit int32: a bin of the most pieces, one a row, with
    // all but one of them as empty slots before it.
    const bool lists = n_lists < (1 << 23) &&
                       int64_t(n_bwd) * (2 * std::min(H, kBwdRows) - 1) <= int64_t(INT32_MAX);
    plan->n_points = np64;
    plan->n_cells = n_cells;
    plan->nz = nz;

    // the plan's arrays whose sizes the geometry fixes
    int rc;
    Arena fixed;
    fixed.cap = 2 * Arena::piece(size_t(np) * 4) + Arena::piece((size_t(n_cells) + 1) * 4) +
                Arena::piece(size_t(n_seg) * 8) + Arena::piece(size_t(n_combo) * 4) +
                Arena::piece((size_t(n_lists) + 1) * 4);
    if ((rc = dev_alloc(&fixed.base, fixed.cap, "the plan"))) return rc;
    plan->mem_fixed = fixed.base;
    if ((rc = fixed.take(&plan->cell_of_point, size_t(np), "cell_of_point"))) return rc;
    if ((rc = fixed.take(&plan->sorted_point, size_t(np), "sorted_point"))) return rc;
    if ((rc = fixed.take(&plan->cell_start, size_t(n_cells) + 1, "cell_start"))) return rc;
    if ((rc = fixed.take(&plan->column_table, size_t(n_seg), "column_table"))) return rc;
    if ((rc = fixed.take(&plan->combo_cells, size_t(n_combo), "combo cells"))) return rc;
    if ((rc = fixed.take(&plan->bwd_offs, size_t(n_lists) + 1, "backward lists"))) return rc;

    // temporaries, carved from one arena that is given back on every exit path below
    const int64_t sort_cap = np64 > n_cells ? np64 : int64_t(n_cells);
    const int sort_tiles_cap = int((sort_cap + kSortTile - 1) / kSortTile);
    Arena arena;
    double *d_calib = nullptr;
    uint32_t *keys_a = nullptr, *keys_b = nullptr;
    int32_t *vals_a = nullptr, *vals_b = nullptr, *hist = nullptr, *small = nullptr;
    int32_t *scan_sums = nullptr;
    int32_t *flag_a = nullptr, *flag_b = nullptr;
    int32_t *combo_cell = nullptr, *combo_flag = nullptr;
    int32_t *cell_generic = nullptr, *cell_ncombo = nullptr, *head_scan = nullptr;
    int32_t *run_scan = nullptr, *run_begin = nullptr, *pos_of_cell = nullptr;

    auto bits_for = [](int64_t max_key) {
        int b = 1;
        while ((int64_t(1) << b) <= max_key) ++b;
        return b;
    };
    auto fill = [&](int32_t *p, int64_t n, int32_t v) {
        if (n > 0) hipLaunchKernelGGL(k_fill, dim3(blocks_for(n)), dim3(kBlock), 0, stream, p, n, v);
    };
    // the counters, read back and joined over their shards (maxima: 1, 2, 6;
    // the others are sums, or kept in one shard only); waits for the stream
    int32_t h[kCounters];
    auto read_counters = [&]() -> int {
        int32_t all[kShards * kCounters];
        BEVPOOL_HIP(hipMemcpyAsync(all, small, sizeof(all), hipMemcpyDeviceToHost, stream));
        BEVPOOL_HIP(hipStreamSynchronize(stream));
        for (int i = 0; i < kCounters; ++i) {
            h[i] = all[i];
            for (int u = 1; u < kShards; ++u) {
                const int32_t v = all[u * kCounters + i];
                h[i] = (i == 1 || i == 2 || i == 6) ? std::max(h[i], v) : h[i] + v;
            }
        }
        return BEVPOOL_OK;
    };

    auto run = [&]() -> int {
        int rc2;
        {
            // upper bounds of every temporary taken below: the partial slots
            // (n_part) are at most the combos, the kept points at most the
            // points, the generic cells at most the cells. The runtime keeps
            // about 64 MB of freed memory to hand out again and unmaps what is
            // beyond (270 us a piece), which a plan closed before the next one is
            // built should stay below: 53 MB of block and plan for 2 M points.
            const size_t i4 = sizeof(int32_t);
            const size_t sort_b = Arena::piece(size_t(sort_cap) * i4);
            const size_t cells1_b = Arena::piece((size_t(n_cells) + 1) * i4);
            const size_t combo1_b = Arena::piece((size_t(n_seg) + 1) * i4);
            arena.cap = Arena::piece(size_t(g.n_cams) * 16 * sizeof(double)) +
                        Arena::piece((size_t(sort_cap) + 1) * i4) + 2 * sort_b +   // keys_a, keys_b, vals_b
                        Arena::piece(size_t(std::max<int64_t>(n_seg, n_cells)) * i4) +   // vals_a
                        Arena::piece(size_t(sort_tiles_cap) * kRadixBins * i4) +
                        Arena::piece(size_t(kShards) * kCounters * i4) + Arena::piece(size_t(kScanSums) * i4) +
                        5 * cells1_b +                 // flag_a, flag_b, cell_generic, cell_ncombo, run_begin
                        Arena::piece(size_t(n_cells) * i4) +          // pos_of_cell
                        2 * combo1_b +                 // combo_flag, head_scan
                        2 * Arena::piece(size_t(n_seg) * i4) +        // seg_cell, seg_range
                        Arena::piece(size_t(n_bwd) * i4);             // bwd_counts
            const size_t need = arena.cap;
            arena.base = bevpool_workspace_out(plan->device, &arena.cap);
            if (!arena.base || arena.cap < need) {
                (void)hipFree(arena.base);
                arena.cap = need;
                if ((rc2 = dev_alloc(&arena.base, need, "plan temporaries"))) return rc2;
            }
        }
        const bool cal_in_args = g.n_cams <= kArgCams;
        if (!host_cells && !cal_in_args &&
            (rc2 = arena.take(&d_calib, size_t(g.n_cams) * 16, "calibration")))
            return rc2;
        // (vals_a serves the sorts of the slots and of the gathered cells only)
        if ((rc2 = arena.take(&keys_a, size_t(sort_cap) + 1, "sort keys"))) return rc2;
        if ((rc2 = arena.take(&keys_b, size_t(sort_cap), "sort keys"))) return rc2;
        if ((rc2 = arena.take(&vals_a, size_t(std::max<int64_t>(n_seg, n_cells)), "sort values"))) return rc2;
        if ((rc2 = arena.take(&vals_b, size_t(sort_cap), "sort values"))) return rc2;
        if ((rc2 = arena.take(&hist, size_t(sort_tiles_cap) * kRadixBins, "radix histogram"))) return rc2;
        // kShards shards of counters: [0..1] cell stats, [2] planes in use, [3]
        // multi-combo cells, [4..5] class counters, [6] most segments of a
        // combo, [7] their kept points, [8] generic cells, [9] empty cells,
        // [10] kept points, [11] segments of multi-combo cells, [12] backward
        // slots, [13] gather runs
        if ((rc2 = arena.take(&small, size_t(kShards) * kCounters, "plan counters"))) return rc2;
        if ((rc2 = arena.take(&scan_sums, size_t(kScanSums), "scan chunk sums"))) return rc2;
        if ((rc2 = arena.take(&flag_a, size_t(n_cells) + 1, "flags"))) return rc2;
        if ((rc2 = arena.take(&flag_b, size_t(n_cells) + 1, "flags"))) return rc2;

        fill(small, kShards * kCounters, 0);
        if (host_cells) {
            // a stored association: the cell map as exported, checked by the caller
            BEVPOOL_HIP(hipMemcpyAsync(plan->cell_of_point, host_cells, sizeof(int32_t) * size_t(np),
                                       hipMemcpyHostToDevice, stream));
        } else {
            ProjectArgs pa;
            if (cal_in_args) {
                // up to kArgCams cameras: no host-to-device copy
                pa.intr = pa.extr = nullptr;
                memcpy(pa.cal, intrinsics, sizeof(double) * 4 * g.n_cams);
                memcpy(pa.cal + 4 * g.n_cams, extrinsics, sizeof(double) * 12 * g.n_cams);
            } else {
                BEVPOOL_HIP(hipMemcpyAsync(d_calib, intrinsics, sizeof(double) * 4 * g.n_cams,
                                           hipMemcpyHostToDevice, stream));
                BEVPOOL_HIP(hipMemcpyAsync(d_calib + 4 * g.n_cams, extrinsics,
                                           sizeof(double) * 12 * g.n_cams, hipMemcpyHostToDevice,
                                           stream));
                pa.intr = d_calib;
                pa.extr = d_calib + 4 * g.n_cams;
            }

            // Sec. III-B, precomputation: cell of every point, then the points
            // sorted by (cell, id) and the interval table.
            project_args(pa, g, nz, plan->cell_of_point);
            hipLaunchKernelGGL(k_project, dim3(blocks_for(pa.n_threads)), dim3(kBlock), 0, stream, pa);
        }
        BEVPOOL_HIP(hipGetLastError());
        // the passes alternate between two value buffers and end in
        // sorted_point: the first writes to it when their number is odd
        const int cell_bits = bits_for(n_cells);
        const bool odd_passes = radix_passes(cell_bits) % 2 == 1;
        uint32_t *skeys = keys_a;
        int32_t *sids = odd_passes ? vals_b : plan->sorted_point;
        if ((rc2 = radix_sort(plan->cell_of_point, n_cells, skeys, keys_b, sids,
                              odd_passes ? plan->sorted_point : vals_b, np, cell_bits, hist, scan_sums, stream)))
            return rc2;
        hipLaunchKernelGGL(k_cell_start, dim3(blocks_for(int64_t(np) / kStartItems + 1)), dim3(kBlock), 0,
                           stream, skeys, np, n_cells, plan->cell_start);
        // per-cell counters of the combo walk, cleared by k_cell_stats
        if ((rc2 = arena.take(&cell_generic, size_t(n_cells), "cell classes"))) return rc2;
        if ((rc2 = arena.take(&cell_ncombo, size_t(n_cells), "cell combos"))) return rc2;
        hipLaunchKernelGGL(k_cell_stats, dim3(reduce_blocks(n_cells)), dim3(kBlock), 0, stream,
                           plan->cell_start, n_cells, small, cell_generic, cell_ncombo);
        BEVPOOL_HIP(hipGetLastError());

        // combos, cell classes and the column table
        combo_cell = plan->combo_cells;
        if ((rc2 = arena.take(&combo_flag, size_t(n_seg) + 1, "segment flags"))) return rc2;
        int32_t *seg_cell = nullptr, *seg_range = nullptr;
        if ((rc2 = arena.take(&seg_cell, size_t(n_seg), "segment cells"))) return rc2;
        if ((rc2 = arena.take(&seg_range, size_t(n_seg), "segment rows"))) return rc2;
        ComboArgs ca;
        ca.cell_of_point = plan->cell_of_point;
        ca.N = N;
        ca.D = D;
        ca.H = H;
        ca.W = W;
        ca.allow_clean = H < kMaxFeatH ? 1 : 0;
        ca.combo_cell = combo_cell;
        ca.cell_generic = cell_generic;
        ca.cell_ncombo = cell_ncombo;
        ca.planes = planes;
        ca.seg_cell = seg_cell;
        ca.seg_range = seg_range;
        ca.counters = small;
        // the backward lists' slots are counted here; their number comes back
        // with the counts of the first classification (0 without lists)
        BwdListArgs bl;
        bl.cell_of_point = plan->cell_of_point;
        bl.N = N;
        bl.D = D;
        bl.H = H;
        bl.W = W;
        bl.quads_w = quads_w;
        bl.blocks_h = blocks_h;
        bl.div_q = make_fastdiv(uint32_t(quads_w));
        bl.div_b = make_fastdiv(uint32_t(blocks_h));
        bl.div_d = make_fastdiv(uint32_t(D));
        bl.total = n_bwd;
        bl.n_lists = n_lists;
        if ((rc2 = arena.take(&bl.counts, size_t(n_bwd), "backward slots"))) return rc2;
        bl.offs = plan->bwd_offs;
        if (lists) {
            hipLaunchKernelGGL(k_bwd_counts, dim3(blocks_for(n_bwd)), dim3(kBlock), 0, stream, bl);
            hipLaunchKernelGGL(k_bwd_places, dim3(n_lists), dim3(kBlock), 0, stream, bl);
            device_scan(bl.offs, int64_t(n_lists) + 1, small + 12, scan_sums, stream);
        }
        // (k_combo_table writes every entry of every plane: no clearing first)
        hipLaunchKernelGGL(k_combo_walk, dim3(reduce_blocks(n_combo)), dim3(kBlock), 0, stream, ca);
        int32_t stats[4], counters[2], n_gen = 0, n_empty = 0, kept = 0, n_part = 0;
        // (the class counters 4 and 5 are cleared by k_combo_walk or
        // k_demote_multi, which run before each classification)
        auto classify = [&]() -> int {
            hipLaunchKernelGGL(k_cell_class, dim3(reduce_blocks(n_cells)), dim3(kBlock), 0, stream, ca,
                               plan->cell_start, n_cells, flag_a, flag_b);
            hipLaunchKernelGGL(k_combo_table, dim3(blocks_for(n_seg_act)), dim3(kBlock), 0, stream,
                               ca, plan->column_table, combo_flag);
            const Scan scans[3] = {{flag_a, int64_t(n_cells) + 1, small + 8},      // generic cells
                                   {flag_b, int64_t(n_cells) + 1, small + 9},      // empty cells
                                   {combo_flag, n_seg_act + 1, small + 11}};       // segments of multi cells
            device_scan(scans, scan_sums, stream);
            BEVPOOL_HIP(hipGetLastError());
            int rc3;
            if ((rc3 = read_counters())) return rc3;
            stats[0] = h[0];
            stats[1] = h[1];
            stats[2] = h[6];       // most segments of a column-served combo
            stats[3] = h[7];       // kept points of column-served combos
            counters[0] = h[4];
            counters[1] = h[5];
            n_gen = h[8];          // generic cells
            n_empty = h[9];        // empty cells
            kept = h[10];          // kept points (k_cell_stats)
            n_part = h[11];        // combos of multi-combo cells (partial slots)
            plan->n_bwd_slots = h[12];
            return BEVPOOL_OK;
        };
        if ((rc2 = classify())) return rc2;
        if (ca.planes > 1 && int64_t(stats[3]) * 2 < int64_t(kept)) {
            // segments serve under half of the kept points (a strongly tilted
            // rig): the extra passes would cost more than they save, so the
            // partition is rebuilt with whole combos only
            ca.planes = 1;
            n_seg_act = n_combo;
            hipLaunchKernelGGL(k_clear_table, dim3(blocks_for(n_seg)), dim3(kBlock), 0, stream,
                               plan->column_table, n_seg);
            fill(cell_generic, n_cells, 0);
            fill(cell_ncombo, n_cells, 0);
            hipLaunchKernelGGL(k_clear_pair, dim3(1), dim3(2 * kShards), 0, stream, small, 6);
            hipLaunchKernelGGL(k_combo_walk, dim3(reduce_blocks(n_combo)), dim3(kBlock), 0, stream, ca);
            if ((rc2 = classify())) return rc2;
        }
        if (n_part > n_empty) {
            hipLaunchKernelGGL(k_demote_multi, dim3(blocks_for(n_cells)), dim3(kBlock), 0, stream, ca,
                               n_cells);
            if ((rc2 = classify())) return rc2;
        }
        plan->n_nonempty = stats[0];
        plan->max_per_cell = stats[1];
        plan->n_kept = kept;
        plan->n_column = counters[0];
        plan->n_generic_heavy = counters[1];
        plan->n_generic = n_gen;
        plan->n_empty = n_empty;
        plan->n_partials = n_part;
        // planes in use, from the final table (cells demoted to generic leave
        // their segments' planes empty)
        hipLaunchKernelGGL(k_planes_used, dim3(reduce_blocks(n_seg_act)), dim3(kBlock), 0, stream,
                           plan->column_table, n_seg_act, int32_t(n_combo), small);

        BEVPOOL_HIP(hipGetLastError());

        // cells without points, ascending
        // (with them the other arrays that the counts size; a multi-combo cell
        // has two slots or more)
        const int32_t multi_cap = n_part / 2;
        Arena counted;
        counted.cap = Arena::piece(size_t(n_empty) * 4) + Arena::piece((size_t(multi_cap) + 1) * 4) +
                      Arena::piece(size_t(multi_cap) * 4) + Arena::piece(size_t(multi_cap) * kCombineInline * 4) +
                      Arena::piece(size_t(n_gen) * 16) + 2 * Arena::piece(size_t(plan->n_bwd_slots) * 16) +
                      Arena::piece(size_t(plan->n_bwd_slots) * 4);
        if ((rc2 = dev_alloc(&counted.base, counted.cap, "the plan"))) return rc2;
        plan->mem_counted = counted.base;
        if ((rc2 = counted.take(&plan->empty_cells, size_t(n_empty), "empty_cells"))) return rc2;
        if ((rc2 = counted.take(&plan->multi_begin, size_t(multi_cap) + 1, "multi_begin"))) return rc2;
        if ((rc2 = counted.take(&plan->multi_cell, size_t(multi_cap), "multi_cell"))) return rc2;
        if ((rc2 = counted.take(&plan->multi_rows, size_t(multi_cap) * kCombineInline, "multi_rows"))) return rc2;
        if ((rc2 = counted.take(&plan->generic_hdr, size_t(n_gen), "generic_hdr"))) return rc2;
        if ((rc2 = counted.take(&plan->bwd_cells, size_t(plan->n_bwd_slots), "backward lists"))) return rc2;
        if ((rc2 = counted.take(&plan->bwd_masks, size_t(plan->n_bwd_slots), "backward lists"))) return rc2;
        if ((rc2 = counted.take(&plan->bwd_bins, size_t(plan->n_bwd_slots), "backward lists"))) return rc2;
        bl.cells = plan->bwd_cells;
        bl.masks = plan->bwd_masks;
        bl.bins = plan->bwd_bins;
        if (lists) hipLaunchKernelGGL(k_bwd_lists, dim3(blocks_for(n_bwd)), dim3(kBlock), 0, stream, bl);
        hipLaunchKernelGGL(k_empty_list, dim3(blocks_for(n_cells)), dim3(kBlock), 0, stream, flag_b,
                           n_cells, plan->empty_cells);

        // partial-sum slots of the multi-combo cells, kept in the first
        // n_part empty rows
        if ((rc2 = arena.take(&head_scan, size_t(n_part) + 1, "multi heads"))) return rc2;
        uint32_t *mkeys = keys_a;
        int32_t *mvals = vals_a;
        if (n_part > 0) {
            hipLaunchKernelGGL(k_multi_compact, dim3(blocks_for(n_seg_act)), dim3(kBlock), 0, stream,
                               seg_cell, combo_flag, int32_t(n_seg_act), keys_a, vals_a);
            if ((rc2 = radix_sort(nullptr, 0, mkeys, keys_b, mvals, vals_b, n_part, cell_bits, hist, scan_sums, stream)))
                return rc2;
            hipLaunchKernelGGL(k_multi_slots, dim3(blocks_for(n_part)), dim3(kBlock), 0, stream,
                               mkeys, mvals, n_part, plan->empty_cells, plan->column_table,
                               head_scan);
            // the number of multi-combo cells lands in counter 3
            device_scan(head_scan, int64_t(n_part) + 1, small + 3, scan_sums, stream);
        } else {
            fill(head_scan, 1, 0);
        }
        BEVPOOL_HIP(hipGetLastError());
        hipLaunchKernelGGL(k_multi_cells, dim3(blocks_for(int64_t(n_part) + 1)), dim3(kBlock), 0,
                           stream, mkeys, head_scan, n_part, plan->multi_begin, plan->multi_cell);
        if (multi_cap > 0)
            hipLaunchKernelGGL(k_multi_rows, dim3(blocks_for(int64_t(multi_cap) * kCombineInline)),
                               dim3(kBlock), 0, stream, plan->multi_begin, small + 3,
                               plan->empty_cells, plan->multi_rows);
        BEVPOOL_HIP(hipGetLastError());
        // (counter 3 is 0 without slots: no scan has written it)
        auto read_rest = [&]() -> int {
            int rc3;
            if ((rc3 = read_counters())) return rc3;
            plan->n_multi = h[3];
            plan->n_planes = h[2] > 0 ? h[2] : 1;
            plan->n_runs = h[13];
            return BEVPOOL_OK;
        };

        // generic cells by descending point count
        if (n_gen == 0) {
            // every cell with points is column-served (a level rig): no runs
            // (generic_runs stays null: a resource of no bytes)
            return read_rest();
        }
        uint32_t *gen_key = keys_a;   // the sort buffers are free again after k_multi_cells
        int32_t *gen_cell = vals_a;
        hipLaunchKernelGGL(k_compact_generic, dim3(blocks_for(n_cells)), dim3(kBlock), 0, stream,
                           plan->cell_start, n_cells, flag_a, plan->max_per_cell, gen_key, gen_cell);
        BEVPOOL_HIP(hipGetLastError());
        if ((rc2 = radix_sort(nullptr, 0, gen_key, keys_b, gen_cell, vals_b, n_gen, bits_for(plan->max_per_cell), hist,
                              scan_sums, stream)))
            return rc2;

        // runs of the generic cells, in list order (their flags in the keys'
        // place: the sort has left the cells in vals_a or vals_b)
        run_scan = reinterpret_cast<int32_t *>(keys_a);
        if ((rc2 = arena.take(&run_begin, size_t(n_gen) + 1, "run offsets"))) return rc2;
        if ((rc2 = arena.take(&pos_of_cell, size_t(n_cells), "cell positions"))) return rc2;
        const FastDiv div_hw = make_fastdiv(uint32_t(HW)), div_d = make_fastdiv(uint32_t(D));
        if (kept > 0)
            hipLaunchKernelGGL(k_run_flags, dim3(blocks_for(kept)), dim3(kBlock), 0, stream,
                               plan->sorted_point, kept, plan->cell_of_point, flag_a, HW, div_hw,
                               div_d, D, run_scan);
        device_scan(run_scan, int64_t(kept) + 1, nullptr, scan_sums, stream);
        if (n_gen > 0)
            hipLaunchKernelGGL(k_generic_counts, dim3(blocks_for(n_gen)), dim3(kBlock), 0, stream,
                               gen_cell, n_gen, plan->cell_start, run_scan, run_begin, pos_of_cell);
        device_scan(run_begin, int64_t(n_gen) + 1, small + 13, scan_sums, stream);
        if (n_gen > 0)
            hipLaunchKernelGGL(k_generic_hdr, dim3(blocks_for(n_gen)), dim3(kBlock), 0, stream,
                               gen_cell, n_gen, plan->cell_start, run_begin, plan->generic_hdr);
        BEVPOOL_HIP(hipGetLastError());
        if ((rc2 = read_rest())) return rc2;
        if ((rc2 = dev_alloc(&plan->generic_runs, size_t(plan->n_runs), "generic_runs"))) return rc2;
        if (kept > 0)
            hipLaunchKernelGGL(k_generic_runs, dim3(blocks_for(kept)), dim3(kBlock), 0, stream,
                               plan->sorted_point, kept, plan->cell_of_point, plan->cell_start,
                               run_scan, pos_of_cell, run_begin, HW, D, div_hw, div_d,
                               plan->generic_runs);
        BEVPOOL_HIP(hipGetLastError());
        BEVPOOL_HIP(hipStreamSynchronize(stream));
        return BEVPOOL_OK;
    };
    rc = run();
    if (rc != BEVPOOL_OK) (void)hipStreamSynchronize(stream);
    bevpool_workspace_in(plan->device, arena.base, arena.cap);
    return rc;
}

// ---------------------------------------------------------------- association without allocation
//
// bevpool_associate_noalloc: the association of the "Precomputation"
// paragraph (every point's cell, the points sorted by cell, the interval
// table) into caller buffers, for callers that cannot allocate. Its
// temporaries (the calibration, the radix sort's key arrays and second value
// array, histograms, scan sums) live in one file-scope device
// array of fixed size, which each device holds while the library is loaded.
// Host code never uses the array's name as an address: the device address
// comes from hipGetSymbolAddress, once per device, with that device current.
namespace bevpool {
namespace {

constexpr size_t scratch_piece(size_t b) { return (b + 255) & ~size_t(255); }
constexpr int64_t kAssocTiles = (kAssocMaxPoints + kSortTile - 1) / kSortTile;
constexpr int64_t kAssocSums = (kAssocTiles * kRadixBins + kScanChunk - 1) / kScanChunk;
static_assert(kAssocSums <= kScanBlocks, "one chunk a workgroup");
constexpr size_t kOffCalib = 0;
constexpr size_t kOffKeysA = kOffCalib + scratch_piece(size_t(kAssocMaxCams) * 16 * sizeof(double));
constexpr size_t kOffKeysB = kOffKeysA + scratch_piece(size_t(kAssocMaxPoints) * 4);
constexpr size_t kOffValsB = kOffKeysB + scratch_piece(size_t(kAssocMaxPoints) * 4);
constexpr size_t kOffHist = kOffValsB + scratch_piece(size_t(kAssocMaxPoints) * 4);
constexpr size_t kOffSums = kOffHist + scratch_piece(size_t(kAssocTiles) * kRadixBins * 4);
constexpr size_t kAssocScratchBytes = kOffSums + scratch_piece(size_t(kAssocSums) * 4);
static_assert(kAssocScratchBytes == kAssocScratchTotal, "scratch size stated in internal.h");

static __device__ __align__(256) char noalloc_scratch[kAssocScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
char *g_scratch_ptr[kMaxDevices] = {};

// Device address of the current device's scratch (looked up on first use).
int scratch_of_device(int dev, char **out) {
    if (dev < 0 || dev >= kMaxDevices)
        return bevpool_fail(BEVPOOL_ERR_INVALID_ARG, "device %d is beyond the %d supported", dev,
                            kMaxDevices);
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        BEVPOOL_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(noalloc_scratch)));
        if (!p) return bevpool_fail(BEVPOOL_ERR_HIP, "no device address for the scratch array");
        g_scratch_ptr[dev] = static_cast<char *>(p);
    }
    *out = g_scratch_ptr[dev];
    return BEVPOOL_OK;
}

// The calibration travels in the kernel arguments, so the call reads the
// caller's host arrays before it returns and copies nothing from host memory.
struct CalibArgs {
    double v[kAssocMaxCams * 16];   // [N][4] intrinsics, then [N][12] extrinsics
    int32_t n;                      // values used
};
__global__ void k_store_calib(CalibArgs a, double *dst) {
    for (int i = threadIdx.x; i < a.n; i += blockDim.x) dst[i] = a.v[i];
}

}  // namespace
}  // namespace bevpool

int bevpool_associate_into(const double *intrinsics, const double *extrinsics,
                           const bevpool_geometry &g, int32_t *cell_of_point,
                           int32_t *sorted_point, int32_t *cell_start, hipStream_t stream) {
    using namespace bevpool;
    const int64_t np64 = int64_t(g.n_cams) * g.n_depth * g.feat_h * g.feat_w;
    if (np64 > kAssocMaxPoints || g.n_cams > kAssocMaxCams)
        return bevpool_fail(BEVPOOL_ERR_INVALID_ARG,
                            "%lld points on %d cameras exceed the no-allocation maximum of %lld points "
                            "on %d cameras", (long long)np64, g.n_cams, (long long)kAssocMaxPoints,
                            kAssocMaxCams);
    int dev = -1;
    BEVPOOL_HIP(hipGetDevice(&dev));
    char *base = nullptr;
    int rc = scratch_of_device(dev, &base);
    if (rc != BEVPOOL_OK) return rc;
    double *calib = reinterpret_cast<double *>(base + kOffCalib);
    uint32_t *keys_a = reinterpret_cast<uint32_t *>(base + kOffKeysA);
    uint32_t *keys_b = reinterpret_cast<uint32_t *>(base + kOffKeysB);
    int32_t *vals_b = reinterpret_cast<int32_t *>(base + kOffValsB);
    int32_t *hist = reinterpret_cast<int32_t *>(base + kOffHist);
    int32_t *sums = reinterpret_cast<int32_t *>(base + kOffSums);
    const int32_t np = int32_t(np64), n_cells = g.nx * g.ny;

    CalibArgs ca;
    ca.n = 16 * g.n_cams;
    for (int i = 0; i < 4 * g.n_cams; ++i) ca.v[i] = intrinsics[i];
    for (int i = 0; i < 12 * g.n_cams; ++i) ca.v[4 * g.n_cams + i] = extrinsics[i];
    hipLaunchKernelGGL(k_store_calib, dim3(1), dim3(kBlock), 0, stream, ca, calib);

    ProjectArgs pa;
    pa.intr = calib;
    pa.extr = calib + 4 * g.n_cams;
    project_args(pa, g, 1, cell_of_point);
    hipLaunchKernelGGL(k_project, dim3(blocks_for(pa.n_threads)), dim3(kBlock), 0, stream, pa);
    BEVPOOL_HIP(hipGetLastError());
    // stable LSD radix sort of (cell, point id) on the cell's bits; the passes
    // end in sorted_point
    int bits = 1;
    while ((int64_t(1) << bits) <= int64_t(n_cells)) ++bits;
    const bool odd_passes = radix_passes(bits) % 2 == 1;
    uint32_t *skeys = keys_a;
    int32_t *sids = odd_passes ? vals_b : sorted_point;
    rc = radix_sort(cell_of_point, n_cells, skeys, keys_b, sids, odd_passes ? sorted_point : vals_b, np, bits, hist,
                    sums, stream);
    if (rc != BEVPOOL_OK) return rc;
    hipLaunchKernelGGL(k_cell_start, dim3(blocks_for(int64_t(np) / kStartItems + 1)), dim3(kBlock), 0, stream, skeys,
                       np, n_cells, cell_start);
    BEVPOOL_HIP(hipGetLastError());
    return BEVPOOL_OK;
}
