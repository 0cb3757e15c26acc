// Gradients of the per-frame BEV pooling (BEVFusion, arXiv 2205.13542,
// Sec. III-B: the pooling is one layer of a model trained end to end). The
// pooling is bilinear in (P, F); for G = d loss / d out:
//   dP[b][p]      = F[b][pixel(p)] . G[b][cell(p)]   for a kept point p, else 0
//   dF[b][pixel]  = sum over the kept points p of the pixel of P[b][p] G[b][cell(p)]
//
// k_backward_mma (feature and gradient rows of whole, aligned 4-element quads)
// runs both on the matrix cores (v_mfma_f32_16x16x4f32, fp32 in and out). The
// plan lists for 4 adjacent columns and 16 rows of one camera, in depth order,
// slots of one cell for each column with a mask of the rows whose points lie in
// that cell: one slot for a depth bin of a level camera, several where a tilted
// camera's rows cross cells. A workgroup takes all 4 columns of a list, or 2
// (four_columns below). For one column and the gradient rows G[s] of its slots'
// cells, with M the masks,
//   dF[h][c] = sum_s M[s][h] P[d(s)][h] G[s][c]
//   dP[d(s)][h] = sum_c G[s][c] F[h][c]   where M[s][h] is set
// The workgroup's four waves take consecutive parts of the list, 16 slots per
// step. The second product takes the channels as its K dimension in the order
// 16t + 4q + e (t the tile, q the lane quarter, e the element), so that F and G
// arrive as 16-byte quads; the first takes the slots as K and reads the step's
// gradient rows back transposed from the wave's own LDS copy. P and dP of the
// columns move as one piece where the map's width is a multiple of theirs. A
// bin's slots lie in one step, so the step's dP rows are whole and are stored
// once. The waves' dF sums are added in LDS in wave order. Both forms add in the
// same order: their results are the same bits.
//
// What bounds it: gathered rows and P and dP, whose lanes each touch a line of
// their own, through L1 and L2; the matrix cores alone take 4.4 of the 24 us of 6
// cameras x 118 bins x 32 x 88, C = 80, level, fp32, in cache. There the loads in
// flight count: two columns at three waves per SIMD take 22.8 us, four at two
// 24.4; cameras tilted by 1 degree 31 and 36 us, by 5 degrees 49 and 61 us (the
// kernel below: 56 us in the last two). 128 channels in one
// launch read P once (236 bins x 64 x 176: 322 us in two launches of 80 and 48
// channels, 165 us in one), with a dP product in two sums: one of 128 products
// rounds worse, 2.0e-7 against 1.5e-7 from exact. Four columns of 128 channels
// spill 19 of the 256 registers at two waves per SIMD (two columns none, 173 us
// there). Tried and no faster: 8 waves
// per workgroup; three waves per SIMD with four columns, by spilling; the next
// two columns' rows in flight; two columns' products interleaved.
//
// k_backward (other rows, and where by_rows says so): pixel-stationary work on
// the vector ALUs. A workgroup owns kBCols pixel columns x kBRows rows of one
// camera, and its kBWaves waves take consecutive parts of the depth bins. A
// group of 16 lanes owns one column; lane j holds channels j, j + 16, ... of the
// slice of the kBRows feature rows, read once, and the kBRows rows' dF sums. For
// each depth bin the group reads one gradient row when the combo (camera, depth
// bin, column) is clean, or one per kept row otherwise.
// dF gets P x G; dP gets the dot product F . G, reduced across the 16 lanes
// by a transpose-reduce (8 shuffles for the 8 rows' sums). A wave parks the
// dP values of a chunk of depth bins in LDS and writes them after the chunk
// (vector loads and stores share one in-order counter, so a store inside the
// loop would hold up the waits for the next loads). The waves' dF sums are
// added in LDS in wave order and stored once.
//
// Nothing is accumulated with atomics, so repeated calls give bitwise equal
// results. Channel slices run as successive launches; slices after the first
// add their dot products to dP.
#include <stdint.h>

#include <algorithm>

#include "device.h"
#include "internal.h"

namespace bevpool {
namespace {

__device__ __forceinline__ bool finite(float v) { return fabsf(v) <= 3.402823466e+38f; }

// dF of one pixel over its own points, for a lane group: value k of lane j is channel
// c0 + 16k + j (past the slice: not to be used). The
// kernels below add 0 x G of cells that do not hold the row's point, which is
// not 0 for an infinity or a NaN: a row with a sum that is not finite is formed
// again by this, so that only pixels with a point in such a cell see it (mixed
// precision meets infinities when the loss scale is too large). 16 depth bins at
// a time, one in each lane, then their rows.
template <int DT, int NCH>
__device__ __forceinline__ Row<NCH> kept_row(Rsrc P, Rsrc G, const int32_t *cop, int n, int D, int H, int W, int C,
                                             int h, int w, bool in, int c0, int j) {
    constexpr int kRows = 4;                   // gradient rows in flight
    const int base = int(threadIdx.x) & 48;    // the group's first lane
    Row<NCH> v;
#pragma unroll
    for (int k = 0; k < NCH; ++k) v.v[k] = 0.f;
    for (int d0 = 0; d0 < D; d0 += 16) {
        const uint32_t pt = (uint32_t(n * D + d0 + j) * uint32_t(H) + uint32_t(h)) * uint32_t(W) + uint32_t(w);
        const int cell = in && d0 + j < D ? cop[pt] : -1;
        const float p = Elem<DT>::load(P, cell >= 0 ? pt * uint32_t(Elem<DT>::kBytes) : kOff);
        for (int u0 = 0; u0 < 16; u0 += kRows) {
            Row<NCH> g[kRows];
#pragma unroll
            for (int u = 0; u < kRows; ++u) {
                const int c = __shfl(cell, base | (u0 + u));
                load_row<BEVPOOL_F32, NCH, false>(g[u], G, c >= 0 ? (uint32_t(c) * uint32_t(C) + uint32_t(c0)) * 4u : kOff);
            }
#pragma unroll
            for (int u = 0; u < kRows; ++u) {
                const float pu = __shfl(p, base | (u0 + u));
#pragma unroll
                for (int k = 0; k < NCH; ++k) v.v[k] = __builtin_fmaf(pu, g[u].v[k], v.v[k]);
            }
        }
    }
    return v;
}

constexpr int kBRows = 8;                      // pixel rows per lane group
constexpr int kBCols = 4;                      // pixel columns per workgroup (lane groups of a wave)
constexpr int kBWaves = 4;                     // depth parts per workgroup
constexpr int kBBlock = kBWaves * kWaveSize;
constexpr int kBStages = 4;                    // depth bins in flight per wave
constexpr int kBChunk = 32;                    // combo cells held in registers per pass (2 per lane)

struct BwdArgs {
    const char *P, *F;
    const float *G;
    float *dP, *dF;
    const int32_t *cop, *combo_cells;
    int32_t N, D, H, W, HW, C, c0, cn;         // channel slice [c0, c0 + cn)
    uint32_t p_bytes, f_bytes, g_bytes, dp_bytes, df_bytes;   // per frame
    uint32_t cop_bytes, cc_bytes;
    int32_t items_w, items_h;                  // column blocks and row blocks per camera
    int32_t part;                              // depth bins per wave
    int32_t accumulate_dp, want_dp, want_df;
};

// One depth bin of a lane group: its combo's cell, each row's cell (lane j:
// row j & 7), each row's probability, and the clean combo's gradient row.
template <int NCH>
struct BStage {
    int cc, cell;
    float pv;
    Row<NCH> g;
};

// Sum of v[0..7] over the 16 lanes of a group, by halving rounds: after
// them lanes j and j ^ 8 hold the total of row j & 7.
__device__ __forceinline__ float transpose_reduce(const float (&v)[kBRows], int j) {
    float a[4], b[2];
    const bool h2 = (j & 4) != 0, h1 = (j & 2) != 0, h0 = (j & 1) != 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float keep = h2 ? v[4 + i] : v[i], send = h2 ? v[i] : v[4 + i];
        a[i] = keep + __shfl_xor(send, 4, 16);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const float keep = h1 ? a[2 + i] : a[i], send = h1 ? a[i] : a[2 + i];
        b[i] = keep + __shfl_xor(send, 2, 16);
    }
    const float keep = h0 ? b[1] : b[0], send = h0 ? b[0] : b[1];
    const float c = keep + __shfl_xor(send, 1, 16);
    return c + __shfl_xor(c, 8, 16);
}

// acc[r] += pv_r * g and dot[r] = f[r] . g for the kBRows rows, pv_r from
// lane r of the group. What a tail lane's last value holds lies past the slice:
// it stays out of the dot product (its feature is 0, but 0 x infinity is not).
template <int R, int NCH>
struct RowTerms {
    static __device__ __forceinline__ void run(float (&acc)[kBRows][NCH], float (&dot)[kBRows],
                                               const Row<NCH> (&f)[kBRows], const Row<NCH> &g,
                                               float pv) {
        const float p = row_bcast<R>(pv);
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < NCH; ++k) {
            acc[R][k] = __builtin_fmaf(p, g.v[k], acc[R][k]);
            s = __builtin_fmaf(f[R].v[k], g.v[k], s);
        }
        dot[R] = s;
        RowTerms<R + 1, NCH>::run(acc, dot, f, g, pv);
    }
};
template <int NCH>
struct RowTerms<kBRows, NCH> {
    static __device__ __forceinline__ void run(float (&)[kBRows][NCH], float (&)[kBRows],
                                               const Row<NCH> (&)[kBRows], const Row<NCH> &, float) {}
};

// The same for a combo that is not clean: row R reads the gradient row of
// its own cell (lane R's cell of the group), if it has one. The rows' loads
// are issued kBEach at a time before their terms, so that one round trip
// serves them (loading and using each row in turn made every row wait for
// all loads in flight).
constexpr int kBEach = 4;
template <int R0, int U, int NCH>
__device__ __forceinline__ void each_loads(Row<NCH> (&g)[kBEach], Rsrc G, uint32_t g_ch, int C, int cell) {
    if constexpr (U < kBEach) {
        const int c = row_bcast<R0 + U>(cell);
        const uint32_t addr = uint32_t(max(c, 0)) * uint32_t(C) * 4u + g_ch;
        load_row<BEVPOOL_F32, NCH, false>(g[U], G, c >= 0 ? addr : kOff);
        each_loads<R0, U + 1, NCH>(g, G, g_ch, C, cell);
    }
}
template <int R0, int U, int NCH>
__device__ __forceinline__ void each_terms(float (&acc)[kBRows][NCH], float (&dot)[kBRows],
                                           const Row<NCH> (&f)[kBRows], const Row<NCH> (&g)[kBEach],
                                           float pv, bool tail_ok) {
    if constexpr (U < kBEach) {
        constexpr int R = R0 + U;
        const float p = row_bcast<R>(pv);
        float s = 0.f;
#pragma unroll
        for (int k = 0; k < NCH; ++k) {
            acc[R][k] = __builtin_fmaf(p, g[U].v[k], acc[R][k]);
            const float x = __builtin_fmaf(f[R].v[k], g[U].v[k], s);
            s = k < NCH - 1 || tail_ok ? x : s;
        }
        dot[R] = s;
        each_terms<R0, U + 1, NCH>(acc, dot, f, g, pv, tail_ok);
    }
}
template <int R0, int NCH>
__device__ __forceinline__ void row_terms_each(float (&acc)[kBRows][NCH], float (&dot)[kBRows],
                                               const Row<NCH> (&f)[kBRows], Rsrc G, uint32_t g_ch,
                                               int C, int cell, float pv, bool tail_ok) {
    if constexpr (R0 < kBRows) {
        Row<NCH> g[kBEach];
        each_loads<R0, 0, NCH>(g, G, g_ch, C, cell);
        each_terms<R0, 0, NCH>(acc, dot, f, g, pv, tail_ok);
        row_terms_each<R0 + kBEach, NCH>(acc, dot, f, G, g_ch, C, cell, pv, tail_ok);
    }
}

template <int NCH>
constexpr int bwd_stride() { return kBRows * NCH * 16 + 16; }   // one lane group's dF sums in LDS

// (five values a lane: held to the 168 registers of three waves per SIMD)
template <int DT, int NCH>
__global__ __launch_bounds__(kBBlock) __attribute__((amdgpu_waves_per_eu(NCH == 5 ? 3 : 1)))
void k_backward(BwdArgs a) {
    __shared__ float s_df[(kBWaves - 1) * kBCols * bwd_stride<NCH>()];
    // dP of a chunk: [wave][depth bin of the chunk][row][column]
    __shared__ float s_dp[kBWaves * kBChunk * kBRows * kBCols];
    constexpr uint32_t ES = Elem<DT>::kBytes;
    const int b = blockIdx.y;
    // the row blocks of one column block share its gradient rows: placed on
    // one XCD, two at a time on one CU
    const int item = xcd_cu_remap<2>(blockIdx.x, gridDim.x);
    const int rb = item % a.items_h;
    const int t = item / a.items_h;
    const int cb = t % a.items_w, n = t / a.items_w;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int j = lane & 15, grp = lane >> 4;
    const int w = cb * kBCols + grp;
    const int h0 = rb * kBRows;
    const int jr = j & 7;                      // this lane's row for indices and probabilities
    const bool in_w = w < a.W;
    const bool row_ok = in_w && h0 + jr < a.H;
    const bool tail_ok = j + 16 * (NCH - 1) < a.cn;

    const Rsrc P = make_rsrc(a.P + int64_t(b) * a.p_bytes, a.p_bytes);
    const Rsrc F = make_rsrc(a.F + int64_t(b) * a.f_bytes, a.f_bytes);
    const Rsrc G = make_rsrc(reinterpret_cast<const char *>(a.G) + int64_t(b) * a.g_bytes, a.g_bytes);
    const Rsrc dP = make_rsrc(reinterpret_cast<const char *>(a.dP) + int64_t(b) * a.dp_bytes, a.dp_bytes);
    const Rsrc dF = make_rsrc(reinterpret_cast<const char *>(a.dF) + int64_t(b) * a.df_bytes, a.df_bytes);
    const Rsrc cop = make_rsrc(a.cop, a.cop_bytes);
    const Rsrc ccs = make_rsrc(a.combo_cells, a.cc_bytes);

    // the group's feature rows, once
    Row<NCH> f[kBRows];
    const uint32_t f_row = uint32_t(a.W) * uint32_t(a.C) * ES;
    const uint32_t f_col = in_w ? (uint32_t(n * a.HW + h0 * a.W + w) * uint32_t(a.C) + uint32_t(a.c0)) * ES : kOff;
#pragma unroll
    for (int r = 0; r < kBRows; ++r) {
        load_row<DT, NCH, false>(f[r], F, h0 + r < a.H ? f_col + uint32_t(r) * f_row : kOff);
        // the last value of a tail lane lies past the slice: it must not
        // enter the dot products
        if (!tail_ok) f[r].v[NCH - 1] = 0.f;
    }

    float acc[kBRows][NCH];
#pragma unroll
    for (int r = 0; r < kBRows; ++r)
#pragma unroll
        for (int k = 0; k < NCH; ++k) acc[r][k] = 0.f;

    const uint32_t g_ch = uint32_t(a.c0) * 4u;
    const uint32_t gC = uint32_t(a.C) * 4u;
    const int d_lo = min(a.D, wave * a.part), d_hi = min(a.D, d_lo + a.part);
    // point id of (n, d, h0 + jr, w) is pt0 + d * HW
    const uint32_t pt0 = uint32_t((n * a.D) * a.HW + (h0 + jr) * a.W + w);

    for (int dc = d_lo; dc < d_hi; dc += kBChunk) {
        // the combo cells of this chunk's depth bins: lane j holds bins dc + j and dc + 16 + j
        const int dn = min(kBChunk, d_hi - dc);
        const uint32_t cc_base = uint32_t((n * a.D + dc) * a.W + w) * 4u;
        const int cc_a = in_w && j < dn ? int(__builtin_amdgcn_raw_buffer_load_b32(ccs, int(cc_base + uint32_t(j * a.W) * 4u), 0, 0)) : -1;
        const int cc_b = in_w && 16 + j < dn ? int(__builtin_amdgcn_raw_buffer_load_b32(ccs, int(cc_base + uint32_t((16 + j) * a.W) * 4u), 0, 0)) : -1;
        auto load_stage = [&](BStage<NCH> &st, int i) {   // depth bin dc + i
            const bool ok = i < dn;
            const int cc_src = i < 16 ? cc_a : cc_b;
            st.cc = ok ? __shfl(cc_src, (lane & 48) | (i & 15), 64) : -1;
            const uint32_t p = pt0 + uint32_t(dc + i) * uint32_t(a.HW);
            st.cell = ok && row_ok ? int(__builtin_amdgcn_raw_buffer_load_b32(cop, int(p * 4u), 0, 0)) : -1;
            st.pv = Elem<DT>::load(P, ok && row_ok ? p * ES : kOff);
            load_row<BEVPOOL_F32, NCH, false>(st.g, G, st.cc >= 0 ? uint32_t(st.cc) * gC + g_ch : kOff);
        };
        BStage<NCH> st[kBStages];
#pragma unroll
        for (int u = 0; u < kBStages; ++u) {
            load_stage(st[u], u);
            __builtin_amdgcn_sched_barrier(0);
        }
        for (int i0 = 0; i0 < dn; i0 += kBStages) {
#pragma unroll
            for (int u = 0; u < kBStages; ++u) {
                const int i = i0 + u;
                // a dropped row adds nothing and gets dP = 0
                const bool kept = st[u].cell >= 0;
                const float pv = kept ? st[u].pv : 0.f;
                float dot[kBRows];
                if (!tail_ok) st[u].g.v[NCH - 1] = 0.f;
                if (st[u].cc >= 0) {
                    RowTerms<0, NCH>::run(acc, dot, f, st[u].g, pv);
                } else if (st[u].cc == -2) {
                    row_terms_each<0, NCH>(acc, dot, f, G, g_ch, a.C, st[u].cell, pv, tail_ok);
                } else {
#pragma unroll
                    for (int r = 0; r < kBRows; ++r) dot[r] = 0.f;
                }
                if (a.want_dp) {
                    const float s = transpose_reduce(dot, j);
                    if (j < kBRows && i < dn)
                        s_dp[((wave * kBChunk + i) * kBRows + j) * kBCols + grp] = kept ? s : 0.f;
                }
                load_stage(st[u], i + kBStages);
            }
        }
        if (a.want_dp) {
            // the chunk's dP, 4 columns (16 contiguous bytes) per 4 lanes:
            // value q of the wave is column q % 4, row q / 4 % 8, bin q / 32
            __builtin_amdgcn_wave_barrier();
            for (int q = lane; q < dn * kBRows * kBCols; q += kWaveSize) {
                const int qc = q % kBCols, qr = (q / kBCols) % kBRows, qi = q / (kBCols * kBRows);
                const int wq = cb * kBCols + qc, hq = h0 + qr;
                const uint32_t off = wq < a.W && hq < a.H
                    ? uint32_t(((n * a.D + dc + qi) * a.H + hq) * a.W + wq) * 4u : kOff;
                float v = s_dp[(wave * kBChunk + qi) * kBRows * kBCols + q % (kBRows * kBCols)];
                if (a.accumulate_dp) v += __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(dP, int(off), 0, 0));
                store_f32(dP, off, v);
            }
            __builtin_amdgcn_wave_barrier();
        }
    }

    if (!a.want_df) return;
    // waves 1.. park their sums in LDS; wave 0 adds them in wave order
    constexpr int BS = bwd_stride<NCH>();
    if (wave > 0) {
        float *slot = s_df + ((wave - 1) * kBCols + grp) * BS + j;
#pragma unroll
        for (int r = 0; r < kBRows; ++r)
#pragma unroll
            for (int k = 0; k < NCH; ++k) slot[(r * NCH + k) * 16] = acc[r][k];
    }
    __syncthreads();
    if (wave > 0) return;
    for (int v = 1; v < kBWaves; ++v) {
        const float *slot = s_df + ((v - 1) * kBCols + grp) * BS + j;
#pragma unroll
        for (int r = 0; r < kBRows; ++r)
#pragma unroll
            for (int k = 0; k < NCH; ++k) acc[r][k] += slot[(r * NCH + k) * 16];
    }
    const uint32_t df_col = in_w ? (uint32_t(n * a.HW + h0 * a.W + w) * uint32_t(a.C) + uint32_t(a.c0)) * 4u : kOff;
    const uint32_t df_row = uint32_t(a.W) * uint32_t(a.C) * 4u;
    float zero = 0.f;                          // NaN once a sum is not finite
#pragma unroll
    for (int r = 0; r < kBRows; ++r) {
        store_row<NCH, false>(dF, h0 + r < a.H ? df_col + uint32_t(r) * df_row : kOff, acc[r], tail_ok);
#pragma unroll
        for (int k = 0; k < NCH; ++k) zero = __builtin_fmaf(acc[r][k], 0.f, zero);
    }
    if (__ballot(zero != 0.f) == 0) return;
    uint64_t bad = 0u;                         // bit r * NCH + k: value k of row r
#pragma unroll
    for (int r = 0; r < kBRows; ++r)
#pragma unroll
        for (int k = 0; k < NCH; ++k)
            bad |= !finite(acc[r][k]) && in_w && h0 + r < a.H && (k < NCH - 1 || tail_ok) ? uint64_t(1) << (r * NCH + k) : 0u;
#pragma unroll 1
    for (int r = 0; r < kBRows; ++r) {
        const uint32_t mine = uint32_t(bad >> (r * NCH)) & ((1u << NCH) - 1u);
        if (__ballot(mine != 0u) == 0) continue;
        // (a group without one runs along)
        const Row<NCH> x = kept_row<DT, NCH>(P, G, a.cop, n, a.D, a.H, a.W, a.C, h0 + r, w, in_w && h0 + r < a.H, a.c0, j);
#pragma unroll
        for (int k = 0; k < NCH; ++k)
            store_f32(dF, mine >> k & 1u ? df_col + uint32_t(r) * df_row + uint32_t(j + 16 * k) * 4u : kOff, x.v[k]);
    }
}


// ---------------------------------------------------------------- matrix cores

constexpr int kMWaves = 4;                     // parts of a list per workgroup
constexpr int kMBlock = kMWaves * kWaveSize;
constexpr int kMRows = kBwdRows;               // pixel rows per workgroup (M of the instruction)
constexpr int kMChunk = kBwdStep;              // slots per step (N of the dP product)
constexpr int kMSlice = 128;                   // channels per launch, at most
static_assert(kBwdCols == 4 && kMRows == 16 && kMChunk == 16, "the shape of the slots and of the instruction");

typedef float f4v __attribute__((ext_vector_type(4)));

struct MmaArgs {
    const char *P, *F;
    const float *G;
    float *dP, *dF;
    const int32_t *cop;
    const int32_t *offs, *bins;                // the plan's backward lists
    const int4 *cells, *masks;
    int32_t D, H, W, C, c0, cn;                // channel slice [c0, c0 + cn), cn a multiple of 4
    uint32_t p_bytes, f_bytes, g_bytes, dp_bytes, df_bytes;
    int32_t quads_w, blocks_h;                 // column quads and row blocks per camera
    int32_t accumulate_dp, want_dp, want_df;
};

// LDS row stride (floats) of a step's gradient rows: an odd multiple of 16,
// so that the four rows one transposed read touches fall in distinct banks.
template <int T>
constexpr int mma_stride() { return 16 * (T | 1); }

// V consecutive elements as fp32.
template <int DT, int V>
__device__ __forceinline__ void load_piece(Rsrc r, uint32_t off, float *v) {
    if constexpr (V == 4) {
        Elem<DT>::load4(r, off, v);
    } else if constexpr (V == 2 && DT == BEVPOOL_F32) {
        const auto x = __builtin_amdgcn_raw_buffer_load_b64(r, int(off), 0, 0);
        v[0] = __uint_as_float(x[0]);
        v[1] = __uint_as_float(x[1]);
    } else if constexpr (V == 2) {
        const uint32_t x = __builtin_amdgcn_raw_buffer_load_b32(r, int(off), 0, 0);
        if constexpr (DT == BEVPOOL_BF16) {
            v[0] = __uint_as_float(x << 16);
            v[1] = __uint_as_float(x & 0xFFFF0000u);
        } else {
            v[0] = float(__builtin_bit_cast(_Float16, uint16_t(x & 0xFFFFu)));
            v[1] = float(__builtin_bit_cast(_Float16, uint16_t(x >> 16)));
        }
    } else {
        v[0] = Elem<DT>::load(r, off);
    }
}

// Slot k + j of a list in lane (q, j): the cells, row masks (two columns to a
// word: kept rows, rows whose dP it writes) and bin. Past the wave's last slot
// it holds that slot, which takes part in nothing once end_slot has run.
template <int COLS>
struct Slot {
    int c[COLS], keep[COLS / 2], write[COLS / 2];
    int d;
};

template <int COLS>
__device__ __forceinline__ void end_slot(Slot<COLS> &t, bool ok) {
#pragma unroll
    for (int i = 0; i < COLS; ++i) t.c[i] = ok ? t.c[i] : -1;
#pragma unroll
    for (int i = 0; i < COLS / 2; ++i) {
        t.keep[i] = ok ? t.keep[i] : 0;
        t.write[i] = ok ? t.write[i] : 0;
    }
}

template <int DT, int T, int COLS, int V>
__global__ __launch_bounds__(kMBlock) __attribute__((amdgpu_waves_per_eu(COLS == 2 && T <= 5 ? 3 : 2)))
void k_backward_mma(MmaArgs a) {
    static_assert(COLS % V == 0 && kBwdCols % COLS == 0, "whole pieces and parts of a list's columns");
    constexpr int S = mma_stride<T>();
    constexpr int kFq = 4 * T + 1;             // quads per feature row in LDS (odd: no bank conflicts)
    constexpr int kSum = T * 4 * kWaveSize;    // one wave's dF sums of a column
    // LDS words from one bin of a step's dP to the next: kMRows x COLS values,
    // and a quad so that bins start in different banks
    constexpr int kDpStride = kMRows * COLS + 4;
    constexpr int kGs = kMChunk * S > kMChunk * kDpStride ? kMChunk * S : kMChunk * kDpStride;
    constexpr uint32_t ES = Elem<DT>::kBytes;
    // feature rows and the waves' step buffers; for the sums at the end, one
    // or two columns of every wave
    constexpr int kLds = COLS * kMRows * kFq * 4 + kMWaves * kGs;
    constexpr int kSumCols = 2 * kMWaves * kSum <= kLds ? 2 : 1;
    static_assert(kSumCols * kMWaves * kSum <= kLds, "the columns' sums fit");
    __shared__ __attribute__((aligned(16))) float s_all[kLds];
    f4v *s_f = reinterpret_cast<f4v *>(s_all);
    float *s_g = s_all + COLS * kMRows * kFq * 4;
    const int b = blockIdx.y;
    // the row blocks of a list's columns share its gradient rows: two of them on
    // one CU; neighbouring columns share P lines: placed on one XCD
    const int item = xcd_cu_remap<2>(blockIdx.x, gridDim.x);
    const int rb = item % a.blocks_h;
    const int tt = item / a.blocks_h;
    constexpr int kParts = kBwdCols / COLS;    // workgroups of a list, by columns
    const int sub = tt % kParts, cq = tt / kParts % a.quads_w, n = tt / kParts / a.quads_w;
    const int list = tt / kParts * a.blocks_h + rb;
    const int w0 = cq * kBwdCols + sub * COLS, h0 = rb * kMRows;
    if (kParts > 1 && w0 >= a.W) return;       // a part past the map
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int q = lane >> 4, j = lane & 15;

    const Rsrc P = make_rsrc(a.P + int64_t(b) * a.p_bytes, a.p_bytes);
    const Rsrc F = make_rsrc(a.F + int64_t(b) * a.f_bytes, a.f_bytes);
    const Rsrc G = make_rsrc(reinterpret_cast<const char *>(a.G) + int64_t(b) * a.g_bytes, a.g_bytes);
    const Rsrc dP = make_rsrc(reinterpret_cast<const char *>(a.dP) + int64_t(b) * a.dp_bytes, a.dp_bytes);
    const Rsrc dF = make_rsrc(reinterpret_cast<const char *>(a.dF) + int64_t(b) * a.df_bytes, a.df_bytes);
    const uint32_t HW = uint32_t(a.H) * uint32_t(a.W);

    // this wave's slots of the list
    const int s0 = a.offs[list], s1 = a.offs[list + 1];
    const int part = ((s1 - s0 + kMWaves - 1) / kMWaves + kMChunk - 1) / kMChunk * kMChunk;
    const int lo = min(s1, s0 + wave * part), hi = min(s1, lo + part);
    // (clamped and masked later: no branch and no wait at the loads)
    auto load_slot = [&](Slot<COLS> &t, int k) {
        const int at = min(k + j, hi - 1);
        if constexpr (COLS == 4) {
            const int4 c = a.cells[at], m = a.masks[at];
            t.c[0] = c.x;
            t.c[1] = c.y;
            t.c[2] = c.z;
            t.c[3] = c.w;
            t.keep[0] = m.x;
            t.keep[1] = m.y;
            t.write[0] = m.z;
            t.write[1] = m.w;
        } else {
            const int2 c = reinterpret_cast<const int2 *>(a.cells)[int64_t(at) * 2 + sub];
            const int32_t *m = reinterpret_cast<const int32_t *>(a.masks) + int64_t(at) * 4 + sub;
            t.c[0] = c.x;
            t.c[1] = c.y;
            t.keep[0] = m[0];
            t.write[0] = m[2];
        }
        t.d = a.bins[at];
    };
    // the gradient rows of a column's 16 slots, slot j's row in the lanes
    // (., j) as quads in the channel order of the dP product
    f4v g[T];
    auto load_rows = [&](int cell) {
        const uint32_t row = uint32_t(max(cell, 0)) * uint32_t(a.C) + uint32_t(a.c0 + 4 * q);
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const bool ok = (cell >= 0) & (16 * t + 4 * q < a.cn);
            const auto v = __builtin_amdgcn_raw_buffer_load_b128(G, int(ok ? (row + uint32_t(16 * t)) * 4u : kOff), 0, 0);
            g[t] = f4v{__uint_as_float(v[0]), __uint_as_float(v[1]), __uint_as_float(v[2]), __uint_as_float(v[3])};
        }
    };
    // the feature rows of the workgroup's columns and rows go to LDS: quad
    // 4t + q of row (i, r) holds channels c0 + 16t + 4q .. + 3. All of a
    // thread's loads are issued before the first is waited for.
    constexpr int kQuads = COLS * kMRows * 4 * T;
    constexpr int kFill = (kQuads + kMBlock - 1) / (kMBlock);
    float fill[kFill][4];
#pragma unroll
    for (int u = 0; u < kFill; ++u) {
        const int x = threadIdx.x + u * kMBlock;
        const int qd = x % (4 * T), i = (x / (4 * T)) % COLS, r = x / (4 * T * COLS);
        const bool ok = (h0 + r < a.H) & (w0 + i < a.W) & (4 * qd < a.cn);
        const uint32_t addr = ((uint32_t(n) * HW + uint32_t(h0 + r) * uint32_t(a.W) + uint32_t(w0 + i)) * uint32_t(a.C) +
                               uint32_t(a.c0 + 4 * qd)) * ES;
        Elem<DT>::load4(F, ok ? addr : kOff, fill[u]);
    }
    Slot<COLS> sl;
    if (lo < hi) {
        load_slot(sl, lo);
        end_slot(sl, lo + j < hi);
        load_rows(sl.c[0]);
    }
#pragma unroll
    for (int u = 0; u < kFill; ++u) {
        const int x = threadIdx.x + u * kMBlock;
        const int qd = x % (4 * T), i = (x / (4 * T)) % COLS, r = x / (4 * T * COLS);
        if (x < kQuads) s_f[(i * kMRows + r) * kFq + qd] = f4v{fill[u][0], fill[u][1], fill[u][2], fill[u][3]};
    }

    // dF sums: lane (q, j), value r holds row h0 + 4q + r, channel c0 + 16t + j
    f4v accf[COLS][T];
#pragma unroll
    for (int i = 0; i < COLS; ++i)
#pragma unroll
        for (int t = 0; t < T; ++t) accf[i][t] = f4v{0.f, 0.f, 0.f, 0.f};
    float *sg = s_g + wave * kGs;
    // a step's rows in the wave's LDS: row j = slot j, its quads permuted in
    // each group of four by j / 4, so that neither the 16-byte writes (rows 4
    // apart start in the same bank) nor the transposed reads collide
    float *sg_wr = sg + j * S + ((q ^ (j >> 2)) << 2);
    const float *sg_rd[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) sg_rd[s] = sg + (4 * s + q) * S + (((j >> 2) ^ s) << 2) + (j & 3);
    __syncthreads();   // the feature rows are in LDS

    // P of slot 4s + q, row h0 + j (operand A of the dF product) where the
    // slot's cells keep that point: bit COLS * s + i of kept for column i
    float p[4][COLS];
    int kept = 0;
    auto load_probs = [&](const Slot<COLS> &t) {
        kept = 0;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            int m = 0;
#pragma unroll
            for (int i = 0; i < COLS / 2; ++i) {
                const int k01 = __shfl(t.keep[i], 4 * s + q) >> j;
                m |= ((k01 & 1) | (k01 >> 15 & 2)) << (2 * i);
            }
            const int d = __shfl(t.d, 4 * s + q);
            const uint32_t pt = (uint32_t(n * a.D + d) * uint32_t(a.H) + uint32_t(h0 + j)) * uint32_t(a.W) + uint32_t(w0);
#pragma unroll
            for (int i = 0; i < COLS; i += V)
                load_piece<DT, V>(P, (m >> i & ((1 << V) - 1)) != 0 ? (pt + uint32_t(i)) * ES : kOff, &p[s][i]);
            kept |= m << (COLS * s);
        }
    };
    Slot<COLS> next;
    if (lo < hi) {
        load_probs(sl);
        load_slot(next, lo + kMChunk);
    }

    for (int k = lo; k < hi; k += kMChunk) {
        // dP product: lane (q, j), value r is row h0 + 4q + r, slot j
        f4v accp[COLS];
#pragma unroll
        for (int i = 0; i < COLS; ++i) {
            accp[i] = f4v{0.f, 0.f, 0.f, 0.f};
            f4v part = accp[i];
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const f4v f = s_f[(i * kMRows + j) * kFq + 4 * t + q];
                f4v &to = t < 5 ? accp[i] : part;   // sums of at most 80 products, for their rounding
#pragma unroll
                for (int e = 0; e < 4; ++e) to = __builtin_amdgcn_mfma_f32_16x16x4f32(f[e], g[t][e], to, 0, 0, 0);
            }
            if constexpr (T > 5) accp[i] += part;
            // the rows into the wave's LDS; their registers then take the
            // next column's rows, which arrive while the dF product runs
#pragma unroll
            for (int t = 0; t < T; ++t) *reinterpret_cast<f4v *>(&sg_wr[16 * t]) = g[t];
            __builtin_amdgcn_wave_barrier();
            load_rows(i + 1 < COLS ? sl.c[(i + 1) % COLS] : k + kMChunk + j < hi ? next.c[0] : -1);
            __builtin_amdgcn_sched_barrier(0);
            // dF product: K = slot, N = channel, kRead slots quarters' reads
            // in flight at a time
            constexpr int kRead = T <= 5 ? 4 : T <= 6 ? 2 : 1;
#pragma unroll
            for (int s0 = 0; s0 < 4; s0 += kRead) {
                float gt[kRead][T];
#pragma unroll
                for (int s = 0; s < kRead; ++s)
#pragma unroll
                    for (int t = 0; t < T; ++t) gt[s][t] = sg_rd[s0 + s][16 * t];
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int s = 0; s < kRead; ++s) {
                    const float pm = kept >> (COLS * (s0 + s) + i) & 1 ? p[s0 + s][i] : 0.f;
#pragma unroll
                    for (int t = 0; t < T; ++t)
                        accf[i][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(pm, gt[s][t], accf[i][t], 0, 0, 0);
                }
            }
            __builtin_amdgcn_wave_barrier();
        }
        // the next step's P before this step's dP: loads and stores complete
        // in order, so a load behind a store would wait for it
        end_slot(next, k + kMChunk + j < hi);
        load_probs(next);
        __builtin_amdgcn_sched_barrier(0);
        if (a.want_dp) {
            // row h of bin d: the columns, V to a piece
            auto store_dp = [&](int d, int h, bool ok, float (&v)[COLS]) {
                const uint32_t off = ((uint32_t(n * a.D + d) * uint32_t(a.H) + uint32_t(h)) * uint32_t(a.W) + uint32_t(w0)) * 4u;
                if (a.accumulate_dp) {
#pragma unroll
                    for (int i = 0; i < COLS; ++i)
                        v[i] += __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(dP, int((ok & (w0 + i < a.W)) ? off + 4u * i : kOff), 0, 0));
                }
#pragma unroll
                for (int i = 0; i < COLS; i += V) {
                    const int at = int((ok & (w0 + i < a.W)) ? off + 4u * i : kOff);
                    if constexpr (V == 4)
                        __builtin_amdgcn_raw_buffer_store_b128(
                            (__attribute__((ext_vector_type(4))) uint32_t){__float_as_uint(v[0]), __float_as_uint(v[1]),
                                                                           __float_as_uint(v[2]), __float_as_uint(v[3])},
                            dP, at, 0, 0);
                    else if constexpr (V == 2)
                        __builtin_amdgcn_raw_buffer_store_b64(
                            (__attribute__((ext_vector_type(2))) uint32_t){__float_as_uint(v[i]), __float_as_uint(v[i + 1])},
                            dP, at, 0, 0);
                    else
                        store_f32(dP, uint32_t(at), v[i]);
                }
            };
            const bool real = k + j < hi;
            const int d0 = __builtin_amdgcn_readfirstlane(sl.d);
            // bit of column i and the lane's row r in a word of masks
            auto bit = [&](const int (&m)[COLS / 2], int i, int r) { return (m[i / 2] >> (4 * q + r + i % 2 * 16) & 1) != 0; };
            if (__ballot(real & (sl.d != d0 + j)) == 0) {
                // every bin of the step has one slot
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float v[COLS];
#pragma unroll
                    for (int i = 0; i < COLS; ++i) v[i] = bit(sl.keep, i, r) ? accp[i][r] : 0.f;
                    store_dp(sl.d, h0 + 4 * q + r, real & (h0 + 4 * q + r < a.H), v);
                }
            } else {
                // the slots' values meet in LDS (a bin's slots lie in one
                // step), so that every row of a bin is stored once
                float *mine = sg + (sl.d - d0) * kDpStride + 4 * q * COLS;
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int i = 0; i < COLS; ++i)
                        if (bit(sl.write, i, r)) mine[r * COLS + i] = bit(sl.keep, i, r) ? accp[i][r] : 0.f;
                __builtin_amdgcn_wave_barrier();
                // bins of this step: up to the last real slot's
                const int bins = __shfl(sl.d, min(hi - k, kMChunk) - 1) - d0 + 1;
                for (int x = lane; x < bins * kMRows; x += kWaveSize) {
                    const int h = h0 + x % kMRows;
                    typedef float fcv __attribute__((ext_vector_type(COLS)));
                    const fcv u = *reinterpret_cast<const fcv *>(&sg[x / kMRows * kDpStride + x % kMRows * COLS]);
                    float v[COLS];
#pragma unroll
                    for (int i = 0; i < COLS; ++i) v[i] = u[i];
                    store_dp(d0 + x / kMRows, h, h < a.H, v);
                }
                __builtin_amdgcn_wave_barrier();
            }
        }
        sl = next;
        load_slot(next, k + 2 * kMChunk);
    }

    if (!a.want_df) return;
    // the sums of all waves in LDS, kSumCols columns at a time, added in wave
    // order: wave r takes value r of every lane, so that its lane group q holds
    // all channels of row 4q + r
#pragma unroll
    for (int i0 = 0; i0 < COLS; i0 += kSumCols) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kSumCols; ++i)
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    s_all[(wave * kSumCols + i) * kSum + (t * 4 + r) * kWaveSize + lane] = accf[i0 + i][t][r];
        __syncthreads();
        const int h = h0 + 4 * q + wave;
#pragma unroll 1
        for (int i = 0; i < kSumCols; ++i) {
            const int w = w0 + i0 + i;
            const bool in = (h < a.H) & (w < a.W);
            float v[T];
            int bad = 0;
#pragma unroll
            for (int t = 0; t < T; ++t) {
                v[t] = 0.f;
#pragma unroll
                for (int u = 0; u < kMWaves; ++u) v[t] += s_all[(u * kSumCols + i) * kSum + (t * 4 + wave) * kWaveSize + lane];
                bad |= in && 16 * t + j < a.cn && !finite(v[t]) ? 1 << t : 0;
            }
            if (__ballot(bad != 0) != 0) {
                // (a group without one runs along: its rows are not taken)
                const Row<T> x = kept_row<DT, T>(P, G, a.cop, n, a.D, a.H, a.W, a.C, h, w, in, a.c0, j);
#pragma unroll
                for (int t = 0; t < T; ++t) v[t] = bad >> t & 1 ? x.v[t] : v[t];
            }
            const uint32_t row = (uint32_t(n) * HW + uint32_t(h) * uint32_t(a.W) + uint32_t(w)) * uint32_t(a.C) + uint32_t(a.c0 + j);
#pragma unroll
            for (int t = 0; t < T; ++t) store_f32(dF, in && 16 * t + j < a.cn ? (row + uint32_t(16 * t)) * 4u : kOff, v[t]);
        }
    }
}

template <int DT, int COLS, int V>
void launch_mma(const MmaArgs &a, dim3 grid, int tiles, hipStream_t s) {
    const dim3 block(kMBlock);
    switch (tiles) {
        case 1: hipLaunchKernelGGL((k_backward_mma<DT, 1, COLS, V>), grid, block, 0, s, a); break;
        case 2: hipLaunchKernelGGL((k_backward_mma<DT, 2, COLS, V>), grid, block, 0, s, a); break;
        case 3: hipLaunchKernelGGL((k_backward_mma<DT, 3, COLS, V>), grid, block, 0, s, a); break;
        case 4: hipLaunchKernelGGL((k_backward_mma<DT, 4, COLS, V>), grid, block, 0, s, a); break;
        case 5: hipLaunchKernelGGL((k_backward_mma<DT, 5, COLS, V>), grid, block, 0, s, a); break;
        case 6: hipLaunchKernelGGL((k_backward_mma<DT, 6, COLS, V>), grid, block, 0, s, a); break;
        default: hipLaunchKernelGGL((k_backward_mma<DT, 8, COLS, V>), grid, block, 0, s, a); break;
    }
}

template <int COLS, int V>
void launch_mma(const MmaArgs &a, int dtype, dim3 grid, int tiles, hipStream_t s) {
    switch (dtype) {
        case BEVPOOL_F32: launch_mma<BEVPOOL_F32, COLS, V>(a, grid, tiles, s); break;
        case BEVPOOL_BF16: launch_mma<BEVPOOL_BF16, COLS, V>(a, grid, tiles, s); break;
        default: launch_mma<BEVPOOL_F16, COLS, V>(a, grid, tiles, s); break;
    }
}

// Four columns to a workgroup, or two, for `bins` depth bins of all lists and
// frames and P and dP in pieces of `piece` columns. Four read the slots, P and dP
// in half as many accesses, which counts once there is more to move than the
// caches hold; two make twice the workgroups, three to a CU, and keep more loads
// in flight, the more so where a tilted rig's bins have several slots. Times in
// us, four against two, 32 x 88 and 118 bins unless said:
//   80 channels, level: one camera (5 thousand bins) 14.0 / 10.4, six (31) 24.4 /
//   22.8, two frames (62) 37.4 / 36.5, three (93) 45.8 / 50.3, eight (249) 126 /
//   156; eight frames of 40 bins (84) 60 / 56. Tilted by 1 degree: one frame 36 /
//   31, four (125) 91 / 84, five (156) 116 / 127.
//   32 channels, level: 40 bins (11) 9.0 / 8.7, two frames of them (21) 12.6 / 14.0.
//   1 degree: 31 22.4 / 21.9, 62 31.3 / 34.5.
//   128 channels, level: 125 94 / 89, 156 113 / 117, 64 x 176 x 236 bins (249) 165 /
//   173. 1 degree: 31 55 / 46, 249 287 / 263.
//   87 columns (one at a time), level, 80 channels: 125 84 / 80, 249 176 / 194; 128
//   channels: 249 254 / 225.
// Widths of 2 mod 4 move in pairs with two columns: 50 x 28, 80 channels, eight
// frames 65 us, one at a time with four 79.
bool four_columns(int tiles, int64_t bins, bool level, int piece) {
    if (piece == 2 || (tiles > 6 && (piece == 1 || !level))) return false;
    if (piece == 1 || tiles > 6) return bins >= 150000;
    if (tiles <= 2) return bins >= (level ? 20000 : 40000);
    return bins >= (level ? 90000 : 150000);
}

// Whether the per-row kernel is the faster one although the matrix cores could
// take the call, for `slots` slots in `bins` depth bins of the lists. Its time
// hardly grows with the slots, but with the slices: two above 80 channels, where
// the matrix cores take one up to 128. Times in us, rows against matrix cores, 32 x
// 88 x 118 bins, six cameras, one frame, fp32 unless said:
//   80 channels: tilted by 6 degrees (3.8 slots to a bin) 56 / 53, 8 (4.4) 56 / 64,
//   12 (5.3) 54 / 71, every point in a cell of its own (16) 121 / 151; four frames
//   173 / 139, 173 / 162, 177 / 192, 436 / 487; bf16 54 / 53, 54 / 64, 54 / 71, 122 / 154.
//   64: 50 / 46, 50 / 56, 50 / 61, 87 / 128. 128: 101 / 82, 101 / 97, 101 / 105, 178 / 242.
//   96 (rows of two slices of 48): 93 / 73 at 4.4, 92 / 82, 104 / 96 at 8, 178 / 174.
//   32: 45 / 44 at 5.3, 47 / 48 at 8, 49 / 88 at 16; 16: 44 / 36, 46 / 38, 47 / 68.
//   One camera (44 lists), 80: 34 / 41 at 5.3, 46 / 40 at 8, 47 / 73 at 16; 128: 76 /
//   53, 81 / 52, 86 / 96.
// Level, 87 columns (no piece to move), 16 channels: one frame (31 thousand bins)
// 22.8 / 22.9, two 31 / 37, eight 98 / 111; 32 channels, two 43 / 39.
bool by_rows(int64_t slots, int64_t bins, int64_t lists, int batch, int channels, int piece) {
    if (slots == 0) return true;               // a plan without lists
    if (slots == bins) return piece == 1 && channels <= 16 && bins * batch >= 50000;
    if (channels > 80 && channels <= 96) return false;
    const bool few = channels <= 32 || lists * batch < 256;
    return slots > (few ? 8 : 5) * bins;
}

template <int DT>
void launch_bwd(const BwdArgs &a, dim3 grid, int nch, hipStream_t s) {
    const dim3 block(kBBlock);
    switch (nch) {
        case 1: hipLaunchKernelGGL((k_backward<DT, 1>), grid, block, 0, s, a); break;
        case 2: hipLaunchKernelGGL((k_backward<DT, 2>), grid, block, 0, s, a); break;
        case 3: hipLaunchKernelGGL((k_backward<DT, 3>), grid, block, 0, s, a); break;
        case 4: hipLaunchKernelGGL((k_backward<DT, 4>), grid, block, 0, s, a); break;
        default: hipLaunchKernelGGL((k_backward<DT, 5>), grid, block, 0, s, a); break;
    }
}

}  // namespace
}  // namespace bevpool

using namespace bevpool;

int bevpool_launch_backward(const float *G, const void *P, const void *F,
                            const bevpool_plan_s *plan, float *dP, float *dF, int32_t batch,
                            int32_t channels, int32_t dtype, hipStream_t stream) {
    const bevpool_geometry &g = plan->geom;
    const int64_t n_pix = int64_t(g.n_cams) * g.feat_h * g.feat_w;
    const int64_t esize = dtype == BEVPOOL_F32 ? 4 : 2;
    const int64_t p_bytes = plan->n_points * esize;
    const int64_t f_bytes = n_pix * channels * esize;
    const int64_t g_bytes = int64_t(plan->n_cells) * channels * 4;
    const int64_t dp_bytes = plan->n_points * 4;
    const int64_t df_bytes = n_pix * channels * 4;
    constexpr int64_t kLimit = int64_t(1) << 31;
    if (p_bytes >= kLimit || f_bytes >= kLimit || g_bytes >= kLimit || dp_bytes >= kLimit ||
        df_bytes >= kLimit)
        return bevpool_fail(BEVPOOL_ERR_OVERFLOW,
                            "channels=%d: one frame's gradient or input tensor reaches 2 GiB",
                            channels);
    if (batch > 65535)
        return bevpool_fail(BEVPOOL_ERR_INVALID_ARG, "batch=%d exceeds 65535 frames per call", batch);

    // v columns of P and of dP move as one piece
    auto pieces = [&](int v) {
        return g.feat_w % v == 0 && reinterpret_cast<uintptr_t>(P) % (v * esize) == 0 &&
               reinterpret_cast<uintptr_t>(dP) % (4 * v) == 0;
    };
    const int piece = pieces(4) ? 4 : pieces(2) ? 2 : 1;
    const int32_t quads_w = (g.feat_w + kBwdCols - 1) / kBwdCols, blocks_h = (g.feat_h + kBwdRows - 1) / kBwdRows;
    const int64_t lists = int64_t(g.n_cams) * quads_w * blocks_h, bins = lists * g.n_depth;

    // Matrix-core kernel where feature and gradient rows move as 4-element
    // quads: channels % 4 == 0 and aligned rows. Otherwise the per-row kernel.
    const bool quads = channels % 4 == 0 && reinterpret_cast<uintptr_t>(F) % (4 * esize) == 0 &&
                       reinterpret_cast<uintptr_t>(G) % 16 == 0;
    if (quads && !by_rows(plan->n_bwd_slots, bins, lists, batch, channels, piece)) {
        MmaArgs m;
        m.P = static_cast<const char *>(P);
        m.F = static_cast<const char *>(F);
        m.G = G;
        m.dP = dP;
        m.dF = dF;
        m.cop = plan->cell_of_point;
        m.offs = plan->bwd_offs;
        m.bins = plan->bwd_bins;
        m.cells = plan->bwd_cells;
        m.masks = plan->bwd_masks;
        m.D = g.n_depth;
        m.H = g.feat_h;
        m.W = g.feat_w;
        m.C = channels;
        m.p_bytes = uint32_t(p_bytes);
        m.f_bytes = uint32_t(f_bytes);
        m.g_bytes = uint32_t(g_bytes);
        m.dp_bytes = dP ? uint32_t(dp_bytes) : 0u;
        m.df_bytes = dF ? uint32_t(df_bytes) : 0u;
        m.quads_w = quads_w;
        m.blocks_h = blocks_h;
        m.want_dp = dP != nullptr;
        m.want_df = dF != nullptr;
        // equal slices of at most kMSlice channels, whole 16-channel tiles
        const int n = (channels + kMSlice - 1) / kMSlice;
        const int slice = ((channels + n - 1) / n + 15) / 16 * 16;
        for (int c0 = 0; c0 < channels; c0 += slice) {
            m.c0 = c0;
            m.cn = std::min(slice, channels - c0);
            m.accumulate_dp = c0 > 0;
            const int tiles = (m.cn + 15) / 16;
            const bool four = four_columns(tiles, bins * batch, plan->n_bwd_slots == bins, piece);
            const dim3 grid(uint32_t(four ? lists : 2 * lists), batch);
            if (four && piece == 4) launch_mma<4, 4>(m, dtype, grid, tiles, stream);
            else if (four) launch_mma<4, 1>(m, dtype, grid, tiles, stream);
            else if (piece != 1) launch_mma<2, 2>(m, dtype, grid, tiles, stream);
            else launch_mma<2, 1>(m, dtype, grid, tiles, stream);
            BEVPOOL_HIP(hipGetLastError());
        }
        return BEVPOOL_OK;
    }

    const int n_slices = (channels + kBwdSliceChannels - 1) / kBwdSliceChannels;
    const int slice_c = (channels + n_slices - 1) / n_slices;
    const int nch = (slice_c + 15) / 16;

    BwdArgs a;
    a.P = static_cast<const char *>(P);
    a.F = static_cast<const char *>(F);
    a.G = G;
    a.dP = dP;
    a.dF = dF;
    a.cop = plan->cell_of_point;
    a.combo_cells = plan->combo_cells;
    a.N = g.n_cams;
    a.D = g.n_depth;
    a.H = g.feat_h;
    a.W = g.feat_w;
    a.HW = g.feat_h * g.feat_w;
    a.C = channels;
    a.p_bytes = uint32_t(p_bytes);
    a.f_bytes = uint32_t(f_bytes);
    a.g_bytes = uint32_t(g_bytes);
    a.dp_bytes = dP ? uint32_t(dp_bytes) : 0u;
    a.df_bytes = dF ? uint32_t(df_bytes) : 0u;
    a.cop_bytes = uint32_t(plan->n_points * 4);
    a.cc_bytes = uint32_t(int64_t(g.n_cams) * g.n_depth * g.feat_w * 4);
    a.items_w = (g.feat_w + kBCols - 1) / kBCols;
    a.items_h = (g.feat_h + kBRows - 1) / kBRows;
    a.part = (g.n_depth + kBWaves - 1) / kBWaves;
    a.want_dp = dP != nullptr;
    a.want_df = dF != nullptr;
    const dim3 grid(g.n_cams * a.items_w * a.items_h, batch);
    for (int s = 0; s < n_slices; ++s) {
        a.c0 = s * slice_c;
        a.cn = std::min(slice_c, channels - a.c0);
        a.accumulate_dp = s > 0;
        switch (dtype) {
            case BEVPOOL_F32: launch_bwd<BEVPOOL_F32>(a, grid, nch, stream); break;
            case BEVPOOL_BF16: launch_bwd<BEVPOOL_BF16>(a, grid, nch, stream); break;
            default: launch_bwd<BEVPOOL_F16>(a, grid, nch, stream); break;
        }
        BEVPOOL_HIP(hipGetLastError());
    }
    return BEVPOOL_OK;
}
