// Frequency nodes of the split-form likelihood (gw_nodes.h): the plan of a
// batch, the weighting of the data onto the nodes, and the nodes' tables.
//
// Measured on MI355X, a whole gw_lnl_batch call (every bin summed per sample ->
// nodes): 4096 heavy binaries, 3 detectors, 259,585 bins: 1.60 ms -> 60 us;
// 4096 neutron-star rows, 1,040,897 bins from 15 Hz: 6.30 ms -> 0.20 ms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "gw_build_id.h"
#include "gw_device_math.h"
#include "gw_internal.h"
#include "gw_nodes.h"
#include "gw_reduce.h"
#include "gw_template.h"

namespace gw {

typedef double double4_t __attribute__((ext_vector_type(4)));

// Weight t < 16 of a point at s = 2 x - 1 in its cell: sum_j coef[j][t] s^j;
// weight 31 - t is weight t at -s.
static __constant__ double resample_coef[GW_RESAMPLE_DEGREE + 1][kTaps / 2] = {GW_RESAMPLE_COEF_VALUES};
static_assert(GW_RESAMPLE_DEGREE % 2 == 1, "even and odd parts of equal length");

// ---------------------------------------------------------------- the plan
// The plan of a batch from the ranges of its phase coefficients, written to
// `p` (LDS).  All kBlock threads call it; `red` holds kPlanScratch doubles.
constexpr int kPlanSlices = kBlock / kStats;                       // 14 slices of the entries
constexpr int kPlanScratch = kPlanSlices * kStats + 2 * kStatPairs + 3 * kNodeSpacings;   // 5 kNodeSpacings ints at the end

__device__ __forceinline__ void make_node_plan(double f_low, double df, int64_t n_bins, int n_det,
                                               const double *__restrict__ stats, int n_stats, NodePlan &p,
                                               double *red)
{
    double *const half = red + kPlanSlices * kStats, *const mid = half + kStatPairs;
    int *const first = reinterpret_cast<int *>(mid + kStatPairs);
    const int t = threadIdx.x;
    const NodeBand band = node_band(f_low, df, n_bins);      // does not wait for the ranges
    if (t < kPlanSlices * kStats) {
        const int j = t % kStats;
        double m = j % 2 == 0 ? INFINITY : -INFINITY;
        for (int e = t / kStats; e < n_stats; e += kPlanSlices) {
            const double v = stats[(int64_t)e * kStats + j];
            m = j % 2 == 0 ? fmin(m, v) : fmax(m, v);
        }
        red[t] = m;
    }
    __syncthreads();
    if (t < kStatPairs) {
        double lo = INFINITY, hi = -INFINITY;
        for (int e = 0; e < kPlanSlices; ++e) {
            lo = fmin(lo, red[e * kStats + 2 * t]);
            hi = fmax(hi, red[e * kStats + 2 * t + 1]);
        }
        double m, h;
        node_middle(lo, hi, m, h);
        mid[t] = m;
        half[t] = h;
    }
    __syncthreads();
    const RateBound r = node_bound(half, band);
    // probe t: the spacings that the bound at its frequency allows; then those that fail, per spacing
    const int widest = node_allowed(node_rate(r, node_probe(band, t)), df);
    int *const failing = first + kNodeSpacings;
#pragma unroll
    for (int g = 0; g < kNodeSpacings; ++g) {
        const int n = __popcll(__ballot(widest <= g));
        if (t % 64 == g) failing[(t / 64) * kNodeSpacings + g] = n;
    }
    __syncthreads();
    if (failing[0] + failing[kNodeSpacings] + failing[2 * kNodeSpacings] + failing[3 * kNodeSpacings] == kBlock) {
        // no spacing serves even the top of the band: every bin is summed as it is (1 detector x
        // 32,768 bins x 1024 rows with arrival times all over the segment: 64.4 -> 62.5 us)
        if (t == 0) node_totals(0, (int)n_bins, 0, 0, p);
        if (t < kMids) p.mid[t] = 0.0;
        __syncthreads();
        return;
    }
    if (t < kNodeSpacings)
        first[t] = node_first_bin(band, t, failing[t] + failing[kNodeSpacings + t] + failing[2 * kNodeSpacings + t] +
                                               failing[3 * kNodeSpacings + t]);
    __syncthreads();
    if (t < 64) {
        int k_first[kNodeSpacings];
#pragma unroll
        for (int i = 0; i < kNodeSpacings; ++i) k_first[i] = first[i];
        NodeLevel v{};
        int k_bin = 0, chunks = 0, nodes = 0;
        // lane t holds level t from the widest spacing, i.e. from the top of the band
        const int n = node_pick(k_first, (int)n_bins, n_det, t, v, k_bin, chunks, nodes);
        if (t < n) p.level[n - 1 - t] = v;
        if (t == 0) node_totals(n, k_bin, chunks, nodes, p);
        if (t < kMids) {
            // kRecC8 .. kRecC0 from the pairs' order; the constant kRecC5 needs no reference
            constexpr int pair[kMids] = {0, 1, 2, 3, -1, 4, 5, 6, 7, 8};
            int at = -1;
#pragma unroll
            for (int i = 0; i < kMids; ++i)
                if (i == t) at = pair[i];
            p.mid[t] = at >= 0 && n > 0 ? mid[at] : 0.0;
        }
    }
    __syncthreads();
}

__device__ __forceinline__ PhaseCoef reference_coef(const NodePlan &p) { return load_coef(p.mid, 1, 0); }

// ---------------------------------------------------------------- weighting
// Chunk of the weighting: up to kSpreadBins bins of one level (or of the bins
// summed one by one).
//
// D e^{-i ref} of a chunk's bins goes to LDS (or, for single bins, to memory
// as it is).  For the nodes the chunk is a matrix product: with the weights
// of a cell's q bins as a 32 x q matrix A (the same for every cell of a level) and
// the cells' D as columns, Y = A D gives each cell's share of its 32 nodes,
// and a node adds the Y of the (at most 32) cells it serves.  A is formed
// in registers from the weight polynomials, D comes from LDS, and
// v_mfma_f64_16x16x4 does the product: a wave holds 16 columns (node_pack
// cells) of both halves of the taps; with few cells the waves share out the q
// bins instead, and the parts are added with the cells' Y.
// What bounds it: per bin one division per detector, one reference phasor and 64
// n_det multiply-adds (a third more in the matrix instructions' unused columns),
// against 48 + 24 n_det bytes read.  3 detectors, 259,585 bins: 26 us, of which a block
// spends 5 on the plan, 5 waiting for its bins and 5 in the product; 40 us with the
// levels worked out by one thread, two blocks a CU (two turns of chunks) and the sums
// of every chunk reduced through LDS permutes.
template <int NDET>
struct SpreadShape {
    static constexpr int kComp = 2 * NDET;
    static constexpr int kPack = node_pack(NDET);
    static constexpr int kStride = kSpreadBins + 4;          // LDS row of one component, in doubles
    static constexpr int kPacks = 4;                         // packs of cells per batch
    static constexpr int kMaxNodes = kSpreadBins / 8 + kTaps - 1;
    static constexpr int kAcc = (kMaxNodes * kComp + kBlock - 1) / kBlock;
    static constexpr size_t kLds = sizeof(double) * ((size_t)kComp * kStride + (size_t)kPacks * kTaps * 16);
};

template <int NDET>
__device__ __forceinline__ void spread_chunk(const NodeEvent &ev, const NodePlan &plan, int chunk, bool norm,
                                             double *lds_d, double *lds_y, double (&acc)[kPrepPerDet * NDET])
{
    using S = SpreadShape<NDET>;
    constexpr int kComp = S::kComp, kPack = S::kPack, kStride = S::kStride;
    const int t = threadIdx.x, lane = t % 64, wave = t / 64;
    const int64_t n_bins = ev.n_bins;
    // where the chunk lies
    const bool single = chunk < plan.bin_chunks;
    int l = 0;
    if (!single)
        while (l + 1 < plan.n_levels && chunk >= plan.level[l + 1].chunk0) ++l;
    const NodeLevel &v = plan.level[l];
    const int local = single ? chunk : chunk - v.chunk0;
    const int sub = single ? 0 : local % v.subs;
    const int cell0 = single ? 0 : local / v.subs * v.cpc;
    const int j0 = single ? 0 : sub * v.sub_bins;
    const int sub_bins = single ? kSpreadBins : v.sub_bins;
    const int n_here = single ? kSpreadBins : v.cpc * sub_bins;
    const int64_t k_base = single ? (int64_t)chunk * kSpreadBins : v.k0 + (int64_t)cell0 * v.q + j0;
    const int64_t k_end = single ? plan.k_bin : v.k1;
    const PhaseCoef ref = reference_coef(plan);

    // every load of a bin is issued before the first use (one bin at a time:
    // both of a thread's bins would spill at three blocks a CU)
#pragma unroll 1
    for (int b = t; b < kSpreadBins; b += kBlock) {
        const int cell = single ? 0 : (int)((unsigned)b / (unsigned)sub_bins), j = b - cell * sub_bins;
        const int64_t k = k_base + (single ? 0 : (int64_t)cell * v.q) + j;
        const bool live = b < n_here && k < k_end && (single || j0 + j < v.q);
        const int64_t at = live ? k : 0;
        const Tab1 t1 = ev.tab1[at];
        const double amp = ev.tab2[at].amp;
        double psd[NDET];
        double2 x[NDET];
#pragma unroll
        for (int d = 0; d < NDET; ++d) {
            psd[d] = ev.psd[(int64_t)d * n_bins + at];
            x[d] = ev.data[(int64_t)d * n_bins + at];
        }
        double er, ei;
        gw_phasor_turns(turns_phase(ref, t1), er, ei);
#pragma unroll
        for (int d = 0; d < NDET; ++d) {
            const double w = (psd[d] > 0.0 && psd[d] < INFINITY) ? 1.0 / psd[d] : NAN;
            const double scale = 4.0 * ev.df * amp * w;
            const double xr = scale * x[d].x, xi = -scale * x[d].y;
            const double dr = live ? xr * er - xi * ei : 0.0, di = live ? xr * ei + xi * er : 0.0;
            if (live) {
                acc[kPrepPerDet * d] += (x[d].x * x[d].x + x[d].y * x[d].y) * w;
                acc[kPrepPerDet * d + 1] += amp * amp * w;
                if (norm) acc[kPrepPerDet * d + 2] += log(2.0 * GW_PI * psd[d]);
            }
            if (single) {
                if (live) ev.dcoef[(int64_t)d * n_bins + at] = make_double2(dr, di);
            } else {
                lds_d[(2 * d) * kStride + b] = dr;
                lds_d[(2 * d + 1) * kStride + b] = di;
            }
        }
    }
    if (!single && t < 4 * kComp) lds_d[(t / 4) * kStride + kSpreadBins + t % 4] = 0.0;
    if (single) return;
    // the tap this lane weights (and its mirror image)
    double coef[GW_RESAMPLE_DEGREE + 1];
#pragma unroll
    for (int j = 0; j <= GW_RESAMPLE_DEGREE; ++j) coef[j] = resample_coef[j][t % 16];
    __syncthreads();

    // this lane's column, and its place among 4 bins
    const int col = lane % 16, kk = lane / 16;
    const double inv_q2 = 2.0 / (double)v.q;
    const int cell_of_col = col / kComp, comp = col % kComp;
    const bool col_live = cell_of_col < kPack;
    double node[S::kAcc];
#pragma unroll
    for (int i = 0; i < S::kAcc; ++i) node[i] = 0.0;
    const int n_nodes = v.cpc + kTaps - 1;
    for (int cb = 0; cb < v.cpc; cb += kPack * S::kPacks) {
        const int cells = min(kPack * S::kPacks, v.cpc - cb);
        const int packs = (cells + kPack - 1) / kPack;
        // waves share the packs, and the bins of a cell when there are fewer packs than waves
        const int kparts = packs == 1 ? 4 : packs == 2 ? 2 : 1;
        const int groups = 4 / kparts;               // waves per part
        const int part = wave / groups, pack0 = wave % groups;
        const int steps = (sub_bins + 3) / 4;
        const int s0 = steps * part / kparts, s1 = steps * (part + 1) / kparts;
        if (pack0 < packs) {
            const int pk = pack0;                    // kPacks packs at most: one a wave
            double4_t y0 = {0.0, 0.0, 0.0, 0.0}, y1 = y0;
            const int cell = cb + pk * kPack + cell_of_col;
            const bool on = col_live && cell < v.cpc;
            const double *dc = lds_d + comp * kStride + (on ? cell * sub_bins : 0);
#pragma unroll 2
            for (int s = s0; s < s1; ++s) {
                const int j = 4 * s + kk;
                const double x = (double)(j0 + j) * inv_q2 - 1.0;
                const double z = x * x;
                double even = coef[GW_RESAMPLE_DEGREE - 1], odd = coef[GW_RESAMPLE_DEGREE];
#pragma unroll
                for (int i = GW_RESAMPLE_DEGREE - 3; i >= 0; i -= 2) {
                    even = __builtin_fma(even, z, coef[i]);
                    odd = __builtin_fma(odd, z, coef[i + 1]);
                }
                // taps col and 31 - col
                const double w0 = __builtin_fma(x, odd, even), w1 = __builtin_fma(-x, odd, even);
                const double d = on && j < sub_bins ? dc[j] : 0.0;
                y0 = __builtin_amdgcn_mfma_f64_16x16x4f64(w0, d, y0, 0, 0, 0);
                y1 = __builtin_amdgcn_mfma_f64_16x16x4f64(w1, d, y1, 0, 0, 0);
            }
            // row kk + 4 r of a 16 x 16 result is in register r; the second product's rows are
            // the upper taps from the top down
            double *y = lds_y + (part * packs + pk) * kTaps * 16 + col;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                y[(kk + 4 * r) * 16] = y0[r];
                y[(kTaps - 1 - kk - 4 * r) * 16] = y1[r];
            }
        }
        __syncthreads();
        // node n adds tap n - c of every cell c it serves, in cell order
#pragma unroll
        for (int i = 0; i < S::kAcc; ++i) {
            const int item = t + kBlock * i;
            const int n = item / kComp, cm = item % kComp;
            if (n < n_nodes) {
                const int c_lo = max(cb, n - (kTaps - 1)), c_hi = min(cb + cells - 1, n);
                for (int c = c_lo; c <= c_hi; ++c) {
                    const int pk = (c - cb) / kPack, at = (c - cb) % kPack * kComp + cm;
                    for (int pt = 0; pt < kparts; ++pt)
                        node[i] += lds_y[((pt * packs + pk) * kTaps + (n - c)) * 16 + at];
                }
            }
        }
        __syncthreads();
    }
    const int64_t slot = v.k0 + (int64_t)local * n_nodes;
    double *out = reinterpret_cast<double *>(ev.dcoef);
#pragma unroll
    for (int i = 0; i < S::kAcc; ++i) {
        const int item = t + kBlock * i;
        const int n = item / kComp, cm = item % kComp;
        if (n < n_nodes) out[2 * ((int64_t)(cm / 2) * n_bins + slot + n) + cm % 2] = node[i];
    }
}

// One event: every block makes the plan for itself (it costs less than a launch
// of its own) and takes chunks blockIdx.x, + gridDim.x, ...; block 0 leaves
// the plan for the kernels that follow.
// Three blocks a CU where the registers allow it (up to 3 detectors): a
// chunk is a chain of short phases, and one more block hides their latency.
template <int NDET>
__device__ __forceinline__ void spread_block(const NodeEvent &ev, const NodePlan &plan, int block, bool norm,
                                             double *lds, double *red)
{
    constexpr int n = kPrepPerDet * NDET;
    double *const lds_y = lds + SpreadShape<NDET>::kComp * SpreadShape<NDET>::kStride;
    double acc[n];
#pragma unroll
    for (int i = 0; i < n; ++i) acc[i] = 0.0;
    for (int c = block; c < plan.n_chunks; c += ev.spread_blocks)
        spread_chunk<NDET>(ev, plan, c, norm, lds, lds_y, acc);
    // the block's share of the event sums: wave sums, then the waves in order
    const int wave = threadIdx.x / 64;
#pragma unroll
    for (int i = 0; i < n; ++i) {
        const double s = wave_sum(acc[i]);
        if (threadIdx.x % 64 == 0) red[wave * n + i] = s;
    }
    __syncthreads();
    const int t = threadIdx.x;
    if (t < n) ev.prep[(int64_t)block * n + t] = ((red[t] + red[n + t]) + red[2 * n + t]) + red[3 * n + t];
}

// A plan moved by all threads of a block.
__device__ __forceinline__ void copy_plan(NodePlan *to, const NodePlan *from)
{
    const int *src = reinterpret_cast<const int *>(from);
    int *dst = reinterpret_cast<int *>(to);
    for (int i = threadIdx.x; i < (int)(sizeof(NodePlan) / sizeof(int)); i += kBlock) dst[i] = src[i];
}

template <int NDET>
__global__ __launch_bounds__(kBlock, NDET <= 3 ? 3 : 2) void node_spread_kernel(NodeEvent ev, int norm)
{
    extern __shared__ double lds[];
    __shared__ NodePlan plan;
    __shared__ double red[kPlanScratch];
    static_assert(kPlanScratch >= 4 * kPrepPerDet * NDET, "the waves' sums share the plan's scratch");
    make_node_plan(ev.f_low, ev.df, ev.n_bins, NDET, ev.stats, ev.n_stats, plan, red);
    if (blockIdx.x == 0) copy_plan(ev.plan, &plan);
    spread_block<NDET>(ev, plan, blockIdx.x, norm != 0, lds, red);
}

// ---------------------------------------------------------------- ragged calls
__device__ __forceinline__ NodeEvent node_event(const RaggedEvent &re)
{
    NodeEvent ev;
    ev.n_bins = re.n_bins;
    ev.n_det = re.n_det;
    ev.f_low = re.f_low;
    ev.df = re.df;
    ev.data = re.data;
    ev.psd = re.psd;
    ev.tab1 = re.tab1;
    ev.tab2 = re.tab2;
    ev.dcoef = re.dcoef;
    ev.prep = re.prep;
    ev.spread_blocks = re.spread_blocks;
    ev.sums = re.sums;
    ev.stats = re.stats;
    ev.n_stats = re.n_stats;
    ev.plan = re.plan;
    return ev;
}

// Block e: event e's plan.
__global__ __launch_bounds__(kBlock) void ragged_plan_kernel(const RaggedEvent *__restrict__ events)
{
    __shared__ NodePlan plan;
    __shared__ double red[kPlanScratch];
    const RaggedEvent &re = events[blockIdx.x];
    make_node_plan(re.f_low, re.df, re.n_bins, re.n_det, re.stats, re.n_stats, plan, red);
    copy_plan(re.plan, &plan);
}

// Block (e, i) = map[b]: chunks i, + spread_blocks, ... of event e.
template <int NDET>
__global__ __launch_bounds__(kBlock, NDET <= 3 ? 3 : 2) void ragged_spread_kernel(
    const RaggedEvent *__restrict__ events, const int2 *__restrict__ map, int norm)
{
    extern __shared__ double lds[];
    __shared__ NodePlan plan;
    __shared__ double red[4 * kPrepPerDet * NDET];
    const int2 em = map[blockIdx.x];
    const RaggedEvent &re = events[em.x];
    copy_plan(&plan, re.plan);
    const NodeEvent ev = node_event(re);
    __syncthreads();
    spread_block<NDET>(ev, plan, em.y, norm != 0, lds, red);
}

// ---------------------------------------------------------------- nodes and sums
// Work of one event after the weighting, item by item: the tables of node i
// (item < n_nodes), then node sums by groups of kCombineLanes lanes (node,
// detector): lane j adds the partials j, j + 8, ... that reach the node, in chunk order,
// then a fixed butterfly.
constexpr int kCombineLanes = 8;

__device__ __forceinline__ const NodeLevel &node_level_of(const NodePlan &p, int node)
{
    int l = 0;
    while (l + 1 < p.n_levels && node >= p.level[l + 1].node0) ++l;
    return p.level[l];
}

__device__ __forceinline__ void combine_items(const NodeEvent &ev, const NodePlan &p, int64_t first, int64_t stride)
{
    // the tables' items fill whole waves, so that a group's 8 lanes stay together
    const int64_t n_tab = ((int64_t)p.n_nodes + 63) / 64 * 64;
    const int64_t n_sum = (int64_t)p.n_nodes * ev.n_det * kCombineLanes;
    for (int64_t i = first; i < n_tab + n_sum; i += stride) {
        if (i < n_tab) {
            if (i >= p.n_nodes) continue;
            const NodeLevel &v = node_level_of(p, (int)i);
            const int n = (int)i - v.node0;
            Tab1 t1;
            Tab2 t2;
            freq_tables(bin_frequency(ev.f_low, ev.df, v.k0 + (int64_t)(n - kTapsBelow) * v.q), t1, t2);
            reinterpret_cast<Tab1 *>(ev.dcoef + v.k0 + node_slots(v) + node_count(v))[n] = t1;
            continue;
        }
        const int64_t w = (i - n_tab) / kCombineLanes;
        const int j = (int)((i - n_tab) % kCombineLanes);
        const int d = (int)(w / p.n_nodes);
        const int node = (int)(w % p.n_nodes);
        const NodeLevel &v = node_level_of(p, node);
        const int n = node - v.node0;
        const int per = v.cpc + kTaps - 1;
        const int groups = v.n_chunks / v.subs;                    // runs of cpc cells
        const int g_lo = n >= per ? (n - per) / v.cpc + 1 : 0;     // first run whose nodes reach n
        const int g_hi = min(groups - 1, n / v.cpc);
        double re = 0.0, im = 0.0;
        const double2 *src = ev.dcoef + (int64_t)d * ev.n_bins + v.k0;
        for (int c = g_lo * v.subs + j; c < (g_hi + 1) * v.subs; c += kCombineLanes) {
            const double2 x = src[(int64_t)c * per + (n - c / v.subs * v.cpc)];
            re += x.x;
            im += x.y;
        }
#pragma unroll
        for (int off = kCombineLanes / 2; off > 0; off >>= 1) {
            re += __shfl_xor(re, off, 64);
            im += __shfl_xor(im, off, 64);
        }
        if (j == 0) ev.dcoef[(int64_t)d * ev.n_bins + v.k0 + node_slots(v) + n] = make_double2(re, im);
    }
}

// Blocks 0 .. kPrepPerDet n_det - 1: the event sums; the others: the nodes.
__global__ __launch_bounds__(kBlock) void node_combine_kernel(NodeEvent ev, unsigned *__restrict__ queue)
{
    __shared__ NodePlan plan;
    __shared__ double red[kBlock];
    copy_plan(&plan, ev.plan);
    __syncthreads();
    const int n_sums = kPrepPerDet * ev.n_det;
    if ((int)blockIdx.x < n_sums) {
        const double s = column_total(ev.spread_blocks, n_sums, blockIdx.x, ev.prep, red);
        if (threadIdx.x == 0) ev.sums[blockIdx.x] = s;
        if (queue && blockIdx.x == 0 && threadIdx.x < 2 * kQueues) queue[threadIdx.x] = 0u;
        return;
    }
    combine_items(ev, plan, (int64_t)(blockIdx.x - n_sums) * kBlock + threadIdx.x,
                  (int64_t)(gridDim.x - n_sums) * kBlock);
}

// Block (e, i) = map[b] of a ragged call: event e's sums (i = 0), or a share of its nodes.
__global__ __launch_bounds__(kBlock) void ragged_combine_kernel(const RaggedEvent *__restrict__ events,
                                                                const int2 *__restrict__ map)
{
    __shared__ NodePlan plan;
    __shared__ double red[kBlock];
    const int2 em = map[blockIdx.x];
    const RaggedEvent &re = events[em.x];
    if (em.y == 0) {
        const int n_sums = kPrepPerDet * re.n_det;
        for (int j = 0; j < n_sums; ++j) {
            const double s = column_total(re.spread_blocks, n_sums, j, re.prep, red);
            if (threadIdx.x == 0) re.sums[j] = s;
        }
        return;
    }
    copy_plan(&plan, re.plan);
    const NodeEvent ev = node_event(re);
    __syncthreads();
    combine_items(ev, plan, (int64_t)(em.y - 1) * kBlock + threadIdx.x, (int64_t)(re.combine_blocks - 1) * kBlock);
}

// ---------------------------------------------------------------- launchers
template <int NDET>
static hipError_t ragged_spread(const RaggedLaunch &r, const RaggedClass &c, int norm, hipStream_t stream)
{
    hipLaunchKernelGGL(ragged_spread_kernel<NDET>, dim3((unsigned)c.n_spread), dim3(kBlock), SpreadShape<NDET>::kLds,
                       stream, r.events, c.spread_map, norm);
    return hipGetLastError();
}

hipError_t launch_ragged_spread(const RaggedLaunch &r, hipStream_t stream)
{
    const int norm = (r.flags & GW_FLAG_ADD_NORM) ? 1 : 0;
    for (int i = 0; i < r.n_classes; ++i) {
        const RaggedClass &c = r.classes[i];
        hipError_t e = hipErrorInvalidValue;
        switch (c.n_det) {
        case 1: e = ragged_spread<1>(r, c, norm, stream); break;
        case 2: e = ragged_spread<2>(r, c, norm, stream); break;
        case 3: e = ragged_spread<3>(r, c, norm, stream); break;
        case 4: e = ragged_spread<4>(r, c, norm, stream); break;
        case 5: e = ragged_spread<5>(r, c, norm, stream); break;
        case 6: e = ragged_spread<6>(r, c, norm, stream); break;
        case 7: e = ragged_spread<7>(r, c, norm, stream); break;
        case 8: e = ragged_spread<8>(r, c, norm, stream); break;
        default: break;
        }
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_ragged_plans(const RaggedLaunch &r, hipStream_t stream)
{
    hipLaunchKernelGGL(ragged_plan_kernel, dim3((unsigned)r.n_events), dim3(kBlock), 0, stream, r.events);
    return hipGetLastError();
}

hipError_t launch_ragged_combine(const RaggedLaunch &r, hipStream_t stream)
{
    hipLaunchKernelGGL(ragged_combine_kernel, dim3((unsigned)r.n_combine), dim3(kBlock), 0, stream, r.events,
                       r.combine_map);
    return hipGetLastError();
}

template <int NDET>
static hipError_t spread(const NodeEvent &ev, bool norm, hipStream_t stream)
{
    hipLaunchKernelGGL(node_spread_kernel<NDET>, dim3((unsigned)ev.spread_blocks), dim3(kBlock), SpreadShape<NDET>::kLds,
                       stream, ev, norm ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_node_spread(const NodeEvent &ev, bool norm, hipStream_t stream)
{
    switch (ev.n_det) {
    case 1: return spread<1>(ev, norm, stream);
    case 2: return spread<2>(ev, norm, stream);
    case 3: return spread<3>(ev, norm, stream);
    case 4: return spread<4>(ev, norm, stream);
    case 5: return spread<5>(ev, norm, stream);
    case 6: return spread<6>(ev, norm, stream);
    case 7: return spread<7>(ev, norm, stream);
    case 8: return spread<8>(ev, norm, stream);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_node_combine(const NodeEvent &ev, unsigned *queue, hipStream_t stream)
{
    // enough threads for 2,000 nodes of 3 detectors in one pass; more nodes take turns
    const int64_t most = (ev.n_bins / node_spacing(0) + 64) * (kCombineLanes * ev.n_det + 1);
    const int64_t blocks = std::min<int64_t>((most + kBlock - 1) / kBlock, 256);
    hipLaunchKernelGGL(node_combine_kernel, dim3((unsigned)(kPrepPerDet * ev.n_det + blocks)), dim3(kBlock), 0, stream,
                       ev, queue);
    return hipGetLastError();
}

}  // namespace gw

GW_DEFINE_SOURCE_HASH(nodes)
