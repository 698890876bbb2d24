// Frequency nodes of the split-form likelihood (gw_nodes.h): the plan of a
// batch, the weighting of the data onto the nodes, and the nodes' tables.
//
// Measured on MI355X, a whole gw_lnl_batch call (every bin summed per sample ->
// nodes): 4096 heavy binaries, 3 detectors, 259,585 bins: 1.60 ms -> 76 us;
// 4096 neutron-star rows, 1,040,897 bins from 15 Hz: 6.27 ms -> 0.25 ms.
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

// Weight t of a point at s = 2 x - 1 in its cell: sum_j coef[j][t] s^j.
static __constant__ double resample_coef[GW_RESAMPLE_DEGREE + 1][kTaps] = {GW_RESAMPLE_COEF_VALUES};

// ---------------------------------------------------------------- the plan
// Half the batch's range of every phase coefficient about the reference, as
// what it adds to |dx/df| (see node_rate).
struct RateBound {
    double tau, c7, c6, c6l, c5l, c4, c3, c2, c0;
};

// Bound on |dx_d/df| (turns per Hz) of x_d less the reference's phase at
// frequency u^3, over every evaluated sample and detector: the derivative of
//   x = tau f + c7 u^2 + (c6 + c6l L) u + (c5 + c5l L) + c4/u + c3/u^2 + c2/u^3 + c0/u^5
// term by term, each coefficient at the end of its range (the log of the c6 term
// at its largest magnitude, folded into r.c6 by the caller).  Every term
// falls with f, so the bound does.
__device__ __forceinline__ double node_rate(const RateBound &r, double u)
{
    const double v = 1.0 / u;
    double p = 5.0 * r.c0 * v * v + 3.0 * r.c2;
    p = p * v + 2.0 * r.c3;
    p = p * v + r.c4;
    p = p * v + r.c5l;
    p = p + u * (r.c6 + 2.0 * r.c7 * u);
    return r.tau + p * v * v * v * (1.0 / 3.0);
}

// The plan of a batch from the ranges of its phase coefficients, written to
// `p` (LDS).  All kBlock threads call it; `red` holds kPlanScratch doubles.
//
// Reference: the middle of a coefficient's range where the range keeps one sign
// and spans at most a factor 4, else 0.  Then no sample's difference from the
// reference is more than 1.5 times the coefficient itself, and one far-off row of
// a batch cannot cost the others their digits.
constexpr int kPlanSlices = kBlock / kStats;                       // 14 slices of the entries
constexpr int kPlanScratch = kPlanSlices * kStats + 2 * kStatPairs + kNodeSpacings;

__device__ __forceinline__ void make_node_plan(double f_low, double df, int64_t n_bins, int n_det,
                                               const double *__restrict__ stats, int n_stats, NodePlan &p,
                                               double *red)
{
    double *const half = red + kPlanSlices * kStats, *const mid = half + kStatPairs;
    double *const first = mid + kStatPairs;
    const int t = threadIdx.x;
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
        double m = 0.0, h = 0.0;
        if (lo <= hi) {
            const double a = fmin(fabs(lo), fabs(hi)), b = fmax(fabs(lo), fabs(hi));
            if ((lo > 0.0) == (hi > 0.0) && 4.0 * a >= b) m = 0.5 * lo + 0.5 * hi;
            h = fmax(fabs(lo - m), fabs(hi - m));
        }
        mid[t] = m;
        half[t] = h;
    }
    __syncthreads();
    RateBound r;
    r.tau = half[0];
    r.c7 = half[1];
    r.c6l = half[3];
    r.c5l = half[4];
    r.c4 = half[5];
    r.c3 = half[6];
    r.c2 = half[7];
    r.c0 = half[8];
    // |d/du of (c6 + c6l L) u| = |c6 + c6l (L + 1)|; nodes stand up to 16 cells past the band's ends
    const double f_high = f_low + (double)(n_bins - 1) * df;
    const double u_high = cbrt(f_high);
    const double f_past = f_high + 2.0 * kTaps * node_spacing(kNodeSpacings - 1) * df;
    r.c6 = half[2] + half[3] * (fmax(fabs(log(0.5 * f_low)), fabs(log(f_past))) * (1.0 / 3.0) + 1.0);
    // first bin of every spacing: 16 threads each search the lowest frequency
    // from which on the rate bound holds, 17-ary on u (the bound falls with u)
    const int g = t / 16, lane = t % 16;
    if (g < kNodeSpacings) {
        const int q = node_spacing(g);
        const double step = (double)q * df;
        const double f_min = fmax(f_low - 16.0 * step, 0.5 * f_low);
        double lo = cbrt(f_min), hi = u_high;
        const bool never = !(node_rate(r, hi) * step <= GW_RESAMPLE_BAND);
        if (node_rate(r, lo) * step <= GW_RESAMPLE_BAND) hi = lo;
        for (int it = 0; it < 7; ++it) {
            const double w = (hi - lo) * (1.0 / 17.0);
            const bool ok = node_rate(r, lo + w * (double)(lane + 1)) * step <= GW_RESAMPLE_BAND;
            const unsigned bits = (unsigned)(__ballot(!ok) >> (16 * (g % 4))) & 0xffffu;
            const int n_bad = __popc(bits);          // the bound falls with u: the low points fail first
            const double base = lo;
            lo = base + w * (double)n_bad;
            hi = n_bad == 16 ? hi : base + w * (double)(n_bad + 1);
        }
        if (lane == 0) {
            const double k = ceil((hi * hi * hi + 16.0 * step - f_low) / df);
            first[g] = never || !(k < (double)n_bins) ? (double)n_bins : fmax(k, 0.0);
        }
    }
    __syncthreads();
    if (t == 0) {
        int64_t k_first[kNodeSpacings];
        for (int i = 0; i < kNodeSpacings; ++i) k_first[i] = (int64_t)first[i];
        node_levels(k_first, n_bins, n_det, p);
        p.mid[kRecC8] = mid[0];
        p.mid[kRecC7] = mid[1];
        p.mid[kRecC6] = mid[2];
        p.mid[kRecC6L] = mid[3];
        p.mid[kRecC5] = 0.0;
        p.mid[kRecC5L] = mid[4];
        p.mid[kRecC4] = mid[5];
        p.mid[kRecC3] = mid[6];
        p.mid[kRecC2] = mid[7];
        p.mid[kRecC0] = mid[8];
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
// What bounds it: one division, one reference phasor and 64 n_det
// multiply-adds per bin, against 72 + 48 bytes read.
template <int NDET>
struct SpreadShape {
    static constexpr int kComp = 2 * NDET;
    static constexpr int kPack = node_pack(NDET);
    static constexpr int kStride = kSpreadBins + 4;          // LDS row of one component, in doubles
    static constexpr int kPacks = 8;                         // packs of cells per batch
    static constexpr int kMaxNodes = kSpreadBins / 8 + kTaps - 1;
    static constexpr int kAcc = (kMaxNodes * kComp + kBlock - 1) / kBlock;
    static constexpr size_t kLds = sizeof(double) * ((size_t)kComp * kStride + (size_t)kPacks * kTaps * 16);
};

template <int NDET>
__device__ __forceinline__ void spread_chunk(const NodeEvent &ev, const NodePlan &plan, int chunk, bool norm,
                                             double *lds_d, double *lds_y, double *red)
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

    double acc[kPrepPerDet * NDET];
#pragma unroll
    for (int i = 0; i < kPrepPerDet * NDET; ++i) acc[i] = 0.0;
    for (int b = t; b < kSpreadBins; b += kBlock) {
        const int cell = b / sub_bins, j = b - cell * sub_bins;
        const int64_t k = single ? k_base + b : k_base + (int64_t)cell * v.q + j;
        const bool live = b < n_here && k < k_end && (single || j0 + j < v.q);
        double er = 0.0, ei = 0.0, amp = 0.0;
        if (live) {
            gw_phasor_turns(turns_phase(ref, ev.tab1[k]), er, ei);
            amp = ev.tab2[k].amp;
        }
#pragma unroll
        for (int d = 0; d < NDET; ++d) {
            double dr = 0.0, di = 0.0;
            if (live) {
                const double s = ev.psd[(int64_t)d * n_bins + k];
                const double w = (s > 0.0 && s < INFINITY) ? 1.0 / s : NAN;
                const double2 x = ev.data[(int64_t)d * n_bins + k];
                const double scale = 4.0 * ev.df * amp * w;
                const double xr = scale * x.x, xi = -scale * x.y;
                dr = xr * er - xi * ei;
                di = xr * ei + xi * er;
                acc[kPrepPerDet * d] += (x.x * x.x + x.y * x.y) * w;
                acc[kPrepPerDet * d + 1] += amp * amp * w;
                if (norm) acc[kPrepPerDet * d + 2] += log(2.0 * GW_PI * s);
            }
            if (single) {
                if (live) ev.dcoef[(int64_t)d * n_bins + k] = make_double2(dr, di);
            } else {
                lds_d[(2 * d) * kStride + b] = dr;
                lds_d[(2 * d + 1) * kStride + b] = di;
            }
        }
    }
    if (!single && t < 4 * kComp) lds_d[(t / 4) * kStride + kSpreadBins + t % 4] = 0.0;
    // the chunk's share of the event sums: wave sums, then the waves in order
#pragma unroll
    for (int i = 0; i < kPrepPerDet * NDET; ++i) {
        const double s = wave_sum(acc[i]);
        if (lane == 0) red[wave * kPrepPerDet * NDET + i] = s;
    }
    __syncthreads();
    if (t < kPrepPerDet * NDET) {
        constexpr int n = kPrepPerDet * NDET;
        ev.prep[(int64_t)chunk * n + t] = ((red[t] + red[n + t]) + red[2 * n + t]) + red[3 * n + t];
    }
    if (single) {
        __syncthreads();
        return;
    }

    // weights: this lane's taps (both halves) and its place among 4 bins
    const int col = lane % 16, kk = lane / 16;
    double c0[GW_RESAMPLE_DEGREE + 1], c1[GW_RESAMPLE_DEGREE + 1];
#pragma unroll
    for (int j = 0; j <= GW_RESAMPLE_DEGREE; ++j) {
        c0[j] = resample_coef[j][col];
        c1[j] = resample_coef[j][16 + col];
    }
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
        const int kparts = packs == 1 ? 4 : packs < 4 ? 2 : 1;
        const int groups = 4 / kparts;               // waves per part
        const int part = wave / groups, pack0 = wave % groups;
        const int steps = (sub_bins + 3) / 4;
        const int s0 = steps * part / kparts, s1 = steps * (part + 1) / kparts;
        for (int pk = pack0; pk < packs; pk += 2 * groups) {
            // two packs at a time share the weights
            double4_t y00 = {0.0, 0.0, 0.0, 0.0}, y01 = y00, y10 = y00, y11 = y00;
            const int cell_a = cb + pk * kPack + cell_of_col, cell_b = cell_a + groups * kPack;
            const bool two = pk + groups < packs;
            const bool live_a = col_live && cell_a < v.cpc, live_b = col_live && two && cell_b < v.cpc;
            const double *da = lds_d + comp * kStride + (live_a ? cell_a * sub_bins : 0);
            const double *db = lds_d + comp * kStride + (live_b ? cell_b * sub_bins : 0);
            for (int s = s0; s < s1; ++s) {
                const int j = 4 * s + kk;
                const double x = (double)(j0 + j) * inv_q2 - 1.0;
                double w0 = c0[GW_RESAMPLE_DEGREE], w1 = c1[GW_RESAMPLE_DEGREE];
#pragma unroll
                for (int i = GW_RESAMPLE_DEGREE - 1; i >= 0; --i) {
                    w0 = __builtin_fma(w0, x, c0[i]);
                    w1 = __builtin_fma(w1, x, c1[i]);
                }
                if (j >= sub_bins) w0 = w1 = 0.0;
                const double a = live_a && j < sub_bins ? da[j] : 0.0;
                y00 = __builtin_amdgcn_mfma_f64_16x16x4f64(w0, a, y00, 0, 0, 0);
                y01 = __builtin_amdgcn_mfma_f64_16x16x4f64(w1, a, y01, 0, 0, 0);
                if (two) {
                    const double b = live_b && j < sub_bins ? db[j] : 0.0;
                    y10 = __builtin_amdgcn_mfma_f64_16x16x4f64(w0, b, y10, 0, 0, 0);
                    y11 = __builtin_amdgcn_mfma_f64_16x16x4f64(w1, b, y11, 0, 0, 0);
                }
            }
            // row kk + 4 r of a 16 x 16 result is in register r
            double *ya = lds_y + (part * packs + pk) * kTaps * 16 + col;
            double *yb = ya + groups * kTaps * 16;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                ya[(kk + 4 * r) * 16] = y00[r];
                ya[(16 + kk + 4 * r) * 16] = y01[r];
                if (two) {
                    yb[(kk + 4 * r) * 16] = y10[r];
                    yb[(16 + kk + 4 * r) * 16] = y11[r];
                }
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
template <int NDET>
__global__ __launch_bounds__(kBlock) void node_spread_kernel(NodeEvent ev, int norm)
{
    extern __shared__ double lds[];
    __shared__ NodePlan plan;
    __shared__ double red[kPlanScratch];
    make_node_plan(ev.f_low, ev.df, ev.n_bins, NDET, ev.stats, ev.n_stats, plan, red);
    if (blockIdx.x == 0) {
        const int *src = reinterpret_cast<const int *>(&plan);
        int *dst = reinterpret_cast<int *>(ev.plan);
        for (int i = threadIdx.x; i < (int)(sizeof(NodePlan) / sizeof(int)); i += kBlock) dst[i] = src[i];
    }
    double *const lds_y = lds + SpreadShape<NDET>::kComp * SpreadShape<NDET>::kStride;
    for (int c = blockIdx.x; c < plan.n_chunks; c += gridDim.x)
        spread_chunk<NDET>(ev, plan, c, norm != 0, lds, lds_y, red);
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
    {
        const int *src = reinterpret_cast<const int *>(ev.plan);
        int *dst = reinterpret_cast<int *>(&plan);
        for (int i = threadIdx.x; i < (int)(sizeof(NodePlan) / sizeof(int)); i += kBlock) dst[i] = src[i];
    }
    __syncthreads();
    const int n_sums = kPrepPerDet * ev.n_det;
    if ((int)blockIdx.x < n_sums) {
        const double s = column_total(plan.n_chunks, n_sums, blockIdx.x, ev.prep, red);
        if (threadIdx.x == 0) ev.sums[blockIdx.x] = s;
        if (queue && blockIdx.x == 0 && threadIdx.x < 2 * kQueues) queue[threadIdx.x] = 0u;
        return;
    }
    combine_items(ev, plan, (int64_t)(blockIdx.x - n_sums) * kBlock + threadIdx.x,
                  (int64_t)(gridDim.x - n_sums) * kBlock);
}

// ---------------------------------------------------------------- launchers
template <int NDET>
static hipError_t spread(const NodeEvent &ev, bool norm, int n_cu, hipStream_t stream)
{
    const int64_t blocks = std::min<int64_t>(node_max_chunks(ev.n_bins), (int64_t)n_cu * 2);
    hipLaunchKernelGGL(node_spread_kernel<NDET>, dim3((unsigned)blocks), dim3(kBlock), SpreadShape<NDET>::kLds, stream,
                       ev, norm ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_node_spread(const NodeEvent &ev, bool norm, int n_cu, hipStream_t stream)
{
    switch (ev.n_det) {
    case 1: return spread<1>(ev, norm, n_cu, stream);
    case 2: return spread<2>(ev, norm, n_cu, stream);
    case 3: return spread<3>(ev, norm, n_cu, stream);
    case 4: return spread<4>(ev, norm, n_cu, stream);
    case 5: return spread<5>(ev, norm, n_cu, stream);
    case 6: return spread<6>(ev, norm, n_cu, stream);
    case 7: return spread<7>(ev, norm, n_cu, stream);
    case 8: return spread<8>(ev, norm, n_cu, stream);
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
