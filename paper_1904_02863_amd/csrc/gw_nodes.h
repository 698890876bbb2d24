// Frequency nodes of the split-form likelihood: the geometry shared by the
// kernels that form them (gw_nodes.hip), the pass that sums over them
// (gw_kernels.hip) and the host code that lays out the workspace.
//
// The only sum over bins that depends on the sample is
//     Z_d = sum_k D_d,k e^{-2 pi i x_d(f_k)},
// x_d the template's phase at detector d in turns.  Neighbouring bins of one
// template are far from independent: its phase turns by its local time,
// |dx_d/df|, a fraction of a second over most of the band, against bins
// delta_f = 1/T apart.  So the phasor of a bin is interpolated from nodes q
// bins apart (32 weights of gw_resample_weights.h, for phases that turn by at
// most GW_RESAMPLE_BAND per node), the weights are applied to the data once for all
// samples,
//     nu_d,n = sum_k w_n(k) D_d,k,        Z_d = sum_n nu_d,n e^{-2 pi i x_d(f_n)},
// and the per-sample sum runs over the nodes: 1,656 instead of 259,585
// frequencies for 4096 heavy binaries in 128 s, 18,691 (14,704 of them single
// bins below 44 Hz) instead of 1,040,897 for neutron stars from 15 Hz in 512 s.
//
// A phasor of constant rate is interpolated to 4e-16.  A chirp's rate falls over a bin's 32
// nodes, and where its lowest node is at the limit the bin is off by more: in the
// lowest cell of a level by 4e-12 while the spacing is a hundredth of the frequency,
// by up to 2e-10 where it is as wide; five cells up by 1e-13 and less.  Averaged over a
// level that is 4e-12 at most.  What it does to lnL: 25 batches, from priors down to a
// millionth of their width, f_low from 3 to 20 Hz, were within 3e-16 of <d,d> of the sums over
// every bin, those from 3 Hz within 7e-15.
//
// Before the weights, D is multiplied by the phasor of a reference template
// (the middle of the batch's range in every phase coefficient), so what has to
// be resolved is only how the batch's templates differ from it.  R(f), a
// bound on that difference's |dx/df| over every sample and detector that
// falls with f (see node_rate), fixes the spacing: q bins from the first bin
// K(q) on at which every frequency that a bin's 32 nodes reach keeps
// R q delta_f <= GW_RESAMPLE_BAND.  Bins below every K(q) are summed one by one.
#pragma once

#include <cmath>
#include <cstdint>

#include <hip/hip_runtime.h>

#include "gw_internal.h"
#include "gw_resample_weights.h"

namespace gw {

constexpr int kTaps = GW_RESAMPLE_TAPS;              // nodes a bin is interpolated from
constexpr int kTapsBelow = GW_RESAMPLE_HALF - 1;     // of them below the bin's own cell
// Node spacings, in bins, about a factor 1.4 apart.  Each costs 31 nodes beyond its
// level's ends.  Spacings of 4 and 6 would serve more bins (neutron stars from 15 Hz in
// 512 s: 9,497 single bins and 5,156 nodes, against 14,704 and 3,987), but a level of
// them has no room in its part of D for its partials, nodes and tables (node_room_ok).
constexpr int kNodeSpacings = 15;
__host__ __device__ constexpr int node_spacing(int i)
{
    constexpr int q[kNodeSpacings] = {8, 12, 16, 24, 32, 48, 64, 96, 128, 192, 256, 384, 512, 768, 1024};
    return q[i];
}
// A level covers at least kNodeMinCells cells (a cell: the q bins between two
// nodes), so that its 31 extra nodes stay below what it saves over the next
// smaller spacing; the lowest level, which saves single bins, kNodeLowCells.
constexpr int kNodeMinCells = 64, kNodeLowCells = 40;
constexpr int kSpreadBins = 512;                     // bins a block weights at a time
// Phase coefficients whose range over the batch is taken: tau (its lowest and
// highest over the detectors), c7, c6, c6l, c5l, c4, c3, c2, c0; one
// (minimum, maximum) pair each.
constexpr int kStatPairs = 9;
constexpr int kStats = 2 * kStatPairs;
constexpr int kStatEntries = 256;                    // entries the plan is made from directly
constexpr int kMids = 10;                            // reference coefficients, in RecordField order

// One level: bins [k0, k1) with nodes q bins apart.  Node n of the level, n =
// 0 .. cells + 30, stands at bin k0 + (n - 15) q; cell c is interpolated from
// nodes c .. c + 31.  Chunks of the weighting: cpc cells each, every cell cut into
// `subs` parts of sub_bins bins.
struct NodeLevel {
    int64_t k0, k1;
    int q, cells, cpc, subs, sub_bins, n_chunks;
    int chunk0;       // first chunk, counted over the bins' chunks and all levels
    int node0;        // first node, counted over all levels
};

struct NodePlan {
    int64_t k_bin;                // bins [0, k_bin) are summed one by one
    int n_levels, n_nodes;        // nodes of all levels
    int bin_chunks, n_chunks;     // chunks of the weighting: of the bins, of everything
    double mid[kMids];            // reference coefficients
    NodeLevel level[kNodeSpacings];
};

__host__ __device__ inline int node_count(const NodeLevel &v) { return v.cells + kTaps - 1; }

// Cells that share the 16 columns of one matrix instruction (two columns per
// detector: real and imaginary part).
__host__ __device__ constexpr int node_pack(int n_det)
{
    return n_det <= 1 ? 8 : n_det == 2 ? 4 : n_det <= 4 ? 2 : 1;
}

__host__ __device__ inline void node_chunks(int n_det, NodeLevel &v)
{
    const int pack = node_pack(n_det);
    if (v.q * pack <= kSpreadBins) {
        v.cpc = kSpreadBins / v.q;
        v.subs = 1;
        v.sub_bins = v.q;
    } else {
        v.cpc = pack;
        v.subs = (v.q * pack + kSpreadBins - 1) / kSpreadBins;
        v.sub_bins = (v.q + v.subs - 1) / v.subs;
    }
    v.n_chunks = (v.cells + v.cpc - 1) / v.cpc * v.subs;
}

// A chunk of the weighting leaves cpc + 31 partial node values; they, the
// level's nodes and the nodes' tables stand in the level's own part of the D
// array, which holds nothing else: per detector, from bin k0 on, the chunks'
// partials, then the nodes, then (detector 0) two entries per node for Tab1.
// node_room_ok states that this fits: true for every level of at least
// kNodeLowCells cells.
__host__ __device__ inline int64_t node_slots(const NodeLevel &v)
{
    return (int64_t)v.n_chunks * (v.cpc + kTaps - 1);
}
__host__ __device__ inline bool node_room_ok(const NodeLevel &v)
{
    return node_slots(v) + 3 * (int64_t)node_count(v) <= v.k1 - v.k0;
}

// Half the batch's range of every phase coefficient about the reference, as
// what it adds to |dx/df| (see node_rate).
struct RateBound {
    double tau, c7, c6, c6l, c5l, c4, c3, c2, c0;
};

// Bound on |dx_d/df| (turns per Hz) of x_d less the reference's phase at
// frequency u^3, over every evaluated sample and detector: the derivative of
//   x = tau f + c7 u^2 + (c6 + c6l L) u + (c5 + c5l L) + c4/u + c3/u^2 + c2/u^3 + c0/u^5
// term by term, each coefficient at the end of its range (the log of the c6 term
// at its largest magnitude, folded into r.c6).  Every term falls with f, so the bound does.
__host__ __device__ inline double node_rate(const RateBound &r, double u)
{
    const double v = 1.0 / u;
    double p = 5.0 * r.c0 * v * v + 3.0 * r.c2;
    p = p * v + 2.0 * r.c3;
    p = p * v + r.c4;
    p = p * v + r.c5l;
    p = p + u * (r.c6 + 2.0 * r.c7 * u);
    return r.tau + p * v * v * v * (1.0 / 3.0);
}

// Reference of a coefficient that runs from lo to hi over the batch, and half its
// range about it: the middle where the range keeps one sign and spans at most a
// factor 4, else 0.  Then no sample's difference from the reference is more than
// 1.5 times the coefficient itself, and one far-off row of a batch cannot cost the
// others their digits.
__host__ __device__ inline void node_middle(double lo, double hi, double &mid, double &half)
{
    mid = half = 0.0;
    if (!(lo <= hi)) return;                     // no sample is evaluated
    const double a = fmin(fabs(lo), fabs(hi)), b = fmax(fabs(lo), fabs(hi));
    if ((lo > 0.0) == (hi > 0.0) && 4.0 * a >= b) mid = 0.5 * lo + 0.5 * hi;
    half = fmax(fabs(lo - mid), fabs(hi - mid));
}

// The band as the plan sees it: the bound is tried at kBlock frequencies from
// half of f_low up, even in u (about 1% apart in f), the last one the top of the
// band.  Nodes stand up to 16 cells past its ends.
struct NodeBand {
    double f_low, df, u_low, u_high, du;
    double l_most;        // the largest |ln u| + 1 at any node
    int64_t n_bins;
};

__host__ __device__ inline NodeBand node_band(double f_low, double df, int64_t n_bins)
{
    NodeBand b;
    const double f_high = f_low + (double)(n_bins - 1) * df;
    const double f_past = f_high + 2.0 * kTaps * node_spacing(kNodeSpacings - 1) * df;
    b.f_low = f_low;
    b.df = df;
    b.n_bins = n_bins;
    b.u_low = cbrt(0.5 * f_low);
    b.u_high = cbrt(f_high);
    b.du = (b.u_high - b.u_low) * (1.0 / (kBlock - 1));
    b.l_most = fmax(fabs(log(0.5 * f_low)), fabs(log(f_past))) * (1.0 / 3.0) + 1.0;
    return b;
}

__host__ __device__ inline double node_probe(const NodeBand &b, int t)
{
    return t == kBlock - 1 ? b.u_high : b.u_low + b.du * (double)t;
}

// half[j]: half the range of pair j (kStatPairs).
__host__ __device__ inline RateBound node_bound(const double *half, const NodeBand &b)
{
    RateBound r;
    r.tau = half[0];
    r.c7 = half[1];
    r.c6l = half[3];
    r.c5l = half[4];
    r.c4 = half[5];
    r.c3 = half[6];
    r.c2 = half[7];
    r.c0 = half[8];
    r.c6 = half[2] + half[3] * b.l_most;         // |d/du of (c6 + c6l L) u| = |c6 + c6l (L + 1)|
    return r;
}

// How many spacings a rate allows (spacings rise with their index).
__host__ __device__ inline int node_allowed(double rate, double df)
{
    int n = 0;
#pragma unroll
    for (int g = 0; g < kNodeSpacings; ++g) n += rate * ((double)node_spacing(g) * df) <= GW_RESAMPLE_BAND;
    return n;
}

// First bin of spacing g when `failing` of the kBlock probes, which are the lowest
// ones since the bound falls with f, do not allow it (n_bins: it cannot be used).
__host__ __device__ inline int node_first_bin(const NodeBand &b, int g, int failing)
{
    const double reach = (double)((kTapsBelow + 1) * node_spacing(g)) * b.df;   // a bin's nodes reach this far down
    const double u = node_probe(b, failing);
    const double k = ceil((fmax(u * u * u, b.f_low - reach) + reach - b.f_low) / b.df);
    return failing == kBlock || !(k < (double)b.n_bins) ? (int)b.n_bins : (int)fmax(k, 0.0);
}

// Levels for first bins k_first[i] of spacing node_spacing(i) (n_bins where a
// spacing cannot be used), from the widest down; what no level takes is left
// to single bins.  node_pick returns how many levels there are, where the
// single bins end, and of level number `want`, counted from the widest, and those below
// it their chunks and nodes together; it fills v with level `want` (so that the
// kernels can have one thread per level).
__host__ __device__ inline int node_pick(const int *k_first, int n_bins, int n_det, int want, NodeLevel &v, int &k_bin,
                                         int &chunks, int &nodes)
{
    int end = n_bins, n = 0, last = kNodeSpacings;
    chunks = nodes = 0;
    v.q = 0;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
        if (end == 0) break;
#pragma unroll
        for (int i = kNodeSpacings - 1; i >= 0; --i) {
            const int k = k_first[i], q = node_spacing(i);
            if (i < last && k < end && end - k >= (pass == 0 ? kNodeMinCells : kNodeLowCells) * q) {
                NodeLevel w;
                w.k0 = k;
                w.k1 = end;
                w.q = q;
                w.cells = (int)(((unsigned)(end - k) + (unsigned)q - 1u) / (unsigned)q);
                node_chunks(n_det, w);
                if (n >= want) {
                    chunks += w.n_chunks;
                    nodes += node_count(w);
                }
                if (n == want) v = w;
                ++n;
                end = k;
                last = i;
            }
        }
    }
    k_bin = end;
    v.chunk0 = (k_bin + kSpreadBins - 1) / kSpreadBins + chunks - (v.q > 0 ? v.n_chunks : 0);
    v.node0 = nodes - (v.q > 0 ? node_count(v) : 0);
    return n;
}

// A plan's counts, from `chunks` and `nodes` of all its levels (node_pick, want 0).
__host__ __device__ inline void node_totals(int n_levels, int k_bin, int chunks, int nodes, NodePlan &p)
{
    p.k_bin = k_bin;
    p.n_levels = n_levels;
    p.n_nodes = nodes;
    p.bin_chunks = (k_bin + kSpreadBins - 1) / kSpreadBins;
    p.n_chunks = p.bin_chunks + chunks;
}

// The plan's levels and counts one level at a time (the device has a thread per level).
inline void node_levels(const int *k_first, int n_bins, int n_det, NodePlan &p)
{
    NodeLevel v;
    int k_bin = 0, chunks = 0, nodes = 0;
    const int n = node_pick(k_first, n_bins, n_det, 0, v, k_bin, chunks, nodes);
    node_totals(n, k_bin, chunks, nodes, p);
    for (int l = 0; l < n; ++l) node_pick(k_first, n_bins, n_det, n - 1 - l, p.level[l], k_bin, chunks, nodes);
}

// Chunks of the weighting that any plan of n_bins bins can have: a chunk of a
// level holds at least 3/8 of kSpreadBins bins but for the level's last cells.
__host__ __device__ inline int64_t node_max_chunks(int64_t n_bins)
{
    return (n_bins + kSpreadBins * 3 / 8 - 1) / (kSpreadBins * 3 / 8) + 4 * kNodeSpacings + 1;
}

// Blocks of the weighting: one per chunk, up to three per CU (what fits at
// once); more chunks take turns.
inline int node_spread_blocks(int64_t n_bins, int n_cu)
{
    const int64_t c = node_max_chunks(n_bins), most = 3 * (int64_t)n_cu;
    return (int)(c < most ? c : most);
}

// The work split of the sum over `units` bins and nodes: the host's plan
// (n_chunks chunks in `rounds` rounds), or fewer rounds while they would be
// left with less than kUnitsRound units a chunk, and of one round fewer chunks
// below kUnitsChunk.
constexpr int kUnitsRound = 48, kUnitsChunk = 16;
__host__ __device__ inline void node_split(int64_t units, int n_chunks, int rounds, int &eff_chunks, int &eff_rounds)
{
    const int64_t per = rounds > 0 ? n_chunks / rounds : n_chunks;
    const int64_t r = rounds > 0 ? units / (per * kUnitsRound) : 0;
    eff_rounds = rounds > 0 ? (int)(r < 1 ? 1 : r > rounds ? rounds : r) : 0;
    eff_chunks = (int)per * (eff_rounds > 1 ? eff_rounds : 1);
    const int64_t most = (units + kUnitsChunk - 1) / kUnitsChunk;
    if (eff_rounds <= 1 && eff_chunks > most) eff_chunks = (int)(most < 1 ? 1 : most);
}

__host__ __device__ inline int node_chunks_of(int64_t units, int n_chunks, int rounds)
{
    int c, r;
    node_split(units, n_chunks, rounds, c, r);
    return units > 0 ? c : 0;
}

// One event as the node kernels see it.
struct NodeEvent {
    int64_t n_bins;
    int n_det;
    double f_low, df;
    const double2 *data;
    const double *psd;
    const Tab1 *tab1;
    const Tab2 *tab2;
    double2 *dcoef;       // [n_det][n_bins]: D of the single bins, and every level's partials and nodes
    double *prep;         // [spread_blocks][kPrepPerDet n_det] sums over each block's chunks
    int spread_blocks;    // blocks of the weighting
    double *sums;
    double *stats;        // [n_stats][kStats]
    int n_stats;
    NodePlan *plan;
};

// A call takes the nodes (how many, the batch decides) when its direct sum has
// at least this many (bin, group of 256 samples) pairs.  The nodes' kernels take 10 to 15 us
// more than the event preparation they replace: a small direct sum takes less than that,
// and a batch that turns out to need every bin pays them on top.  Both grow with the
// detectors as the direct sum does, so that FP64 calls of 1 to 8 share a line.
// Measured, us, direct / nodes of a batch near one point / of arrival times all over the segment:
//                      65,536 pairs         131,072               262,144
//   FP64   1 detector  33.1 / 35.6 / 46.0   47.8 / 34.3 / 61.1    80.5 / 32.8 / 94.8
//          3           43.3 / 47.8 / 54.4   68.6 / 42.5 / 79.8     121 / 40.3 /  130
//          8           76.1 / 77.3 / 92.4    131 / 67.2 /  145     241 / 63.3 /  261
//   mixed  1           28.5 / 39.2 / 40.9   39.7 / 44.5 / 53.4    64.1 / 36.7 / 74.9
//          3           40.2 / 51.5 / 55.5   60.9 / 53.4 / 74.5     105 / 46.2 /  117
//          8           68.2 / 87.6 / 84.5    116 / 77.1 /  131     212 / 70.2 /  239
// (16,384, 32,768 and 65,536 bins x 1024 rows.)  The line lies above the point where near
// batches begin to gain, where the others lose 20 to 30%; from four times there on
// they lose 4 to 14%, 3 detectors x 259,585 bins x 4096 rows 0.5%.  Longer segments leave fewer of
// their bins single: 65,536 bins x 1 group, 3 detectors, 49.9 / 41.2 / 64.1 and, mixed,
// 51.3 / 45.0 / 66.1, so that the mixed path takes the FP64 line there.
constexpr int64_t kNodeMinBins = 8192;
__host__ __device__ constexpr int64_t node_min_work(int64_t n_bins, int n_det, bool mixed)
{
    return mixed && n_bins < 65536 ? (n_det <= 2 ? 163840 : 122880) : 98304;
}

// Stats entries the sample kernel writes: one per block of 64 samples.
inline int64_t node_stat_entries(int64_t n_samples) { return (n_samples + 63) / 64; }

// A ragged call takes the nodes when its events together have that much work (each in
// its own measure) and one of them is that long.  64 neutron-star events of 8 to 256 s, 512 rows each: 8.50 ms summing
// every bin, 0.91 ms on nodes (0.37 of it the weighting, 0.46 the sums).
// Its events are cut into items of at least kRaggedUnits bins and nodes each,
// kRaggedItems items per resident block where there is that much work: an item
// costs a block about 5 us beside its sums, and fewer leave the last ones uneven (2, 3,
// 4, 8, 16 items a block: 485, 461, 462, 483, 526 us).  No item is longer than kRaggedMost,
// so that a call whose events are summed bin by bin ends evenly: the same events with
// arrival times all over their segments take 8.83, 8.86, 8.96, 9.28 and 10.1 ms with a limit of
// 512, 1024, 2048, 4096 and none, 16 of them 2.45, 2.42, 2.57, 2.70 and 2.71 ms (before there
// were nodes, 8.6 and 2.55 ms).
constexpr int kRaggedUnits = 64, kRaggedItems = 4, kRaggedMost = 1024;
// Bins and nodes of an item of `work` of them (times sample groups) on `grid` blocks.
__host__ __device__ inline int64_t ragged_item_units(double work, int grid)
{
    const double even = work / ((double)kRaggedItems * (double)grid);
    return even < (double)kRaggedUnits ? kRaggedUnits : even > (double)kRaggedMost ? kRaggedMost : (int64_t)even + 1;
}
// Blocks of the weighting of one event of a ragged call (about four chunks each),
// and of the node sums (the first takes the event sums; with a quarter of the others
// they took 64 us instead of 45).
inline int ragged_spread_blocks(int64_t n_bins) { return (int)((n_bins + 4 * kSpreadBins - 1) / (4 * kSpreadBins)); }
inline int ragged_combine_blocks(int64_t n_bins)
{
    const int64_t b = (n_bins + 2047) / 2048;
    return 1 + (int)(b < 256 ? b : 256);
}
// The most chunks an event of a ragged call of n_groups sample groups is cut
// into (the chunks' partial sums take 64 MB or less over the call).
inline int ragged_max_chunks(int64_t n_bins, int64_t n_groups, bool mixed)
{
    const int64_t share = 32768 / n_groups + 1, most = (n_bins + kRaggedUnits - 1) / kRaggedUnits;
    const int64_t c = share < most ? share : most;
    return (int)(mixed && c < 2 ? 2 : c);
}

// ---- launchers (gw_nodes.hip, gw_kernels.hip) ----
// Ragged calls: plans, weighting (per detector count) and node sums.
hipError_t launch_ragged_plans(const RaggedLaunch &r, hipStream_t stream);
hipError_t launch_ragged_spread(const RaggedLaunch &r, hipStream_t stream);
hipError_t launch_ragged_combine(const RaggedLaunch &r, hipStream_t stream);
// Sample records and the range of their phase coefficients, one entry of
// `stats` per 64 samples (reduced to kStatEntries when there are more).
hipError_t launch_node_samples(const gw_grid &grid, int n_det, const SamplePrep &sp, double *stats,
                               hipStream_t stream);
// Plan, D, event sums' partials, and every level's weighted partial nodes.
hipError_t launch_node_spread(const NodeEvent &ev, bool norm, hipStream_t stream);
// Nodes from their partials, the nodes' tables, the event sums; zeroes the queue.
hipError_t launch_node_combine(const NodeEvent &ev, unsigned *queue, hipStream_t stream);

}  // namespace gw
