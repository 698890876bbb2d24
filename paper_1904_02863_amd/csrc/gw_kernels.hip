// HIP kernels of the batched TaylorF2 likelihood for gfx950 (MI355X).
//
// The likelihood is Eq. (cbclike) of arXiv:1904.02863 (Sec. III).  With the
// noise-weighted inner product <a, b> = 4 df sum a* b / S its exponent splits
// exactly (an algebraic identity, not an approximation) into
//     lnL = -1/2 <d,d> + sum_det [ Re <d, h_det> - 1/2 <h_det, h_det> ].
// For the TaylorF2 template h_det,k = P_det a_k e^{-i Phi_det,k} with
// a_k = f_k^-7/6 and a per-(sample, detector) complex amplitude P_det, so
//     <h_det, h_det> = |P_det|^2 Q_det,         Q_det = 4 df sum_k a_k^2 / S_det,k
//     <d, h_det>     = P_det Z_det,             Z_det = sum_k D_det,k e^{-i Phi_det,k}
//     D_det,k = 4 df a_k conj(d_det,k) / S_det,k.
// Only Z needs a pass over (sample, bin, detector); <d,d>, Q and D are built
// once per event.  The per-detector phases differ by the time translation
// exp(-2 pi i f dt_det) described after Eq. (cbclike):
//     Phi_det,k = Phi_0,k + 2 pi f_k delta_det,  delta_det = dt_det - dt_0,
// so e^{-i Phi_0} is evaluated once per (sample, bin) with the polynomial
// phasor of gw_device_math.h.  For the other detectors the rotation
// e^{-2 pi i f_k delta} = R_last rho^(k - k_last), rho = e^{-2 pi i df delta},
// is applied by Horner's rule over the bins of a tile,
//     S <- S conj(rho) + D_k e^{-i Phi_0,k},   Z += R_last S at the tile end,
// with R_last evaluated exactly once per tile.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "gw_build_id.h"
#include "gw_device_math.h"
#include "gw_internal.h"
#include "gw_nodes.h"
#include "gw_plan.h"
#include "gw_reduce.h"
#include "gw_template.h"

// Tuning of the tile kernel's inner loop: bins per unrolled step (FP64 and
// mixed paths), and the number of waves per SIMD the register allocation
// must leave room for.  The FP64 kernels run two blocks per CU (their LDS
// holds the phasor table), so 8 bins per step fit their registers; the mixed
// kernels run three, and 4 bins keep them within 168 VGPRs.
#ifndef GW_TILE_UNROLL
#define GW_TILE_UNROLL 8
#endif
#ifndef GW_TILE_UNROLL_MIXED
#define GW_TILE_UNROLL_MIXED 4
#endif
#ifndef GW_TILE_WAVES_PER_EU
#define GW_TILE_WAVES_PER_EU 0
#endif
// 1: the FP64 tile loops take e^{-i Phi} from the LDS table (gw_phasor_table);
// 0: from the polynomial phasor (gw_phasor_turns).
#ifndef GW_PHASOR_TABLE
#define GW_PHASOR_TABLE 1
#endif
#if GW_TILE_WAVES_PER_EU > 0
#define GW_TILE_ATTR __attribute__((amdgpu_waves_per_eu(GW_TILE_WAVES_PER_EU)))
#else
#define GW_TILE_ATTR
#endif

namespace gw {

constexpr int kTileUnroll = GW_TILE_UNROLL, kTileUnrollMixed = GW_TILE_UNROLL_MIXED;

// ---------------------------------------------------------------- event tables
__device__ __forceinline__ void bin_tables(double f_low, double df, int64_t k, Tab1 *tab1, Tab2 *tab2)
{
    freq_tables(bin_frequency(f_low, df, k), tab1[k], tab2[k]);
}

// One event's device arrays as the preparation kernels see them.
struct PrepView {
    int64_t n_bins;
    int n_det;
    double df;
    const double2 *data;
    const double *psd;
    const Tab2 *tab2;
    double2 *dcoef;
    double2 *edir;
    double *vdir;
};

// Bin k of every detector: D = 4 df a conj(d) / S (split form) and, for the
// direct form, d / a and a^2 / S; adds |d|^2/S, a^2/S and (with `norm`)
// ln(2 pi S) to acc[3 d + 0, 1, 2].  A PSD value that is not positive and
// finite makes its weight NaN, which turns <d,d> and hence every lnL of the
// event into NaN.
__device__ __forceinline__ void bin_data(const PrepView &v, int64_t k, bool direct, bool norm,
                                         double acc[kPrepPerDet * kMaxDet])
{
    const double amp = v.tab2[k].amp;
#pragma unroll
    for (int d = 0; d < kMaxDet; ++d) {
        if (d < v.n_det) {
            const double s = v.psd[(int64_t)d * v.n_bins + k];
            const double w = (s > 0.0 && s < INFINITY) ? 1.0 / s : NAN;
            const double2 x = v.data[(int64_t)d * v.n_bins + k];
            const double scale = 4.0 * v.df * amp * w;
            v.dcoef[(int64_t)d * v.n_bins + k] = make_double2(scale * x.x, -scale * x.y);
            if (direct) {
                v.edir[(int64_t)d * v.n_bins + k] = make_double2(x.x / amp, x.y / amp);
                v.vdir[(int64_t)d * v.n_bins + k] = amp * amp * w;
            }
            acc[kPrepPerDet * d] = (x.x * x.x + x.y * x.y) * w;
            acc[kPrepPerDet * d + 1] = amp * amp * w;
            acc[kPrepPerDet * d + 2] = norm ? log(2.0 * GW_PI * s) : 0.0;
        }
    }
}

// Block b of an event's preparation: bins [256 b, 256 b + 256); writes the
// block's sums out[kPrepPerDet d + j] (wave sums, then the 4 waves in order).
// `red` holds at least 4 kPrepPerDet kMaxDet doubles of LDS.
__device__ __forceinline__ void prep_block(const PrepView &v, int64_t b, bool direct, bool norm, double *red,
                                           double *__restrict__ out)
{
    constexpr int kQ = kPrepPerDet * kMaxDet;
    double acc[kQ];
#pragma unroll
    for (int i = 0; i < kQ; ++i) acc[i] = 0.0;
    const int64_t k = b * kBlock + threadIdx.x;
    if (k < v.n_bins) bin_data(v, k, direct, norm, acc);
    const int nq = kPrepPerDet * v.n_det, lane = threadIdx.x % 64, wave = threadIdx.x / 64;
#pragma unroll
    for (int j = 0; j < kQ; ++j) {
        if (j < nq) {
            const double t = wave_sum(acc[j]);
            if (lane == 0) red[wave * kQ + j] = t;
        }
    }
    __syncthreads();
    if ((int)threadIdx.x < nq)
        out[threadIdx.x] = ((red[threadIdx.x] + red[kQ + threadIdx.x]) + red[2 * kQ + threadIdx.x]) +
                           red[3 * kQ + threadIdx.x];
    __syncthreads();
}

// Inclusive Hillis-Steele scan of x over the block (fixed order); `red` is
// kBlock doubles of LDS.  All threads must call it.
__device__ __forceinline__ double block_scan(double x, double *red)
{
    red[threadIdx.x] = x;
    __syncthreads();
    for (int off = 1; off < kBlock; off <<= 1) {
        const double add = (int)threadIdx.x >= off ? red[threadIdx.x - off] : 0.0;
        __syncthreads();
        red[threadIdx.x] += add;
        __syncthreads();
    }
    const double total = red[threadIdx.x];
    __syncthreads();
    return total;
}

// offsets[b] = sum over blocks b' < b of column j of an event's per-block
// partials, for every b < n_blocks (one block: each thread scans a
// contiguous segment of blocks on top of the preceding segments' totals).
__device__ __forceinline__ void block_offsets(int64_t n_blocks, int per, int j, const double *__restrict__ partials,
                                              double *red, double *__restrict__ offsets)
{
    const int64_t seg = (n_blocks + kBlock - 1) / kBlock;
    const int64_t b0 = (int64_t)threadIdx.x * seg, b1 = min(n_blocks, b0 + seg);
    double mine = 0.0;
    for (int64_t b = b0; b < b1; ++b) mine += partials[b * per + j];
    double run = block_scan(mine, red) - mine;      // exclusive: the preceding segments
    for (int64_t b = b0; b < b1; ++b) {
        offsets[b] = run;
        run += partials[b * per + j];
    }
}

// Prefix sums of a^2/S for the ISCO end: block b of the event writes
// qprefix[d][k] = sum_{j <= k} a_j^2 / S_d,j for its 256 bins, from the
// preceding blocks' total qoffsets[d][b] and a scan of its own bins.
__device__ __forceinline__ void prefix_block(const PrepView &v, int64_t b, int64_t n_blocks,
                                             const double *__restrict__ qoffsets, double *red,
                                             double *__restrict__ qprefix)
{
    const int64_t k = b * kBlock + threadIdx.x;
    const double amp = k < v.n_bins ? v.tab2[k].amp : 0.0;
    for (int d = 0; d < v.n_det; ++d) {
        const double offset = qoffsets[(int64_t)d * n_blocks + b];
        double q = 0.0;
        if (k < v.n_bins) {
            const double s = v.psd[(int64_t)d * v.n_bins + k];
            const double w = (s > 0.0 && s < INFINITY) ? 1.0 / s : NAN;
            q = amp * amp * w;
        }
        const double incl = block_scan(q, red);
        if (k < v.n_bins) qprefix[(int64_t)d * v.n_bins + k] = offset + incl;
    }
}

__global__ __launch_bounds__(kBlock) void event_tables_kernel(double f_low, double df, int64_t n_bins,
                                                               Tab1 *__restrict__ tab1, Tab2 *__restrict__ tab2)
{
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x; k < n_bins; k += stride)
        bin_tables(f_low, df, k, tab1, tab2);
}

// Block j: sums[j] = the event-wide sum of quantity j (kPrepPerDet n_det blocks).
// Also zeroes the tile kernel's work-queue counters when there are any.
__global__ __launch_bounds__(kBlock) void event_sums_kernel(int n_blocks, int n_det,
                                                             const double *__restrict__ partials,
                                                             double *__restrict__ sums, unsigned *__restrict__ queue)
{
    __shared__ double red[kBlock];
    const double t = column_total(n_blocks, kPrepPerDet * n_det, blockIdx.x, partials, red);
    if (threadIdx.x == 0) sums[blockIdx.x] = t;
    if (queue && blockIdx.x == 0 && threadIdx.x < kQueues) queue[threadIdx.x] = 0u;
}

// Block d: qoffsets[d][b], the a^2/S total of the blocks before b.
__global__ __launch_bounds__(kBlock) void event_offsets_kernel(int64_t n_blocks, int n_det,
                                                                const double *__restrict__ partials,
                                                                double *__restrict__ qoffsets)
{
    __shared__ double red[kBlock];
    const int d = blockIdx.x;
    block_offsets(n_blocks, kPrepPerDet * n_det, kPrepPerDet * d + 1, partials, red, qoffsets + (int64_t)d * n_blocks);
}

__global__ __launch_bounds__(kBlock) void event_prefix_kernel(PrepView v, int64_t n_blocks,
                                                               const double *__restrict__ qoffsets,
                                                               double *__restrict__ qprefix)
{
    __shared__ double red[kBlock];
    prefix_block(v, blockIdx.x, n_blocks, qoffsets, red, qprefix);
}

__device__ __forceinline__ PrepView prep_view(const RaggedEvent &re)
{
    PrepView v;
    v.n_bins = re.n_bins;
    v.n_det = re.n_det;
    v.df = re.df;
    v.data = re.data;
    v.psd = re.psd;
    v.tab2 = re.tab2;
    v.dcoef = re.dcoef;
    v.edir = re.edir;
    v.vdir = re.vdir;
    return v;
}

// Bin tables of all events of a ragged batch, blocks as in ragged_event_prep_kernel.
__global__ __launch_bounds__(kBlock) void ragged_tables_kernel(const RaggedEvent *__restrict__ events,
                                                               const int2 *__restrict__ block_map)
{
    const int2 em = block_map[blockIdx.x];
    const RaggedEvent &re = events[em.x];
    const int64_t k = (int64_t)em.y * kBlock + threadIdx.x;
    if (k < re.n_bins) bin_tables(re.f_low, re.df, k, re.tab1, re.tab2);
}

// Ragged batch, all events at once: block b handles bins
// [256 local, 256 local + 256) of event e, (e, local) = block_map[b].
__global__ __launch_bounds__(kBlock) void ragged_event_prep_kernel(const RaggedEvent *__restrict__ events,
                                                                    const int2 *__restrict__ block_map,
                                                                    int direct, int norm)
{
    __shared__ double red[kBlock];
    const int2 em = block_map[blockIdx.x];
    const RaggedEvent &re = events[em.x];
    prep_block(prep_view(re), em.y, direct != 0, norm != 0, red,
               re.prep + (int64_t)em.y * kPrepPerDet * re.n_det);
}

// Ragged batch: block e sums event e's per-block partials.
__global__ __launch_bounds__(kBlock) void ragged_event_sums_kernel(const RaggedEvent *__restrict__ events)
{
    __shared__ double red[kBlock];
    const RaggedEvent &re = events[blockIdx.x];
    for (int j = 0; j < kPrepPerDet * re.n_det; ++j) {
        const double t = column_total(re.prep_blocks, kPrepPerDet * re.n_det, j, re.prep, red);
        if (threadIdx.x == 0) re.sums[j] = t;
    }
}

// Ragged batch: block e computes event e's qoffsets for every detector.
__global__ __launch_bounds__(kBlock) void ragged_offsets_kernel(const RaggedEvent *__restrict__ events)
{
    __shared__ double red[kBlock];
    const RaggedEvent &re = events[blockIdx.x];
    for (int d = 0; d < re.n_det; ++d)
        block_offsets(re.prep_blocks, kPrepPerDet * re.n_det, kPrepPerDet * d + 1, re.prep, red,
                      re.qoffsets + (int64_t)d * re.prep_blocks);
}

// Ragged batch: prefix sums of a^2/S, blocks as in ragged_event_prep_kernel.
__global__ __launch_bounds__(kBlock) void ragged_prefix_kernel(const RaggedEvent *__restrict__ events,
                                                                const int2 *__restrict__ block_map)
{
    __shared__ double red[kBlock];
    const int2 em = block_map[blockIdx.x];
    const RaggedEvent &re = events[em.x];
    prefix_block(prep_view(re), em.y, re.prep_blocks, re.qoffsets, red, re.qprefix);
}

// ---------------------------------------------------------------- per-sample preparation
// Row s: mass ratios, the phase polynomial coefficients (in turns), antenna
// patterns F = D : e, delays -n.r/c, and the complex amplitudes
//   P_det = A0 [F+ (1 + cos^2 iota)/2 - i Fx cos iota] e^{i (phi_c + pi/4)}.
// In polarisation mode (n_out == 2, no detectors) channel 0 is h_plus and
// channel 1 is h_cross.  The template's last bin K_s is n_bins - 1, or with
// the ISCO end the last bin with f_k <= f_isco = 1 / (6^(3/2) pi M) (-1 when
// there is none, and for samples that are not evaluated).
//
// A block takes kSampleRows samples, one per lane, and its four waves a part of the work
// each: (0) status, masses and phase coefficients, (1) sky position and
// polarisation, (2) amplitude, (3) phi_c and inclination; then each wave writes some of
// the channels.  A sample is one long chain of dependent FP64 functions and
// there are few samples, so the chain's latency is the kernel's time: the
// parts side by side take about half of what one lane takes for all of them
// (4096 samples: 11.1 us -> 6.2 us).
constexpr int kSampleRows = 64;

struct SampleShare {
    double fp[kMaxDet][kSampleRows], fx[kMaxDet][kSampleRows], dt[kMaxDet][kSampleRows];
    double amp[kSampleRows], rot_re[kSampleRows], rot_im[kSampleRows], plus[kSampleRows], cross[kSampleRows];
};

// 0: evaluate, 1: out of domain (-inf), 2: non-finite (NaN).
__device__ __forceinline__ int sample_status(const double *t, int n_param)
{
    int status = 0;
#pragma unroll
    for (int i = 0; i < kMaxParam; ++i)
        if (i < n_param && !isfinite(t[i])) status = 2;
    if (status == 0 && (!(t[0] > 0.0) || !(t[1] > 0.0 && t[1] <= 1.0) || !(t[2] > 0.0))) status = 1;
    if (status == 0 && param_has_spins(n_param)) {
        const double chi1 = n_param == 7 ? t[5] : t[9], chi2 = n_param == 7 ? t[6] : t[10];
        if (fabs(chi1) > 1.0 || fabs(chi2) > 1.0) status = 1;
    }
    return status;
}

// Phase coefficients cj u^(j-5) and cjl u^(j-5) ln u in turns, and the total
// mass in seconds.
__device__ __forceinline__ void sample_phase(const double *t, int n_param, double cj[8], double cjl[8], double &mtot_s)
{
    const bool spins = param_has_spins(n_param);
    const double chi1 = !spins ? 0.0 : n_param == 7 ? t[5] : t[9], chi2 = !spins ? 0.0 : n_param == 7 ? t[6] : t[10];
    const double mc = t[0], q = t[1];
    const double eta = q / ((1.0 + q) * (1.0 + q));
    mtot_s = mc * pow(eta, -0.6) * GW_MSUN_S;
    const double alpha = cbrt(GW_PI * mtot_s);          // v = alpha u
    const double ln_alpha = log(alpha);
    double phi[8], phil[8];
    gw_pn_coefficients(eta, phi, phil);
    if (spins) gw_pn_spin_terms(1.0 / (1.0 + q), q / (1.0 + q), chi1, chi2, phi, phil);
    const double pref = 3.0 / (128.0 * eta) / GW_TWO_PI;   // phase in turns
    double apow[8];
    const double a2 = alpha * alpha;
    apow[5] = 1.0;
    apow[6] = alpha;
    apow[7] = a2;
    apow[0] = 1.0 / (a2 * a2 * alpha);
    apow[1] = apow[0] * alpha;
    apow[2] = apow[1] * alpha;
    apow[3] = apow[2] * alpha;
    apow[4] = apow[3] * alpha;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        cj[j] = pref * apow[j] * (phi[j] + phil[j] * ln_alpha);
        cjl[j] = pref * apow[j] * phil[j];
    }
}

// Antenna patterns and delays of detectors d < n_out of lane `at` into sh.
__device__ __forceinline__ void sample_sky(double ra, double dec, double psi, int n_out, const DetGeom &geom, int at,
                                           SampleShare &sh)
{
    double cra, sra, cde, sde, cps, sps;
    sincos(ra, &sra, &cra);
    sincos(dec, &sde, &cde);
    sincos(psi, &sps, &cps);
    const double n[3] = {cde * cra, cde * sra, sde};
    const double ea[3] = {-sra, cra, 0.0};
    const double ed[3] = {-sde * cra, -sde * sra, cde};
    double x[3], y[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        x[i] = cps * ea[i] + sps * ed[i];
        y[i] = -sps * ea[i] + cps * ed[i];
    }
    for (int d = 0; d < n_out; ++d) {
        double p = 0.0, c = 0.0;
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const double dij = geom.tensor[d][3 * i + j];
                p += dij * (x[i] * x[j] - y[i] * y[j]);
                c += dij * (x[i] * y[j] + y[i] * x[j]);
            }
        sh.fp[d][at] = p;
        sh.fx[d][at] = c;
        sh.dt[d][at] = -(n[0] * geom.vertex[d][0] + n[1] * geom.vertex[d][1] + n[2] * geom.vertex[d][2]) / GW_C_SI;
    }
}

// K_s of a template that ends at the ISCO of total mass mtot_s.
__device__ __forceinline__ double isco_bin(double f_low, double df, int64_t n_bins, double mtot_s)
{
    const double f_isco = 1.0 / (pow(6.0, 1.5) * GW_PI * mtot_s);
    const double kf = fmin(fmax(floor((f_isco - f_low) / df), -1.0), (double)(n_bins - 1));
    int64_t k = (int64_t)kf;
    // settle the rounding: the same f_k = f_low + k df as every table
    while (k + 1 < n_bins && __dadd_rn(f_low, __dmul_rn((double)(k + 1), df)) <= f_isco) ++k;
    while (k >= 0 && __dadd_rn(f_low, __dmul_rn((double)k, df)) > f_isco) --k;
    return (double)k;
}

// The range of the batch's phase coefficients over the block's samples
// (kStatPairs of gw_nodes.h): entry[2 j], entry[2 j + 1] the smallest and largest
// of pair j, +inf and -inf when none of the samples is evaluated.
__device__ __forceinline__ void write_range(const double (&lo)[kStatPairs], double tau_hi, bool ok,
                                            double *__restrict__ entry)
{
#pragma unroll
    for (int j = 0; j < kStatPairs; ++j) {
        const double a = wave_min(ok ? lo[j] : INFINITY);
        const double b = wave_max(ok ? (j == 0 ? tau_hi : lo[j]) : -INFINITY);
        if (threadIdx.x == 0) {
            entry[2 * j] = a;
            entry[2 * j + 1] = b;
        }
    }
}

// Samples s0 .. s0 + kSampleRows - 1 (below n_samples) by a block of kBlock
// threads, all of which call it; with `entry`, their range too.
__device__ __forceinline__ void prep_samples(double f_low, double df, int64_t n_bins, int64_t s0, int64_t n_samples,
                                             int n_param, int n_out, bool polarisations, bool isco,
                                             const DetGeom &geom, const double *__restrict__ theta,
                                             double *__restrict__ rec, SampleShare &sh, double *__restrict__ entry)
{
    const int lane = threadIdx.x % kSampleRows, wave = threadIdx.x / kSampleRows;
    const bool live = s0 + lane < n_samples;
    const int64_t s = live ? s0 + lane : n_samples - 1, ns = n_samples;
    const double *__restrict__ row = theta + s * n_param;
    const bool sky = param_has_sky(n_param);
    double lo[kStatPairs], tc = 0.0;
    bool ok = false;
    if (wave == 0) {
        double t[kMaxParam];
#pragma unroll
        for (int i = 0; i < kMaxParam; ++i) t[i] = i < n_param ? row[i] : 0.0;
        const int status = sample_status(t, n_param);
        double cj[8], cjl[8], mtot_s;
        sample_phase(t, n_param, cj, cjl, mtot_s);
        tc = t[4];
        ok = live && status == 0;
        const double v[kStatPairs] = {0.0, cj[7], cj[6], cjl[6], cjl[5], cj[4], cj[3], cj[2], cj[0]};
#pragma unroll
        for (int j = 0; j < kStatPairs; ++j) lo[j] = v[j];
        if (live) {
            rec[kRecC7 * ns + s] = cj[7];
            rec[kRecC6 * ns + s] = cj[6];
            rec[kRecC6L * ns + s] = cjl[6];
            rec[kRecC5 * ns + s] = cj[5];
            rec[kRecC5L * ns + s] = cjl[5];
            rec[kRecC4 * ns + s] = cj[4];
            rec[kRecC3 * ns + s] = cj[3];
            rec[kRecC2 * ns + s] = cj[2];
            rec[kRecC0 * ns + s] = cj[0];
            rec[kRecStatus * ns + s] = (double)status;
            double kcut = (double)(n_bins - 1);
            if (isco) kcut = status == 0 ? isco_bin(f_low, df, n_bins, mtot_s) : -1.0;
            rec[kRecKcut * ns + s] = kcut;
        }
    } else if (wave == 1) {
        if (sky && !polarisations) {
            sample_sky(row[5], row[6], row[7], n_out, geom, lane, sh);
        } else {
            for (int d = 0; d < n_out; ++d) {
                sh.fp[d][lane] = 1.0;
                sh.fx[d][lane] = 0.0;
                sh.dt[d][lane] = 0.0;
            }
        }
    } else if (wave == 2) {
        sh.amp[lane] = sqrt(5.0 / 24.0) * pow(GW_PI, -2.0 / 3.0) * pow(row[0] * GW_MSUN_S, 5.0 / 6.0) /
                       (row[2] * GW_MPC_S);
    } else {
        double re, im;
        sincos(row[3] + 0.25 * GW_PI, &im, &re);
        sh.rot_re[lane] = re;
        sh.rot_im[lane] = im;
        const double ci = sky ? cos(row[8]) : 1.0;
        sh.plus[lane] = 0.5 * (1.0 + ci * ci);
        sh.cross[lane] = ci;
    }
    __syncthreads();
    if (live) {
        if (wave == 0) rec[kRecC8 * ns + s] = tc + sh.dt[0][lane];     // 2 pi f tau0 in turns: tau0 u^3
        const double amp0 = sh.amp[lane], plus = sh.plus[lane], ci = sh.cross[lane];
        const double rot_re = sh.rot_re[lane], rot_im = sh.rot_im[lane];
        for (int d = wave; d < n_out; d += kBlock / kSampleRows) {
            double pre, pim;   // P before the e^{i(phi_c + pi/4)} rotation
            if (polarisations) {
                pre = d == 0 ? amp0 * plus : 0.0;
                pim = d == 0 ? 0.0 : -amp0 * ci;
            } else {
                pre = amp0 * sh.fp[d][lane] * plus;
                pim = -amp0 * sh.fx[d][lane] * ci;
            }
            rec[(kRecDet + kRecFieldsPerDet * d) * ns + s] = pre * rot_re - pim * rot_im;
            rec[(kRecDet + kRecFieldsPerDet * d + 1) * ns + s] = pre * rot_im + pim * rot_re;
            rec[(kRecDet + kRecFieldsPerDet * d + 2) * ns + s] = sh.dt[d][lane] - sh.dt[0][lane];
        }
    }
    if (entry && wave == 0) {
        double first = sh.dt[0][lane], last = first;
        for (int d = 1; d < n_out; ++d) {
            first = fmin(first, sh.dt[d][lane]);
            last = fmax(last, sh.dt[d][lane]);
        }
        lo[0] = tc + first;
        write_range(lo, tc + last, ok, entry);
    }
}

__global__ __launch_bounds__(kBlock) void sample_prep_kernel(double f_low, double df, int64_t n_bins,
                                                              int64_t n_samples, int n_param, int n_out,
                                                              int polarisations, int isco, DetGeom geom,
                                                              const double *__restrict__ theta,
                                                              double *__restrict__ rec)
{
    __shared__ SampleShare sh;
    prep_samples(f_low, df, n_bins, (int64_t)blockIdx.x * kSampleRows, n_samples, n_param, n_out, polarisations != 0,
                 isco != 0, geom, theta, rec, sh, nullptr);
}

// One block per 256 consecutive bins, after sample_blocks blocks of kSampleRows
// samples each (sample records, when sample_blocks > 0).  The two parts share
// no data, so one launch runs them side by side; the sample blocks come
// first, since each of their threads has the longer serial work.
__global__ __launch_bounds__(kBlock) void event_data_kernel(PrepView v, int direct, int norm,
                                                             double *__restrict__ partials, int sample_blocks,
                                                             double f_low, SamplePrep sp)
{
    __shared__ union {
        SampleShare sample;
        double red[kBlock];
    } sh;
    if ((int)blockIdx.x < sample_blocks) {
        prep_samples(f_low, v.df, v.n_bins, (int64_t)blockIdx.x * kSampleRows, sp.n_samples, sp.n_param, v.n_det, false,
                     sp.isco != 0, sp.geom, sp.theta, sp.records, sh.sample, nullptr);
        return;
    }
    const int64_t b = (int64_t)blockIdx.x - sample_blocks;
    prep_block(v, b, direct != 0, norm != 0, sh.red, partials + b * kPrepPerDet * v.n_det);
}

// Sample records and their ranges, an entry of `stats` per block.
__global__ __launch_bounds__(kBlock) void node_samples_kernel(double f_low, double df, int64_t n_bins, int n_det,
                                                               SamplePrep sp, double *__restrict__ stats)
{
    __shared__ SampleShare sh;
    prep_samples(f_low, df, n_bins, (int64_t)blockIdx.x * kSampleRows, sp.n_samples, sp.n_param, n_det, false, false,
                 sp.geom, sp.theta, sp.records, sh, stats + (int64_t)blockIdx.x * kStats);
}

// Block j: out[j] = the smallest (j even) or largest (j odd) of column j over
// n entries.
__global__ __launch_bounds__(kBlock) void node_range_kernel(int64_t n, const double *__restrict__ stats,
                                                             double *__restrict__ out)
{
    __shared__ double red[kBlock];
    const int j = blockIdx.x;
    const bool low = j % 2 == 0;
    double m = low ? INFINITY : -INFINITY;
    for (int64_t e = threadIdx.x; e < n; e += kBlock) {
        const double v = stats[e * kStats + j];
        m = low ? fmin(m, v) : fmax(m, v);
    }
    red[threadIdx.x] = m;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            red[threadIdx.x] = low ? fmin(red[threadIdx.x], red[threadIdx.x + w])
                                   : fmax(red[threadIdx.x], red[threadIdx.x + w]);
        __syncthreads();
    }
    if (threadIdx.x == 0) out[j] = red[0];
}

// *k_limit = 1 + the largest K_s of the batch (one block).
__global__ __launch_bounds__(kBlock) void isco_limit_kernel(int64_t n_samples, const double *__restrict__ rec,
                                                             int64_t *__restrict__ k_limit)
{
    __shared__ double red[kBlock];
    double m = -1.0;
    for (int64_t s = threadIdx.x; s < n_samples; s += kBlock) m = fmax(m, rec[kRecKcut * n_samples + s]);
    red[threadIdx.x] = m;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + w]);
        __syncthreads();
    }
    if (threadIdx.x == 0) *k_limit = (int64_t)red[0] + 1;
}

// Ragged batch: blocks 4 i .. 4 i + 3 prepare the rows of group i (of 256).
__global__ __launch_bounds__(kBlock) void ragged_sample_prep_kernel(const RaggedEvent *__restrict__ events,
                                                                     const int2 *__restrict__ groups,
                                                                     const DetGeom *__restrict__ geoms, int n_param,
                                                                     int isco)
{
    __shared__ SampleShare sh;
    constexpr int kParts = kBlock / kSampleRows;
    const int2 eg = groups[blockIdx.x / kParts];
    const RaggedEvent &re = events[eg.x];
    const int64_t s0 = (int64_t)eg.y * kBlock + (int64_t)(blockIdx.x % kParts) * kSampleRows;
    if (s0 >= re.n_samples) return;
    prep_samples(re.f_low, re.df, re.n_bins, s0, re.n_samples, n_param, re.n_det, false, isco != 0, geoms[eg.x],
                 re.theta, re.rec, sh, re.stats ? re.stats + s0 / kSampleRows * kStats : nullptr);
}

// Sets n counters to zero (a kernel rather than a memset, so that it can be
// captured in a graph).
__global__ void zero_counters_kernel(unsigned *__restrict__ p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// ---------------------------------------------------------------- the hot loop
// One event seen by the tile loop.
struct EventView {
    int64_t n_bins, n_samples;
    double f_low, df;
    const Tab1 *tab1;
    const double2 *dcoef;      // split forms: D [n_det][n_bins]
    const double2 *edir;       // direct form: d / a [n_det][n_bins]
    const double *vdir;        // direct form: a^2 / S [n_det][n_bins]
    const double *rec;
    const int64_t *k_limit;    // split form with the ISCO end: 1 + max K_s (device)
    double2 *partials;         // double [chunk][n_samples]: sum_det Re(P_det Z_det) (split), residual sum (direct)
    const NodePlan *plan;      // node kernels: the batch's plan (device), else null
};

// LDS layout of a tile: tab1 [tile], then per detector D (split) or d/a
// (direct) [NDET][tile] double2, then for the direct form a^2/S [NDET][tile].
// LDS of one tile block: the phasor table (FP64 path) and the tiles.
__host__ __device__ constexpr size_t phasor_table_lds(bool mixed)
{
    return (GW_PHASOR_TABLE && !mixed) ? (size_t)GW_PHTAB_N * sizeof(double2) : 0;
}
__host__ __device__ constexpr size_t tile_lds_bytes(int n_det, int tile_bins, int form, bool mixed)
{
    return phasor_table_lds(mixed) +
           (size_t)tile_bins * (sizeof(Tab1) + (size_t)n_det * sizeof(double2) +
                                (form == kFormDirect ? (size_t)n_det * sizeof(double) : 0));
}

// Copies the phasor table into the head of the block's LDS (FP64 path) and
// returns where the tiles begin.  The tile loop's first barrier publishes it.
template <bool MIXED>
__device__ __forceinline__ double *stage_phasor_table(double4 *lds_raw)
{
    if constexpr (GW_PHASOR_TABLE && !MIXED) {
        double2 *tab = reinterpret_cast<double2 *>(lds_raw);
        gw_stage_phasor_table(tab, kBlock);
        return reinterpret_cast<double *>(tab + GW_PHTAB_N);
    }
    return reinterpret_cast<double *>(lds_raw);
}

// The bins (or nodes) 0 .. nk - 1 of one staged tile against this thread's
// sample: the split forms' Z_0 and Horner sums S_d, or the direct form's residual
// sum with its running T_d.  MIXED takes the phasor from the FP32 hardware
// sine and cosine; otherwise it comes from the LDS table, cf scaled for it.
// Bins past jcut carry no template (the forms that end templates).
template <int NDET, bool MIXED, int FORM>
__device__ __forceinline__ void tile_loop(const PhaseCoef &cf, const double2 *ptab, const Tab1 *lt, const double2 *ld,
                                          const double *lv, int tile_bins, int nk, int jcut,
                                          const double (&rho_re)[NDET], const double (&rho_im)[NDET],
                                          double (&sr_)[NDET], double (&si_)[NDET], double &z0r, double &z0i,
                                          double &acc)
{
    constexpr bool kDirect = FORM == kFormDirect;
    constexpr bool kMasked = FORM != kFormSplit;
#pragma unroll(MIXED ? kTileUnrollMixed : kTileUnroll)
    for (int j = 0; j < nk; ++j) {
        const Tab1 tb = lt[j];
        double er, ei;
        if constexpr (MIXED) {
            // FP64 phase and exact reduction to a fractional turn, then the
            // hardware sine and cosine (inputs in turns) in FP32
            const double x = turns_phase(cf, tb);
            const float r = (float)(x - __builtin_rint(x));
            er = (double)__builtin_amdgcn_cosf(r);
            ei = -(double)__builtin_amdgcn_sinf(r);
        } else {
#if GW_PHASOR_TABLE
            gw_phasor_table(turns_phase(cf, tb), ptab, er, ei);
#else
            gw_phasor_turns(turns_phase(cf, tb), er, ei);
#endif
        }
        if (kMasked && j > jcut) {
            er = 0.0;
            ei = 0.0;
        }
        if constexpr (kDirect) {
#pragma unroll
            for (int d = 0; d < NDET; ++d) {
                const double2 e = ld[d * tile_bins + j];
                const double v = lv[d * tile_bins + j];
                // residual d/a - P_d e^{-i Phi_d}
                double rr = __builtin_fma(-er, sr_[d], e.x);
                rr = __builtin_fma(ei, si_[d], rr);
                double ri = __builtin_fma(-er, si_[d], e.y);
                ri = __builtin_fma(-ei, sr_[d], ri);
                acc = __builtin_fma(v, __builtin_fma(rr, rr, ri * ri), acc);
                if (d > 0) {
                    const double tr = sr_[d] * rho_re[d] - si_[d] * rho_im[d];
                    si_[d] = sr_[d] * rho_im[d] + si_[d] * rho_re[d];
                    sr_[d] = tr;
                }
            }
        } else {
            const double2 d0 = ld[j];
            z0r = __builtin_fma(d0.x, er, z0r);
            z0r = __builtin_fma(-d0.y, ei, z0r);
            z0i = __builtin_fma(d0.x, ei, z0i);
            z0i = __builtin_fma(d0.y, er, z0i);
#pragma unroll
            for (int d = 1; d < NDET; ++d) {
                const double2 dv = ld[d * tile_bins + j];
                double tr = dv.x * er;
                tr = __builtin_fma(-dv.y, ei, tr);
                tr = __builtin_fma(sr_[d], rho_re[d], tr);
                tr = __builtin_fma(si_[d], rho_im[d], tr);
                double ti = dv.x * ei;
                ti = __builtin_fma(dv.y, er, ti);
                ti = __builtin_fma(si_[d], rho_re[d], ti);
                ti = __builtin_fma(-sr_[d], rho_im[d], ti);
                sr_[d] = tr;
                si_[d] = ti;
            }
        }
    }
}

// What a tile kernel sums: every bin; the plan's single bins and nodes; or one of
// these (the mixed path runs them as two launches, since its FP32 phasors serve
// the bins, where three blocks a CU without the table run best, and the
// nodes, few and each standing for many bins, take FP64 phasors).
enum NodeMode : int { kNoNodes = 0, kBinsAndNodes, kNodeBins, kNodesOnly };

// A run of evenly spaced frequencies f(i) = f_low + (k0 + i step) df, i in
// [begin, end): the bins themselves (k0 = 0, step = 1), or the nodes of a level.
struct FreqRun {
    const Tab1 *tab1;         // indexed by i
    const double2 *src;       // detector d's values at src + d n_bins, indexed by i
    int64_t k0, begin, end;
    int step;
};

// The 256 samples of `group` (one per thread) against bins [k_begin, k_end)
// of one event, staged through LDS tile by tile and shared by all the
// block's samples; writes the chunk's partial sums of every sample.
// MIXED selects the mixed-precision path: the phase polynomial and its
// reduction to a fractional turn stay FP64 (the phase reaches ~1e4 rad), the
// phasor e^{-i Phi_0} comes from the FP32 hardware sine/cosine, and the
// projection, accumulation and all sums stay FP64.
// FORM (TileForm): the split forms accumulate Z_det (kFormSplitIsco only
// over bins k <= K_s of each sample); the direct form accumulates
// sum_det a^2/S |d/a - P_det e^{-i Phi_det}|^2 with the template zero above K_s.
// NODES (split form, NodeMode): the bins and then nodes [n_begin, n_end) of the
// batch's plan, run by run over its levels, or one of the two, all with the
// coefficients less the plan's reference.  With kNodesOnly the chunk's totals
// below n_add are already those of a kNodeBins pass, and this adds to them.
// All threads of the block must call this with the same arguments.
template <int NDET, bool MIXED, int FORM, int NODES>
__device__ __forceinline__ void tile_chunk(const EventView &ev, int group, int64_t chunk, int64_t k_begin,
                                           int64_t k_end, int64_t n_begin, int64_t n_end, int n_add, int tile_bins,
                                           double *lds)
{
    static_assert(NODES == kNoNodes || FORM == kFormSplit, "nodes serve the split form only");
    static_assert(!MIXED || NODES == kNoNodes || NODES == kNodeBins, "the nodes take FP64 phasors");
    // the phasor table sits just below the tiles (FP64 path; the mixed path has none)
    const double2 *ptab =
        (GW_PHASOR_TABLE && !MIXED) ? reinterpret_cast<const double2 *>(lds) - GW_PHTAB_N : nullptr;
    constexpr bool kDirect = FORM == kFormDirect;
    constexpr bool kMasked = FORM != kFormSplit;
    const int64_t n_bins = ev.n_bins, n_samples = ev.n_samples;
    const double f_low = ev.f_low, df = ev.df;
    const double *__restrict__ vdir = ev.vdir;
    const double *__restrict__ rec = ev.rec;
    const int64_t s = (int64_t)group * kBlock + threadIdx.x;
    const int64_t sr = s < n_samples ? s : n_samples - 1;
    Tab1 *lt = reinterpret_cast<Tab1 *>(lds);
    double2 *ld = reinterpret_cast<double2 *>(lt + tile_bins);
    double *lv = reinterpret_cast<double *>(ld + NDET * tile_bins);

    PhaseCoef cf = load_coef(rec, n_samples, sr);
    if constexpr (NODES != kNoNodes) cf = coef_less(cf, load_coef(ev.plan->mid, 1, 0));
#if GW_PHASOR_TABLE
    // the table phasor takes the phase in units of 1/N turn (exact: N is a power of two)
    if constexpr (!MIXED) cf = scale_coef(cf, (double)GW_PHTAB_N);
#endif
    const int64_t kcut = kMasked ? (int64_t)rec[kRecKcut * n_samples + sr] : n_bins - 1;
    double rho_re[NDET], rho_im[NDET], delta[NDET], p_re[NDET], p_im[NDET];
#pragma unroll
    for (int d = 0; d < NDET; ++d) {
        if (kDirect) {
            p_re[d] = rec[(kRecDet + kRecFieldsPerDet * d) * n_samples + sr];
            p_im[d] = rec[(kRecDet + kRecFieldsPerDet * d + 1) * n_samples + sr];
        }
        if (d == 0) continue;
        delta[d] = rec[(kRecDet + kRecFieldsPerDet * d + 2) * n_samples + sr];
    }
    double zr[NDET], zi[NDET];
#pragma unroll
    for (int d = 0; d < NDET; ++d) { zr[d] = 0.0; zi[d] = 0.0; }
    double acc = 0.0;

    const int n_runs = NODES == kBinsAndNodes || NODES == kNodesOnly ? 1 + ev.plan->n_levels : 1;
    for (int run = NODES == kNodesOnly ? 1 : 0; run < n_runs; ++run) {
        FreqRun fr{ev.tab1, kDirect ? ev.edir : ev.dcoef, 0, k_begin, k_end, 1};
        if constexpr (NODES != kNoNodes) {
            if (run > 0) {
                const NodeLevel &v = ev.plan->level[run - 1];
                const int64_t nodes = v.k0 + node_slots(v);      // where the level's nodes stand in D
                fr.src = ev.dcoef + nodes;
                fr.tab1 = reinterpret_cast<const Tab1 *>(ev.dcoef + nodes + node_count(v));
                fr.k0 = v.k0 - (int64_t)kTapsBelow * v.q;
                fr.step = v.q;
                fr.begin = max(n_begin - v.node0, (int64_t)0);
                fr.end = min(n_end - v.node0, (int64_t)node_count(v));
            }
        }
        if (fr.begin >= fr.end) continue;
#pragma unroll
        for (int d = 1; d < NDET; ++d) gw_phasor_turns((double)fr.step * df * delta[d], rho_re[d], rho_im[d]);
        for (int64_t t0 = fr.begin; t0 < fr.end; t0 += tile_bins) {
            const int nk = (int)min((int64_t)tile_bins, fr.end - t0);
            __syncthreads();
            for (int i = threadIdx.x; i < nk; i += kBlock) {
                lt[i] = fr.tab1[t0 + i];
#pragma unroll
                for (int d = 0; d < NDET; ++d) {
                    ld[d * tile_bins + i] = fr.src[(int64_t)d * n_bins + t0 + i];
                    if (kDirect) lv[d * tile_bins + i] = vdir[(int64_t)d * n_bins + t0 + i];
                }
            }
            __syncthreads();
            // last live bin of this lane within the tile (template end)
            const int jcut = kMasked ? (int)max((int64_t)-1, min(kcut - t0, (int64_t)nk - 1)) : nk - 1;
            // split: Horner sums S_d over the tile; direct: T_d = P_d e^{-2 pi i f delta_d} at the current bin
            double sr_[NDET], si_[NDET];
#pragma unroll
            for (int d = 0; d < NDET; ++d) { sr_[d] = 0.0; si_[d] = 0.0; }
            if (kDirect) {
                const double f_first = bin_frequency(f_low, df, t0);
#pragma unroll
                for (int d = 0; d < NDET; ++d) {
                    if (d == 0) {
                        sr_[0] = p_re[0];
                        si_[0] = p_im[0];
                        continue;
                    }
                    double rr, ri;
                    gw_phasor_turns(f_first * delta[d], rr, ri);
                    sr_[d] = p_re[d] * rr - p_im[d] * ri;
                    si_[d] = p_re[d] * ri + p_im[d] * rr;
                }
            }
            tile_loop<NDET, MIXED, FORM>(cf, ptab, lt, ld, lv, tile_bins, nk, jcut, rho_re, rho_im, sr_, si_, zr[0],
                                         zi[0], acc);
            if (!kDirect && NDET > 1) {
                const double f_last = bin_frequency(f_low, df, fr.k0 + (t0 + nk - 1) * fr.step);
#pragma unroll
                for (int d = 1; d < NDET; ++d) {
                    double rr, ri;
                    gw_phasor_turns(f_last * delta[d], rr, ri);
                    zr[d] = __builtin_fma(rr, sr_[d], zr[d]);
                    zr[d] = __builtin_fma(-ri, si_[d], zr[d]);
                    zi[d] = __builtin_fma(rr, si_[d], zi[d]);
                    zi[d] = __builtin_fma(ri, sr_[d], zi[d]);
                }
            }
        }
    }
    if (s < n_samples) {
        if (!kDirect) {
            // the chunk's share of sum_det Re(P_det Z_det), linear in Z
            acc = 0.0;
#pragma unroll
            for (int d = 0; d < NDET; ++d) {
                const double pr = rec[(kRecDet + kRecFieldsPerDet * d) * n_samples + s];
                const double pi = rec[(kRecDet + kRecFieldsPerDet * d + 1) * n_samples + s];
                acc = __builtin_fma(pr, zr[d], acc);
                acc = __builtin_fma(-pi, zi[d], acc);
            }
        }
        double *out = reinterpret_cast<double *>(ev.partials) + chunk * n_samples + s;
        if (NODES == kNodesOnly && chunk < n_add) acc += *out;
        *out = acc;
    }
}

// One event.  queue == null: one block per work item (chunk, group), the grid
// being about one wave of resident blocks; blocks are dispatched round-robin
// over the 8 XCDs, and when the grid is a multiple of 8 the linear work index
// is remapped so that the blocks of one XCD cover consecutive chunks.
// queue != null: a persistent grid over kQueues work queues (counters zero
// at launch), so that blocks the wave arbiter favours, or CUs that clock
// higher, take more items and every SIMD keeps its waves until the end.
// Queue x holds the chunks c = x (mod kQueues) in index order, all sample
// groups of a chunk together; block b starts on queue b mod kQueues, which
// under round-robin dispatch is the queue of its own XCD, so a chunk's bins
// are fetched into one L2, and when its queue is empty takes items from the
// others in turn.  With the ISCO end (split form) the chunks cover only the
// bins below 1 + max K_s, read from the device, so that no block works on
// bins every template has left.
// NODES: bins below the plan's k_bin, then the nodes; a chunk takes the same
// share of both, and the plan made on the device sets how many of the host's
// chunks and rounds the batch needs.
// Node kernels: at least two waves per SIMD (a SIMD with one issues FP64 at half rate).
template <int NDET, bool MIXED, int FORM, int NODES>
__global__ __launch_bounds__(kBlock, NODES != kNoNodes ? 2 : 1) GW_TILE_ATTR
void lnl_tile_kernel(EventView ev, int n_groups, int n_chunks, int rounds, int tile_bins, unsigned *__restrict__ queue)
{
    extern __shared__ double4 lds_raw[];
    __shared__ int next_chunk, next_group;
    int64_t n_eff = FORM == kFormSplitIsco ? min(ev.n_bins, max((int64_t)0, *ev.k_limit)) : ev.n_bins;
    int64_t n_nodes = 0;
    int n_add = 0;
    if constexpr (NODES != kNoNodes) {
        n_eff = NODES == kNodesOnly ? 0 : ev.plan->k_bin;
        n_nodes = NODES == kNodeBins ? 0 : ev.plan->n_nodes;
        if (NODES != kBinsAndNodes && n_eff + n_nodes == 0) return;
        if (NODES == kNodesOnly) n_add = node_chunks_of(ev.plan->k_bin, n_chunks, rounds);
        node_split(n_eff + n_nodes, n_chunks, rounds, n_chunks, rounds);
    }
    // Items: without a queue one per block, (group, chunk) in chunk runs per XCD; on nodes,
    // when every queue's items fit the blocks that start on it, item b / 8 of
    // queue b mod 8, without its counter (the counters cost a launch of one
    // item per block about 10 us); else from the queues.
    const unsigned nb = gridDim.x, b = blockIdx.x, home = b % kQueues;
    const bool fixed = queue == nullptr ||
                       (NODES != kNoNodes && (unsigned)(n_groups * ((n_chunks + kQueues - 1) / kQueues)) <= nb / kQueues);
    int chunk = -1, group = 0;
    if (fixed) {
        if (queue == nullptr) {
            const unsigned w = (nb % 8u == 0u) ? (b % 8u) * (nb / 8u) + b / 8u : b;
            chunk = (int)(w / (unsigned)n_groups);
            group = (int)(w % (unsigned)n_groups);
            if (chunk >= n_chunks) return;
        } else if (!queue_item((int)home, (int)(b / kQueues), n_groups, n_chunks, chunk, group)) {
            return;
        }
    }
    double *const tiles = stage_phasor_table<MIXED>(lds_raw);
    bool home_empty = false;             // wave 0: the block's own queue has run out
    for (;;) {
        if (!fixed) {
            __syncthreads();             // every thread has read the item and left the LDS tiles
            if (threadIdx.x < 64) {
                int c = -1, g = 0;
                for (;;) {
                    int x = (int)home;
                    if (home_empty) {
                        // the counters of all queues at once; the nearest one with items left
                        const int l = threadIdx.x % kQueues;
                        int cl, gl;
                        const unsigned taken = __hip_atomic_load(queue + l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        const unsigned left =
                            (unsigned)__ballot(queue_item(l, (int)taken, n_groups, n_chunks, cl, gl)) & 0xffu;
                        if (left == 0u) break;
                        x = (int)((home + (unsigned)(__ffs((left | left << 8) >> home) - 1)) % kQueues);
                    }
                    int k = 0;
                    if (threadIdx.x == 0) k = (int)atomicAdd(queue + x, 1u);
                    k = __shfl(k, 0, 64);
                    if (queue_item(x, k, n_groups, n_chunks, c, g)) break;
                    c = -1;
                    home_empty = true;
                }
                if (threadIdx.x == 0) {
                    next_chunk = c;
                    next_group = g;
                }
            }
            __syncthreads();
            chunk = next_chunk;
            group = next_group;
            if (chunk < 0) break;
        }
        int64_t k_begin, k_end, n_begin = 0, n_end = 0;
        chunk_range(n_eff, chunk, n_chunks, rounds, k_begin, k_end);
        if constexpr (NODES != kNoNodes) chunk_range(n_nodes, chunk, n_chunks, rounds, n_begin, n_end);
        tile_chunk<NDET, MIXED, FORM, NODES>(ev, group, chunk, k_begin, k_end, n_begin, n_end, n_add, tile_bins, tiles);
        if (fixed) break;
    }
}

// Many events: a persistent grid.  Every block repeatedly takes the next work
// item (event, sample group, bin chunk) from a device counter until the list
// is exhausted; the list is sorted by decreasing cost, so the large items go
// first and the small ones fill the tail.  The counter must be zero at launch.
template <int NDET, bool MIXED, int FORM>
__global__ __launch_bounds__(kBlock) GW_TILE_ATTR void lnl_ragged_kernel(const RaggedEvent *__restrict__ events,
                                                                         const WorkItem *__restrict__ items,
                                                                         int n_items, unsigned *__restrict__ counter,
                                                                         int tile_bins)
{
    extern __shared__ double4 lds_raw[];
    __shared__ int next;
    double *const tiles = stage_phasor_table<MIXED>(lds_raw);
    for (;;) {
        __syncthreads();                 // every thread has read `next` and left the LDS
        if (threadIdx.x == 0) next = (int)atomicAdd(counter, 1u);
        __syncthreads();
        const int it = next;
        if (it >= n_items) break;
        const WorkItem wi = items[it];
        const RaggedEvent &re = events[wi.event];
        EventView ev;
        ev.n_bins = re.n_bins;
        ev.n_samples = re.n_samples;
        ev.f_low = re.f_low;
        ev.df = re.df;
        ev.tab1 = re.tab1;
        ev.dcoef = re.dcoef;
        ev.edir = re.edir;
        ev.vdir = re.vdir;
        ev.rec = re.rec;
        ev.k_limit = nullptr;
        ev.partials = re.partials;
        ev.plan = nullptr;
        const int64_t k_begin = (int64_t)wi.chunk * re.chunk_bins;
        const int64_t k_end = min(re.n_bins, k_begin + re.chunk_bins);
        tile_chunk<NDET, MIXED, FORM, kNoNodes>(ev, wi.group, wi.chunk, k_begin, k_end, 0, 0, 0, tile_bins, tiles);
    }
}

// Sample groups of an event.
__device__ __forceinline__ int64_t groups_of(const RaggedEvent &re) { return (re.n_samples + kBlock - 1) / kBlock; }

// Bins and nodes that a pass of a ragged call sums for every sample: FP64 one
// pass over both; mixed precision the bins (0), then the nodes (1).
__device__ __forceinline__ int64_t pass_units(const RaggedEvent &re, bool mixed, int pass)
{
    const NodePlan &p = *re.plan;
    return mixed ? (pass == 0 ? p.k_bin : (int64_t)p.n_nodes) : p.k_bin + p.n_nodes;
}

// One block: the items of one detector count's events.  An event's units are known only now, and
// differ by far more than its bins do (a short event keeps its bins, a long one
// is nearly all nodes), so the items' size is set here: about kRaggedItems
// items per resident block (ragged_item_units).  Writes every event's
// chunks (split), the first item of each (first, [2][n + 1]) and zero counters.
__global__ __launch_bounds__(kBlock) void ragged_split_kernel(const RaggedEvent *__restrict__ events,
                                                              const int *__restrict__ members, int n, int mixed,
                                                              int2 grids, unsigned *__restrict__ first,
                                                              unsigned *__restrict__ counter)
{
    __shared__ double red[kBlock];
    const int per = (n + kBlock - 1) / kBlock;
    const int i0 = min(n, (int)threadIdx.x * per), i1 = min(n, i0 + per);
    if (threadIdx.x < 2) counter[threadIdx.x] = 0u;
    for (int pass = 0; pass < (mixed ? 2 : 1); ++pass) {
        double work = 0.0;
        for (int i = i0; i < i1; ++i) {
            const RaggedEvent &re = events[members[i]];
            work += (double)(pass_units(re, mixed != 0, pass) * groups_of(re));
        }
        work = block_sum(work, red);
        const int grid = pass == 0 ? grids.x : grids.y;
        const int64_t size = ragged_item_units(work, grid);
        double items = 0.0;
        for (int i = i0; i < i1; ++i) {
            const RaggedEvent &re = events[members[i]];
            const int64_t most = mixed ? re.n_chunks / 2 : re.n_chunks;
            const int64_t c = min(most, (pass_units(re, mixed != 0, pass) + size - 1) / size);
            re.split[pass] = (int)c;
            if (!mixed) re.split[1] = 0;
            items += (double)(c * groups_of(re));
        }
        const double upto = block_scan(items, red);
        double at = upto - items;
        unsigned *const f = first + (int64_t)pass * (n + 1);
        for (int i = i0; i < i1; ++i) {
            const RaggedEvent &re = events[members[i]];
            f[i] = (unsigned)at;
            at += (double)((int64_t)re.split[pass] * groups_of(re));
        }
        if (threadIdx.x == kBlock - 1) f[n] = (unsigned)upto;
    }
}

// The persistent kernel of a ragged call on frequency nodes: item k of pass `pass`
// belongs to the event i with first[i] <= k < first[i + 1], chunk by chunk, the
// chunk's sample groups together; a chunk takes the same share of the event's
// bins and nodes.
template <int NDET, bool MIXED, int NODES>
__global__ __launch_bounds__(kBlock, 2) GW_TILE_ATTR
void ragged_node_kernel(const RaggedEvent *__restrict__ events, const int *__restrict__ members, int n,
                        const unsigned *__restrict__ first, unsigned *__restrict__ counter, int tile_bins)
{
    constexpr int kPass = NODES == kNodesOnly ? 1 : 0;
    extern __shared__ double4 lds_raw[];
    __shared__ int next_event, next_item;
    double *const tiles = stage_phasor_table<MIXED>(lds_raw);
    first += (int64_t)kPass * (n + 1);
    const unsigned n_items = first[n];
    for (;;) {
        __syncthreads();                 // every thread has read the item and left the LDS tiles
        if (threadIdx.x < 64) {
            unsigned k = 0;
            if (threadIdx.x == 0) k = atomicAdd(counter + kPass, 1u);
            k = (unsigned)__shfl((int)k, 0, 64);
            int lo = -1;
            if (k < n_items) {
                // the last event whose first item is not past k, 64 candidates at a time
                lo = 0;
                for (int span = n; span > 1;) {
                    const int step = (span + 63) / 64, off = (int)threadIdx.x * step;
                    const int m = __popcll(__ballot(off < span && first[lo + min(off, span - 1)] <= k)) - 1;
                    lo += m * step;
                    span = min(step, span - m * step);
                }
            }
            if (threadIdx.x == 0) {
                next_event = lo < 0 ? -1 : members[lo];
                next_item = lo < 0 ? 0 : (int)(k - first[lo]);
            }
        }
        __syncthreads();
        if (next_event < 0) break;
        const RaggedEvent &re = events[next_event];
        const int groups = (int)groups_of(re);
        const int chunk = next_item / groups, group = next_item % groups;
        EventView ev;
        ev.n_bins = re.n_bins;
        ev.n_samples = re.n_samples;
        ev.f_low = re.f_low;
        ev.df = re.df;
        ev.tab1 = re.tab1;
        ev.dcoef = re.dcoef;
        ev.edir = nullptr;
        ev.vdir = nullptr;
        ev.rec = re.rec;
        ev.k_limit = nullptr;
        ev.partials = re.partials;
        ev.plan = re.plan;
        const int n_chunks = re.split[kPass];
        int64_t k_begin = 0, k_end = 0, n_begin = 0, n_end = 0;
        if constexpr (NODES != kNodesOnly) chunk_range(re.plan->k_bin, chunk, n_chunks, 0, k_begin, k_end);
        if constexpr (NODES != kNodeBins) chunk_range(re.plan->n_nodes, chunk, n_chunks, 0, n_begin, n_end);
        tile_chunk<NDET, MIXED, kFormSplit, NODES>(ev, group, (kPass ? re.split[0] : 0) + chunk, k_begin, k_end, n_begin,
                                                   n_end, 0, tile_bins, tiles);
    }
}

// lnL of row s from its chunk totals: split forms -1/2 <d,d> + sum_det
// [Re(P Z_det) - 1/2 |P|^2 Q_det], Q_det from the event sums or, with the
// ISCO end, 4 df times the prefix sum of a^2/S up to K_s; direct form -2 df
// times the residual sum.  GW_FLAG_ADD_NORM subtracts sum ln(2 pi S).
// sums: the event-wide totals of |d|^2/S, a^2/S, ln(2 pi S) per detector.
__device__ __forceinline__ double assemble_row(int64_t s, int64_t n_samples, int n_det, int64_t n_bins, double df,
                                               unsigned flags, double total, const double *__restrict__ rec,
                                               const double *__restrict__ sums, const double *__restrict__ qprefix)
{
    double dd = 0.0, norm = 0.0;
    for (int d = 0; d < n_det; ++d) {
        dd += sums[kPrepPerDet * d];
        norm += sums[kPrepPerDet * d + 2];
    }
    dd *= 4.0 * df;
    double out;
    if (flags & GW_FLAG_DIRECT) {
        out = -2.0 * df * total;
    } else {
        const bool isco = (flags & GW_FLAG_TERM_ISCO) != 0;
        const int64_t kcut = (int64_t)rec[kRecKcut * n_samples + s];
        double acc = -0.5 * dd + total;
        for (int d = 0; d < n_det; ++d) {
            const double pr = rec[(kRecDet + kRecFieldsPerDet * d) * n_samples + s];
            const double pi = rec[(kRecDet + kRecFieldsPerDet * d + 1) * n_samples + s];
            double q = 4.0 * df * sums[kPrepPerDet * d + 1];
            if (isco) q = kcut >= 0 ? 4.0 * df * qprefix[(int64_t)d * n_bins + kcut] : 0.0;
            acc -= 0.5 * (pr * pr + pi * pi) * q;
        }
        out = acc;
    }
    if (flags & GW_FLAG_ADD_NORM) out -= norm;
    const int status = (int)rec[kRecStatus * n_samples + s];
    if (status == 1) out = -INFINITY;
    if (status == 2 || isnan(dd)) out = NAN;
    return out;
}

// Row s with its chunks summed in order (one thread per row).
__device__ __forceinline__ double finalize_row(int64_t s, int64_t n_samples, int n_det, int n_chunks,
                                               int64_t n_bins, double df, unsigned flags,
                                               const double2 *__restrict__ partials, const double *__restrict__ rec,
                                               const double *__restrict__ sums, const double *__restrict__ qprefix)
{
    const double *pd = reinterpret_cast<const double *>(partials);
    double total = 0.0;
    for (int c = 0; c < n_chunks; ++c) total += pd[(int64_t)c * n_samples + s];
    return assemble_row(s, n_samples, n_det, n_bins, df, flags, total, rec, sums, qprefix);
}

// One event: 16 rows per block, 16 threads per row; thread part p sums the
// chunk totals p, p + 16, ... in order, then the parts are added in order
// 0..15.
constexpr int kFinRows = 16, kFinParts = kBlock / kFinRows;

// Row s's chunk totals added up; true in the thread that has the sum.
__device__ __forceinline__ bool row_total(int64_t s, int64_t n_samples, int n_chunks,
                                          const double2 *__restrict__ partials, double &total)
{
    __shared__ double red[kFinParts][kFinRows];
    const int r = threadIdx.x % kFinRows, part = threadIdx.x / kFinRows;
    if (s < n_samples) {
        const double *pd = reinterpret_cast<const double *>(partials);
        double acc = 0.0;
        for (int c = part; c < n_chunks; c += kFinParts) acc += pd[(int64_t)c * n_samples + s];
        red[part][r] = acc;
    }
    __syncthreads();
    if (part != 0 || s >= n_samples) return false;
    total = 0.0;
    for (int p = 0; p < kFinParts; ++p) total += red[p][r];
    return true;
}

__global__ __launch_bounds__(kBlock) void lnl_finalize_kernel(int64_t n_samples, int n_det, int n_chunks,
                                                               int64_t n_bins, double df, unsigned flags,
                                                               const double2 *__restrict__ partials,
                                                               const double *__restrict__ rec,
                                                               const double *__restrict__ sums,
                                                               const double *__restrict__ qprefix,
                                                               const NodePlan *__restrict__ plan, int rounds,
                                                               int mixed, double *__restrict__ lnl)
{
    if (plan)
        n_chunks = mixed ? max(node_chunks_of(plan->k_bin, n_chunks, rounds),
                               node_chunks_of(plan->n_nodes, n_chunks, rounds))
                         : node_chunks_of(plan->k_bin + plan->n_nodes, n_chunks, rounds);
    const int64_t s = (int64_t)blockIdx.x * kFinRows + threadIdx.x % kFinRows;
    double total;
    if (row_total(s, n_samples, n_chunks, partials, total))
        lnl[s] = assemble_row(s, n_samples, n_det, n_bins, df, flags, total, rec, sums, qprefix);
}

// Ragged batch on frequency nodes: blocks 16 i .. 16 i + 15 finalize the rows of group i.
__global__ __launch_bounds__(kBlock) void ragged_node_finalize_kernel(const RaggedEvent *__restrict__ events,
                                                                      const int2 *__restrict__ groups, unsigned flags)
{
    constexpr int kParts = kBlock / kFinRows;
    const int2 eg = groups[blockIdx.x / kParts];
    const RaggedEvent &re = events[eg.x];
    const int64_t s = (int64_t)eg.y * kBlock + (int64_t)(blockIdx.x % kParts) * kFinRows + threadIdx.x % kFinRows;
    double total;
    if (row_total(s, re.n_samples, re.split[0] + re.split[1], re.partials, total))
        re.lnl[s] = assemble_row(s, re.n_samples, re.n_det, re.n_bins, re.df, flags, total, re.rec, re.sums, nullptr);
}

// Ragged batch: block (event, group) finalizes the group's rows.
__global__ __launch_bounds__(kBlock) void ragged_finalize_kernel(const RaggedEvent *__restrict__ events,
                                                                  const int2 *__restrict__ groups, unsigned flags)
{
    const int2 eg = groups[blockIdx.x];
    const RaggedEvent &re = events[eg.x];
    const int64_t s = (int64_t)eg.y * kBlock + threadIdx.x;
    if (s >= re.n_samples) return;
    re.lnl[s] = finalize_row(s, re.n_samples, re.n_det, re.n_chunks, re.n_bins, re.df, flags, re.partials, re.rec,
                             re.sums, re.qprefix);
}

// ---------------------------------------------------------------- launchers
static int grid_blocks(int64_t n, int cap)
{
    const int64_t b = (n + kBlock - 1) / kBlock;
    return (int)(b < 1 ? 1 : (b > cap ? cap : b));
}

hipError_t launch_event_tables(const gw_grid &grid, Tab1 *tab1, Tab2 *tab2, hipStream_t stream)
{
    hipLaunchKernelGGL(event_tables_kernel, dim3(grid_blocks(grid.n_bins, 4096)), dim3(kBlock), 0, stream,
                       grid.f_low, grid.delta_f, grid.n_bins, tab1, tab2);
    return hipGetLastError();
}

hipError_t launch_event_data(const gw_grid &grid, int n_det, const gw_c128 *data, const double *psd,
                             const EventBuffers &eb, unsigned flags, const SamplePrep *sp, hipStream_t stream)
{
    PrepView v;
    v.n_bins = grid.n_bins;
    v.n_det = n_det;
    v.df = grid.delta_f;
    v.data = reinterpret_cast<const double2 *>(data);
    v.psd = psd;
    v.tab2 = eb.tab2;
    v.dcoef = eb.dcoef;
    v.edir = eb.edir;
    v.vdir = eb.vdir;
    const int direct = (flags & GW_FLAG_DIRECT) ? 1 : 0, norm = (flags & GW_FLAG_ADD_NORM) ? 1 : 0;
    SamplePrep none{};
    const int sample_blocks = sp ? (int)((sp->n_samples + kSampleRows - 1) / kSampleRows) : 0;
    hipLaunchKernelGGL(event_data_kernel, dim3(eb.prep_blocks + sample_blocks), dim3(kBlock), 0, stream, v, direct,
                       norm, eb.prep, sample_blocks, grid.f_low, sp ? *sp : none);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(event_sums_kernel, dim3(kPrepPerDet * n_det), dim3(kBlock), 0, stream, eb.prep_blocks, n_det,
                       eb.prep, eb.sums, eb.queue);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (flags & GW_FLAG_TERM_ISCO) {
        hipLaunchKernelGGL(event_offsets_kernel, dim3(n_det), dim3(kBlock), 0, stream, (int64_t)eb.prep_blocks, n_det,
                           eb.prep, eb.qoffsets);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        hipLaunchKernelGGL(event_prefix_kernel, dim3(eb.prep_blocks), dim3(kBlock), 0, stream, v,
                           (int64_t)eb.prep_blocks, eb.qoffsets, eb.qprefix);
        e = hipGetLastError();
    }
    return e;
}

hipError_t launch_sample_prep(const gw_grid &grid, int64_t n_samples, int n_param, int n_out, bool polarisations,
                              bool isco, const DetGeom &geom, const double *theta, double *records,
                              hipStream_t stream)
{
    hipLaunchKernelGGL(sample_prep_kernel, dim3((unsigned)((n_samples + kSampleRows - 1) / kSampleRows)), dim3(kBlock), 0,
                       stream,
                       grid.f_low, grid.delta_f, grid.n_bins, n_samples, n_param, n_out, polarisations ? 1 : 0,
                       isco ? 1 : 0, geom, theta, records);
    return hipGetLastError();
}

hipError_t launch_isco_limit(int64_t n_samples, const double *records, int64_t *k_limit, hipStream_t stream)
{
    hipLaunchKernelGGL(isco_limit_kernel, dim3(1), dim3(kBlock), 0, stream, n_samples, records, k_limit);
    return hipGetLastError();
}

hipError_t launch_node_samples(const gw_grid &grid, int n_det, const SamplePrep &sp, double *stats,
                               hipStream_t stream)
{
    const int64_t entries = node_stat_entries(sp.n_samples);
    if (entries > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(node_samples_kernel, dim3((unsigned)entries), dim3(kBlock), 0, stream, grid.f_low, grid.delta_f,
                       grid.n_bins, n_det, sp, stats);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || entries <= kStatEntries) return e;
    hipLaunchKernelGGL(node_range_kernel, dim3(kStats), dim3(kBlock), 0, stream, entries, stats,
                       stats + entries * kStats);
    return hipGetLastError();
}

size_t lnl_tile_lds_bytes(int n_det, int tile_bins, int form, bool mixed)
{
    return tile_lds_bytes(n_det, tile_bins, form, mixed);
}

template <int NDET, bool MIXED>
static const void *tile_kernel_form(int form)
{
    switch (form) {
    case kFormSplit: return reinterpret_cast<const void *>(&lnl_tile_kernel<NDET, MIXED, kFormSplit, kNoNodes>);
    case kFormSplitIsco: return reinterpret_cast<const void *>(&lnl_tile_kernel<NDET, MIXED, kFormSplitIsco, kNoNodes>);
    default: return reinterpret_cast<const void *>(&lnl_tile_kernel<NDET, MIXED, kFormDirect, kNoNodes>);
    }
}

template <int NDET, bool MIXED>
static const void *ragged_kernel_form(int form)
{
    switch (form) {
    case kFormSplit: return reinterpret_cast<const void *>(&lnl_ragged_kernel<NDET, MIXED, kFormSplit>);
    case kFormSplitIsco: return reinterpret_cast<const void *>(&lnl_ragged_kernel<NDET, MIXED, kFormSplitIsco>);
    default: return reinterpret_cast<const void *>(&lnl_ragged_kernel<NDET, MIXED, kFormDirect>);
    }
}

template <int NDET>
static const void *node_kernel(NodeMode mode)
{
    switch (mode) {
    case kNodeBins: return reinterpret_cast<const void *>(&lnl_tile_kernel<NDET, true, kFormSplit, kNodeBins>);
    case kNodesOnly: return reinterpret_cast<const void *>(&lnl_tile_kernel<NDET, false, kFormSplit, kNodesOnly>);
    default: return reinterpret_cast<const void *>(&lnl_tile_kernel<NDET, false, kFormSplit, kBinsAndNodes>);
    }
}

static const void *node_kernel_for(int n_det, NodeMode mode)
{
    switch (n_det) {
    case 1: return node_kernel<1>(mode);
    case 2: return node_kernel<2>(mode);
    case 3: return node_kernel<3>(mode);
    case 4: return node_kernel<4>(mode);
    case 5: return node_kernel<5>(mode);
    case 6: return node_kernel<6>(mode);
    case 7: return node_kernel<7>(mode);
    case 8: return node_kernel<8>(mode);
    default: return nullptr;
    }
}

template <int NDET>
static const void *ragged_node_kernel_mode(NodeMode mode)
{
    switch (mode) {
    case kNodeBins: return reinterpret_cast<const void *>(&ragged_node_kernel<NDET, true, kNodeBins>);
    case kNodesOnly: return reinterpret_cast<const void *>(&ragged_node_kernel<NDET, false, kNodesOnly>);
    default: return reinterpret_cast<const void *>(&ragged_node_kernel<NDET, false, kBinsAndNodes>);
    }
}

static const void *ragged_node_kernel_for(int n_det, NodeMode mode)
{
    switch (n_det) {
    case 1: return ragged_node_kernel_mode<1>(mode);
    case 2: return ragged_node_kernel_mode<2>(mode);
    case 3: return ragged_node_kernel_mode<3>(mode);
    case 4: return ragged_node_kernel_mode<4>(mode);
    case 5: return ragged_node_kernel_mode<5>(mode);
    case 6: return ragged_node_kernel_mode<6>(mode);
    case 7: return ragged_node_kernel_mode<7>(mode);
    case 8: return ragged_node_kernel_mode<8>(mode);
    default: return nullptr;
    }
}

// The kernel (tile or ragged) for a detector count, precision and form.
static const void *kernel_for(bool ragged, int n_det, bool mixed, int form)
{
#define GW_KERNEL_CASE(N)                                                                                        \
    case N:                                                                                                    \
        if (ragged) return mixed ? ragged_kernel_form<N, true>(form) : ragged_kernel_form<N, false>(form);      \
        return mixed ? tile_kernel_form<N, true>(form) : tile_kernel_form<N, false>(form);
    switch (n_det) {
        GW_KERNEL_CASE(1)
        GW_KERNEL_CASE(2)
        GW_KERNEL_CASE(3)
        GW_KERNEL_CASE(4)
        GW_KERNEL_CASE(5)
        GW_KERNEL_CASE(6)
        GW_KERNEL_CASE(7)
        GW_KERNEL_CASE(8)
    default: return nullptr;
    }
#undef GW_KERNEL_CASE
}

static int occupancy(const void *fn, size_t lds)
{
    int n = 0;
    if (!fn || hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, fn, kBlock, lds) != hipSuccess) return 1;
    return n < 1 ? 1 : n;
}

int lnl_tile_blocks_per_cu(int n_det, int tile_bins, bool mixed, int form)
{
    return occupancy(kernel_for(false, n_det, mixed, form), tile_lds_bytes(n_det, tile_bins, form, mixed));
}

int lnl_ragged_blocks_per_cu(int n_det, int tile_bins, bool mixed, int form)
{
    return occupancy(kernel_for(true, n_det, mixed, form), tile_lds_bytes(n_det, tile_bins, form, mixed));
}

static NodeMode ragged_mode(bool mixed, int pass) { return !mixed ? kBinsAndNodes : pass == 0 ? kNodeBins : kNodesOnly; }

int ragged_node_blocks_per_cu(int n_det, int tile_bins, bool mixed, int pass)
{
    const NodeMode mode = ragged_mode(mixed, pass);
    return occupancy(ragged_node_kernel_for(n_det, mode),
                     tile_lds_bytes(n_det, tile_bins, kFormSplit, mode == kNodeBins));
}

hipError_t launch_lnl_tiles(const gw_grid &grid, int n_det, int64_t n_samples, const TilePlan &plan, bool mixed,
                            int form, const EventBuffers &eb, const double *records, double2 *partials,
                            hipStream_t stream)
{
    EventView ev;
    ev.n_bins = grid.n_bins;
    ev.n_samples = n_samples;
    ev.f_low = grid.f_low;
    ev.df = grid.delta_f;
    ev.tab1 = eb.tab1;
    ev.dcoef = eb.dcoef;
    ev.edir = eb.edir;
    ev.vdir = eb.vdir;
    ev.rec = records;
    ev.k_limit = eb.k_limit;
    ev.partials = partials;
    ev.plan = eb.node_plan;
    int n_groups = plan.n_groups, n_chunks = plan.n_chunks, rounds = plan.rounds;
    if (plan.rounds > 0 && !eb.queue) return hipErrorInvalidValue;
    auto launch = [&](const void *fn, bool mixed_kernel, int tile_bins, unsigned *queue) {
        if (!fn) return hipErrorInvalidValue;
        void *args[] = {&ev, &n_groups, &n_chunks, &rounds, &tile_bins, &queue};
        return hipLaunchKernel(fn, dim3((unsigned)plan.blocks), dim3(kBlock), args,
                               tile_lds_bytes(n_det, tile_bins, form, mixed_kernel), stream);
    };
    unsigned *queue = plan.rounds > 0 ? eb.queue : nullptr;
    if (!eb.node_plan) return launch(kernel_for(false, n_det, mixed, form), mixed, plan.tile_bins, queue);
    if (form != kFormSplit) return hipErrorInvalidValue;
    if (!mixed) return launch(node_kernel_for(n_det, kBinsAndNodes), false, plan.tile_bins, queue);
    hipError_t e = launch(node_kernel_for(n_det, kNodeBins), true, plan.tile_bins, queue);
    if (e != hipSuccess) return e;
    return launch(node_kernel_for(n_det, kNodesOnly), false, std::min(plan.tile_bins, tile_bins_for(n_det, form, false)),
                  queue ? queue + kQueues : nullptr);
}

hipError_t launch_ragged_tables(const RaggedLaunch &r, hipStream_t stream)
{
    hipLaunchKernelGGL(ragged_tables_kernel, dim3(r.n_prep_blocks), dim3(kBlock), 0, stream, r.events, r.block_map);
    return hipGetLastError();
}

// A ragged pass on frequency nodes: the samples first (the range of their phases
// decides where an event's nodes stand), then as one event's call does it.
static hipError_t launch_ragged_nodes(const RaggedLaunch &r, hipStream_t stream)
{
    hipLaunchKernelGGL(ragged_sample_prep_kernel, dim3(r.n_groups * (kBlock / kSampleRows)), dim3(kBlock), 0, stream,
                       r.events, r.groups, r.geoms, r.n_param, 0);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || (e = launch_ragged_plans(r, stream)) != hipSuccess) return e;
    for (int i = 0; i < r.n_classes; ++i) {
        const RaggedClass &c = r.classes[i];
        hipLaunchKernelGGL(ragged_split_kernel, dim3(1), dim3(kBlock), 0, stream, r.events, c.events, c.n_events,
                           r.mixed ? 1 : 0, make_int2(c.pass_grid[0], c.pass_grid[1]), c.first, c.counter);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    if ((e = launch_ragged_spread(r, stream)) != hipSuccess) return e;
    if ((e = launch_ragged_combine(r, stream)) != hipSuccess) return e;
    for (int i = 0; i < r.n_classes; ++i) {
        const RaggedClass &c = r.classes[i];
        const RaggedEvent *events = r.events;
        const int *members = c.events;
        const unsigned *first = c.first;
        unsigned *counter = c.counter;
        int n = c.n_events, tile_bins = 0;
        void *args[] = {&events, &members, &n, &first, &counter, &tile_bins};
        for (int pass = 0; pass < (r.mixed ? 2 : 1); ++pass) {
            const NodeMode mode = ragged_mode(r.mixed, pass);
            const void *fn = ragged_node_kernel_for(c.n_det, mode);
            if (!fn) return hipErrorInvalidValue;
            tile_bins = c.pass_tile[pass];
            e = hipLaunchKernel(fn, dim3(c.pass_grid[pass]), dim3(kBlock), args,
                                tile_lds_bytes(c.n_det, tile_bins, kFormSplit, mode == kNodeBins), stream);
            if (e != hipSuccess) return e;
        }
    }
    hipLaunchKernelGGL(ragged_node_finalize_kernel, dim3((unsigned)r.n_groups * (kBlock / kFinRows)), dim3(kBlock), 0,
                       stream, r.events, r.groups, r.flags);
    return hipGetLastError();
}

hipError_t launch_ragged(const RaggedLaunch &r, hipStream_t stream)
{
    if (r.nodes) return launch_ragged_nodes(r, stream);
    const int direct = (r.flags & GW_FLAG_DIRECT) ? 1 : 0, norm = (r.flags & GW_FLAG_ADD_NORM) ? 1 : 0;
    const int form = tile_form(r.flags);
    hipLaunchKernelGGL(ragged_event_prep_kernel, dim3(r.n_prep_blocks), dim3(kBlock), 0, stream, r.events,
                       r.block_map, direct, norm);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(ragged_event_sums_kernel, dim3(r.n_events), dim3(kBlock), 0, stream, r.events);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if (r.flags & GW_FLAG_TERM_ISCO) {
        hipLaunchKernelGGL(ragged_offsets_kernel, dim3(r.n_events), dim3(kBlock), 0, stream, r.events);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        hipLaunchKernelGGL(ragged_prefix_kernel, dim3(r.n_prep_blocks), dim3(kBlock), 0, stream, r.events,
                           r.block_map);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    hipLaunchKernelGGL(ragged_sample_prep_kernel, dim3(r.n_groups * (kBlock / kSampleRows)), dim3(kBlock), 0, stream, r.events, r.groups,
                       r.geoms, r.n_param, (r.flags & GW_FLAG_TERM_ISCO) ? 1 : 0);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(zero_counters_kernel, dim3(1), dim3(64), 0, stream, r.counters, 2 * kMaxDet);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    for (int i = 0; i < r.n_classes; ++i) {
        const RaggedClass &c = r.classes[i];
        const void *fn = kernel_for(true, c.n_det, r.mixed, form);
        if (!fn) return hipErrorInvalidValue;
        const RaggedEvent *events = r.events;
        const WorkItem *items = c.items;
        int n_items = c.n_items, tile_bins = r.tile_bins;
        unsigned *counter = c.counter;
        void *args[] = {&events, &items, &n_items, &counter, &tile_bins};
        e = hipLaunchKernel(fn, dim3(c.grid), dim3(kBlock), args,
                            tile_lds_bytes(c.n_det, r.tile_bins, form, r.mixed), stream);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(ragged_finalize_kernel, dim3(r.n_groups), dim3(kBlock), 0, stream, r.events, r.groups,
                       r.flags);
    return hipGetLastError();
}

hipError_t launch_lnl_finalize(const gw_grid &grid, int64_t n_samples, int n_det, const TilePlan &plan,
                               bool mixed, const double2 *partials, const double *records, const EventBuffers &eb,
                               unsigned flags, double *lnl_out, hipStream_t stream)
{
    const int64_t blocks = (n_samples + kFinRows - 1) / kFinRows;
    hipLaunchKernelGGL(lnl_finalize_kernel, dim3((unsigned)blocks), dim3(kBlock), 0, stream, n_samples, n_det,
                       plan.n_chunks, grid.n_bins, grid.delta_f, flags, partials, records, eb.sums, eb.qprefix,
                       eb.node_plan, plan.rounds, mixed ? 1 : 0, lnl_out);
    return hipGetLastError();
}


}  // namespace gw

GW_DEFINE_SOURCE_HASH(kernels)
