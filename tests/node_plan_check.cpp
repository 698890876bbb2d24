// Host check of a batch's node plan (csrc/gw_nodes.h), formed from the functions that the
// device forms it with, for many ranges of phase coefficients, grids and detector
// counts.  A sample's phase less the reference's, differentiated term by term, stays
// within the bound at every frequency a node can have; that bound falls with the frequency
// and keeps every node of a level within the band that its weights serve; no node
// stands below half of f_low; no difference from the reference is more than 1.5 times the
// coefficient itself; and the levels tile the band with consecutive chunks and
// nodes.  Built and run by tests/test_node_plan_host.py; prints "ok N" or the first failure.
#include <cmath>
#include <cstdio>
#include <random>

#include "gw_nodes.h"

#define REQUIRE(c)                                                  \
    do {                                                            \
        if (!(c)) {                                                 \
            std::printf("failed: %s (case %d, q %d)\n", #c, it, q); \
            return 1;                                               \
        }                                                           \
    } while (0)

// tau, c7, c6, c6l, c5l, c4, c3, c2, c0 as kStatPairs orders them: d/df of the phase at u^3
static double slope(const double *c, double u)
{
    const double dx_du = 2.0 * c[1] * u + c[2] + c[3] * (std::log(u) + 1.0) + c[4] / u - c[5] / (u * u) -
                         2.0 * c[6] / (u * u * u) - 3.0 * c[7] / std::pow(u, 4) - 5.0 * c[8] / std::pow(u, 6);
    return c[0] + dx_du / (3.0 * u * u);
}

int main()
{
    std::mt19937_64 rng(11);
    auto uni = [&](double a, double b) { return std::uniform_real_distribution<double>(a, b)(rng); };
    int q = 0, with_levels = 0, with_bins = 0, without = 0;
    const int n_cases = 3000;
    for (int it = 0; it < n_cases; ++it) {
        const double f_low = std::exp(uni(std::log(2.0), std::log(40.0))), df = std::exp(uni(std::log(1e-3), std::log(1.0)));
        const int64_t n_bins = 1 + (int64_t)std::exp(uni(std::log(300.0), std::log(2e6)));
        const int n_det = 1 + (int)(rng() % 8);
        // coefficients of the size a binary's chirp has (mass in seconds 1e-6 .. 4e-4), and a relative range of them
        const double m = std::exp(uni(std::log(1e-6), std::log(4e-4))), a = std::cbrt(M_PI * m);
        const double size[gw::kStatPairs] = {uni(0.0, 2.0) / df * 1e-3, a * a, a, a, 1.0, 1.0 / a, 1.0 / (a * a),
                                             1.0 / std::pow(a, 3), 1.0 / std::pow(a, 5)};
        double lo[gw::kStatPairs], hi[gw::kStatPairs], mid[gw::kStatPairs], half[gw::kStatPairs];
        for (int j = 0; j < gw::kStatPairs; ++j) {
            const double c = uni(-1.0, 1.0) * size[j] * 0.1, w = size[j] * std::exp(uni(std::log(1e-9), std::log(1.0)));
            lo[j] = c - w * 0.1;
            hi[j] = c + w * 0.1;
            gw::node_middle(lo[j], hi[j], mid[j], half[j]);
        }
        const gw::NodeBand band = gw::node_band(f_low, df, n_bins);
        const gw::RateBound r = gw::node_bound(half, band);
        int failing[gw::kNodeSpacings] = {}, first[gw::kNodeSpacings];
        double before = INFINITY;
        for (int t = 0; t < gw::kBlock; ++t) {
            const double rate = gw::node_rate(r, gw::node_probe(band, t));
            REQUIRE(rate <= before);
            before = rate;
            const int allowed = gw::node_allowed(rate, df);
            for (int g = 0; g < gw::kNodeSpacings; ++g) failing[g] += allowed <= g;
        }
        for (int g = 0; g < gw::kNodeSpacings; ++g) first[g] = gw::node_first_bin(band, g, failing[g]);
        gw::NodePlan p{};
        gw::node_levels(first, (int)n_bins, n_det, p);
        // what the device takes as "no nodes" before it looks for levels
        if (gw::node_allowed(gw::node_rate(r, band.u_high), df) == 0) {
            REQUIRE(p.n_levels == 0 && p.k_bin == n_bins);
            ++without;
        }
        // the samples' slopes
        for (int s = 0; s < 8; ++s) {
            double c[gw::kStatPairs];
            for (int j = 0; j < gw::kStatPairs; ++j) {
                const double v = s < 2 ? (s ? hi[j] : lo[j]) : lo[j] + (hi[j] - lo[j]) * uni(0.0, 1.0);
                c[j] = v - mid[j];
                REQUIRE(std::fabs(c[j]) <= 1.5 * std::fabs(v) * (1.0 + 1e-12));
            }
            const double top = f_low + (double)n_bins * df + 2.0 * gw::kTaps * 1024.0 * df;
            for (int k = 0; k < 20; ++k) {
                const double u = std::cbrt(std::exp(uni(std::log(0.5 * f_low), std::log(top))));
                REQUIRE(std::fabs(slope(c, u)) <= gw::node_rate(r, u) * (1.0 + 1e-9));
            }
        }
        int64_t at = p.k_bin;
        int chunk = p.bin_chunks, node = 0;
        for (int l = 0; l < p.n_levels; ++l) {
            const gw::NodeLevel &v = p.level[l];
            q = v.q;
            REQUIRE(v.k0 == at && v.chunk0 == chunk && v.node0 == node);
            const double f = f_low + ((double)v.k0 - (double)gw::kTapsBelow * v.q) * df;
            REQUIRE(f >= 0.5 * f_low * (1.0 - 1e-12));
            REQUIRE(gw::node_rate(r, std::cbrt(f)) * v.q * df <= GW_RESAMPLE_BAND * (1.0 + 1e-9));
            at = v.k1;
            chunk += v.n_chunks;
            node += gw::node_count(v);
        }
        q = 0;
        REQUIRE(at == n_bins && chunk == p.n_chunks && node == p.n_nodes);
        with_levels += p.n_levels > 1;
        with_bins += p.k_bin > 0;
    }
    const int it = n_cases;
    REQUIRE(with_levels > n_cases / 10 && with_bins > n_cases / 10 && without > n_cases / 50);
    std::printf("ok %d\n", n_cases);
    return 0;
}
