// Host check of the frequency nodes' geometry (csrc/gw_nodes.h): for many first-bin
// tables, band lengths and detector counts, the levels and single bins
// tile the band; every level's partial nodes, nodes and tables fit its own part of D;
// the chunks of the weighting hold every bin exactly once, within the block's
// LDS rows, and no more of them than the workspace has sums for; a node's
// partials are exactly those of the chunks with a cell among the 32 below it; and the
// work split stays within the host's plan.  Prints "ok N" or the first failure.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "gw_nodes.h"

#define REQUIRE(c)                                                                                     \
    do {                                                                                               \
        if (!(c)) {                                                                                    \
            std::printf("failed: %s (n_bins %lld n_det %d level q %d)\n", #c, (long long)n_bins, n_det, q); \
            return 1;                                                                                  \
        }                                                                                              \
    } while (0)

int main()
{
    std::mt19937_64 rng(7);
    int done = 0;
    for (int it = 0; it < 4000; ++it) {
        const double lg = std::uniform_real_distribution<double>(9.0, it % 50 == 0 ? 21.0 : 18.0)(rng);
        const int64_t n_bins = 1 + (int64_t)std::exp2(lg);
        const int n_det = 1 + (int)(rng() % 8);
        int first[gw::kNodeSpacings];
        int64_t k = it % 3 == 0 ? 0 : (int64_t)(rng() % (uint64_t)(n_bins / 4 + 1));
        for (int i = 0; i < gw::kNodeSpacings; ++i) {
            first[i] = (int)(k < n_bins ? k : n_bins);
            if (rng() % 4) k += (int64_t)(rng() % (uint64_t)(1 + n_bins / 6)) * (int64_t)(rng() % 3) / 2;
        }
        gw::NodePlan p{};
        gw::node_levels(first, (int)n_bins, n_det, p);
        int q = 0;
        int64_t at = p.k_bin;
        int chunk = p.bin_chunks, node = 0;
        REQUIRE(p.bin_chunks == (p.k_bin + gw::kSpreadBins - 1) / gw::kSpreadBins);
        REQUIRE(p.n_levels >= 0 && p.n_levels <= gw::kNodeSpacings);
        for (int l = 0; l < p.n_levels; ++l) {
            const gw::NodeLevel &v = p.level[l];
            q = v.q;
            REQUIRE(v.k0 == at && v.k1 > v.k0 && v.chunk0 == chunk && v.node0 == node);
            REQUIRE(l == 0 || v.q > p.level[l - 1].q);
            REQUIRE((int64_t)v.cells * v.q >= v.k1 - v.k0 && (int64_t)(v.cells - 1) * v.q < v.k1 - v.k0);
            REQUIRE(v.k1 - v.k0 >= (int64_t)(l > 0 ? gw::kNodeMinCells : gw::kNodeLowCells) * v.q && gw::node_room_ok(v));
            REQUIRE(v.subs * v.sub_bins >= v.q && v.cpc * v.sub_bins <= gw::kSpreadBins);
            REQUIRE(v.cpc <= gw::kSpreadBins / gw::node_spacing(0));
            REQUIRE(v.subs == 1 ? v.sub_bins == v.q : v.cpc == gw::node_pack(n_det));
            // every bin in one chunk
            std::vector<int> seen((size_t)(v.k1 - v.k0), 0);
            for (int c = 0; c < v.n_chunks; ++c) {
                const int cell0 = c / v.subs * v.cpc, j0 = c % v.subs * v.sub_bins;
                for (int b = 0; b < v.cpc * v.sub_bins; ++b) {
                    const int cell = b / v.sub_bins, j = b % v.sub_bins;
                    if (j0 + j >= v.q) continue;
                    const int64_t bin = (int64_t)(cell0 + cell) * v.q + j0 + j;
                    if (bin < v.k1 - v.k0) ++seen[(size_t)bin];
                }
            }
            for (int s : seen) REQUIRE(s == 1);
            // a node's partials
            const int per = v.cpc + gw::kTaps - 1, runs = v.n_chunks / v.subs;
            REQUIRE(runs * v.subs == v.n_chunks);
            for (int n = 0; n < gw::node_count(v); ++n) {
                const int lo = n >= per ? (n - per) / v.cpc + 1 : 0;
                const int hi = runs - 1 < n / v.cpc ? runs - 1 : n / v.cpc;
                for (int r = 0; r < runs; ++r) {
                    const bool reaches = n >= r * v.cpc && n < r * v.cpc + per;
                    REQUIRE(reaches == (r >= lo && r <= hi));
                }
            }
            at = v.k1;
            chunk += v.n_chunks;
            node += gw::node_count(v);
        }
        REQUIRE(at == n_bins && p.n_chunks == chunk && p.n_nodes == node);
        REQUIRE(p.n_chunks <= gw::node_max_chunks(n_bins));
        for (int rounds : {0, 1, 4, 6}) {
            const int chunks = (rounds > 0 ? rounds : 1) * (1 + (int)(rng() % 60));
            int ec = 0, er = 0;
            gw::node_split(p.k_bin + p.n_nodes, chunks, rounds, ec, er);
            REQUIRE(ec >= 1 && ec <= chunks && er <= rounds && (rounds > 0 ? er >= 1 && ec % er == 0 : er == 0));
        }
        ++done;
    }
    std::printf("ok %d\n", done);
    return 0;
}
