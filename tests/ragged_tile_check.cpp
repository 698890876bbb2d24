// Host check of the LDS tiles of a ragged call's passes on frequency nodes (gw_plan.h),
// built and run by tests/test_ragged_tile_host.py: for every detector count, precision
// and tile the autotuner may time, each pass's block fits 80 KB (two blocks per
// compute unit), no pass has a larger tile than was asked for, and a tile is at
// least 64 bins; and the items a call is cut into are neither so short that they
// cost more than their sums nor so long that the last ones run alone.  Prints
// "ok <cases>" or the first failure.
#include <cstdio>

#include "gw_nodes.h"
#include "gw_plan.h"

namespace gw {
// the tile kernels' LDS layout: bin tables, D per detector, and the phasor table on the FP64 path
size_t lnl_tile_lds_bytes(int n_det, int tile_bins, int, bool mixed)
{
    return (mixed ? 0 : (size_t)PHASOR_TABLE_BYTES) + (size_t)tile_bins * (32 + 16 * (size_t)n_det);
}
}  // namespace gw

int main()
{
    int cases = 0;
    for (int n_det = 1; n_det <= gw::kMaxDet; ++n_det)
        for (int mixed = 0; mixed < 2; ++mixed)
            for (int tile : {256, 512}) {
                if (gw::lnl_tile_lds_bytes(n_det, tile, gw::kFormSplit, mixed != 0) > 80 * 1024) continue;
                for (int pass = 0; pass <= mixed; ++pass) {
                    const int t = gw::ragged_pass_tile(n_det, tile, mixed != 0, pass);
                    const size_t lds = gw::lnl_tile_lds_bytes(n_det, t, gw::kFormSplit, mixed != 0 && pass == 0);
                    if (t > tile || t < 64 || t % 64 != 0 || lds > 80 * 1024) {
                        std::printf("FAIL %d detectors mixed %d tile %d pass %d: tile %d, %zu bytes\n", n_det, mixed,
                                    tile, pass, t, lds);
                        return 1;
                    }
                    ++cases;
                }
            }
    for (int grid : {1, 256, 512, 768})
        for (double work = 0.0; work < 1e9; work = work * 1.7 + 1.0) {
            const int64_t u = gw::ragged_item_units(work, grid);
            if (u < 64 || u > 1024 || (u > 64 && u < 1024 && (double)u * 4.0 * grid < work)) {
                std::printf("FAIL work %g on %d blocks: items of %lld\n", work, grid, (long long)u);
                return 1;
            }
            ++cases;
        }
    std::printf("ok %d\n", cases);
    return 0;
}
