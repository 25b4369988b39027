// For every line  T H W text bandwidth text_first  on standard input: compares the tiles that BandTiles gives every block of rows
// with the lists of build_plan, and position_major_row with its table; prints the number of entries and rows compared, or where
// they differ.
#include <cstdio>

#include "rf_band.h"

int main() {
    int T, H, W, text, first;
    float bw;
    while (std::scanf("%d %d %d %d %f %d", &T, &H, &W, &text, &bw, &first) == 6) {
        const rf_layout layout = {T, H, W, text};
        const rf_params params = {bw, bw, 2, 0, first ? RF_FLAG_TEXT_FIRST : 0};
        rf::Geometry g;
        if (rf::resolve_geometry(&layout, &params, &g) != RF_OK) return 1;
        rf::TokenTables tables;
        rf::build_tables(g, &tables);
        long long compared = 0;
        for (int n = 0; n < g.N; ++n, ++compared)
            if (rf::position_major_row(n, g.T, g.HW, g.Nv, g.video_shift(), g.text_shift()) != tables.pm_token[n]) return std::printf("row %d\n", n), 2;
        for (int block : {64, 128, 256}) {
            rf::HostPlan p;
            rf::build_plan(g, tables, block, false, &p);
            for (int list : {static_cast<int>(RF_SPATIAL), rf::kListTemporalPM})
                for (int qb = 0; qb < p.nQB; ++qb) {
                    const int e0 = p.row_ptr[list][qb], count = p.row_ptr[list][qb + 1] - e0;
                    const rf::BandTiles b(qb * block, block, list == RF_SPATIAL ? g.HW : g.T, list == RF_SPATIAL ? g.r_spatial : g.r_temporal, g.N, g.Nv);
                    if (b.tiles != count) return std::printf("block %d x %d, list %d: %d tiles, not %d\n", qb, block, list, b.tiles, count), 2;
                    for (int t = 0; t < count; ++t, ++compared)
                        if (b.entry(t, g.N, g.Nv) != p.cols[list][e0 + t]) return std::printf("block %d x %d, list %d, entry %d\n", qb, block, list, t), 2;
                }
        }
        std::printf("%lld\n", compared);
    }
    return 0;
}
