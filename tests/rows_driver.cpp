// Prints choose_form() for every line  T H W text BH D dense room bandwidth stride  on standard input.
#include <cstdio>

#include "rf_internal.h"

int main() {
    int T, H, W, text, BH, D, dense, room, stride;
    float bw;
    while (std::scanf("%d %d %d %d %d %d %d %d %f %d", &T, &H, &W, &text, &BH, &D, &dense, &room, &bw, &stride) == 10) {
        const rf_layout layout = {T, H, W, text};
        const rf_params params = {bw, bw, stride, 0, 0};
        rf::Geometry g;
        if (rf::resolve_geometry(&layout, &params, &g) != RF_OK) return 1;
        const rf::AttnForm f = rf::choose_form(g, BH, D, dense != 0, room != 0);
        std::printf("%d %d %d %d\n", f.rows, f.key_groups, f.queued ? 1 : 0, f.copies ? 1 : 0);
    }
    return 0;
}
