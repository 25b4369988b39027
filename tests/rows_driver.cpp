// Prints choose_form() for every line  T H W text BH D dense room  on standard input.
#include <cstdio>

#include "rf_internal.h"

int main() {
    int T, H, W, text, BH, D, dense, room;
    while (std::scanf("%d %d %d %d %d %d %d %d", &T, &H, &W, &text, &BH, &D, &dense, &room) == 8) {
        const rf_layout layout = {T, H, W, text};
        rf::Geometry g;
        if (rf::resolve_geometry(&layout, nullptr, &g) != RF_OK) return 1;
        const rf::AttnForm f = rf::choose_form(g, BH, D, dense != 0, room != 0);
        std::printf("%d %d %d %d\n", f.rows, f.key_groups, f.queued ? 1 : 0, f.copies ? 1 : 0);
    }
    return 0;
}
