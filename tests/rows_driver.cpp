// Prints choose_rows() for every line  T H W text BH D dense room  on standard input.
#include <cstdio>

#include "rf_internal.h"

int main() {
    int T, H, W, text, BH, D, dense, room;
    while (std::scanf("%d %d %d %d %d %d %d %d", &T, &H, &W, &text, &BH, &D, &dense, &room) == 8) {
        const rf_layout layout = {T, H, W, text};
        rf::Geometry g;
        if (rf::resolve_geometry(&layout, nullptr, &g) != RF_OK) return 1;
        std::printf("%d\n", rf::choose_rows(g, BH, D, dense != 0, room != 0));
    }
    return 0;
}
