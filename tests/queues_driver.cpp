// For every line  heads video_blocks text_blocks order  on standard input: the items of the eight queues in order, as
// "head,ordinal" separated by spaces, one line per queue.
#include <cstdio>

#include "rf_queues.h"

int main() {
    int heads, video, text, order;
    while (std::scanf("%d %d %d %d", &heads, &video, &text, &order) == 4) {
        const rf::Queues<true> qs(heads, video, text, order);
        for (int x = 0; x < 8; ++x) {
            for (int i = 0; i < qs.items(x); ++i) {
                int bh = -1, ordinal = -1;
                qs.locate(i, x, &bh, &ordinal);
                std::printf("%d,%d ", bh, ordinal);
            }
            std::printf("\n");
        }
    }
    return 0;
}
