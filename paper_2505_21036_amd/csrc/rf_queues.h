// Which (head, query block) items of an attention launch each of the eight XCDs takes, and in which order: plain
// integer arithmetic, the same on the host and on the device.
#pragma once
#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define RF_BOTH __host__ __device__ __forceinline__
#else
#define RF_BOTH inline
#endif

namespace rf {

// Queue x holds first its share of the long items (the nTB text-holding blocks of every head: global index
// i = head * nTB + k goes to queue i mod 8), then its part of the nVB other blocks of every head, as the order says.
enum : int {
    ORDER_EIGHTHS = 0,  // of every head, head after head, the ordinals [x * per_xcd, (x+1) * per_xcd) of its block order
    ORDER_HEADS = 1,    // the items [x * per_xcd, (x+1) * per_xcd) of all heads' blocks in a row: whole heads, mostly
    // Whole heads dealt one by one, the first XCD moving on by one every eight heads, as long as every XCD gets three
    // or more; the heads that are left over, or all of fewer, in runs of a few blocks.  For launches whose XCDs cannot
    // help each other: a head's class sets how long its items are and is not known here, and heads in a row
    // (ORDER_HEADS) put heads of one class on one XCD.  Heads in a row / dealt, us: 24 heads of 4109 tokens, the first
    // twelve dense, head_dim 128, 273 / 219; 48 of 17776, likewise, 64, 4393 / 3466; 8 of 16384, one of them dense,
    // 128, 821 / 676.  Classes in turn, where a row is even by itself: 159 / 161, 2306 / 2273 and 517 / 534; 16 of 4109
    // (runs of blocks: the price of a tile in every L2), 131 / 139.
    ORDER_DEALT = 2
};

// far: the heads in work do not fit the memory-side cache; queued: XCDs with nothing left help the others.
inline int item_order(bool far, bool queued, bool dense) { return far ? ORDER_EIGHTHS : queued || dense ? ORDER_HEADS : ORDER_DEALT; }

struct Queues {
    int BH, nVB, nTB, order, per_xcd, whole, shift;
    RF_BOTH Queues(int heads, int video_blocks, int text_blocks, int item_order)
        : BH(heads), nVB(video_blocks), nTB(text_blocks), order(item_order),
          per_xcd(((item_order == ORDER_HEADS ? video_blocks * heads : video_blocks) + 7) >> 3),
          whole(heads >= 24 ? heads >> 3 : 0), shift(0) {
        // runs of four blocks share more tiles through an XCD's L2 than single ones (1-5 %), if there are enough of them
        const int rest = (BH - 8 * whole) * nVB;
        shift = rest >= 256 ? 2 : rest >= 128 ? 1 : 0;
    }
    RF_BOTH int long_items(int x) const { return (nTB * BH - x + 7) >> 3; }
    // ordinals of each head (ORDER_EIGHTHS), or items of all heads
    RF_BOTH int share(int x) const {
        if (order == ORDER_DEALT) {
            const int rest = (BH - 8 * whole) * nVB, cycle = 8 << shift, run = 1 << shift;
            const int last = rest % cycle - x * run;
            return whole * nVB + rest / cycle * run + (last < 0 ? 0 : last < run ? last : run);
        }
        const int left = (order == ORDER_HEADS ? nVB * BH : nVB) - x * per_xcd;
        return left < 0 ? 0 : (left < per_xcd ? left : per_xcd);
    }
    RF_BOTH int items(int x) const { return long_items(x) + (order == ORDER_EIGHTHS ? share(x) * BH : share(x)); }
    // head and position in its block order of the item-th item of queue x
    RF_BOTH void locate(int item, int x, int* bh, int* ordinal) const {
        const int longs = long_items(x), j = item - longs;
        if (j < 0) {
            const int i = item * 8 + x;
            *bh = i / nTB;
            *ordinal = i % nTB;
        } else if (order == ORDER_HEADS) {
            const int i = x * per_xcd + j;
            *bh = i / nVB;
            *ordinal = nTB + i % nVB;
        } else if (order == ORDER_DEALT) {
            const int group = j / nVB;
            if (group < whole) {
                *bh = 8 * group + ((x - group) & 7);
                *ordinal = nTB + j - group * nVB;
            } else {
                const int k = j - whole * nVB, i = ((((k >> shift) << 3) + x) << shift) + (k & ((1 << shift) - 1));
                *bh = 8 * whole + i / nVB;
                *ordinal = nTB + i % nVB;
            }
        } else {
            const int n = share(x);
            *bh = j / n;
            *ordinal = nTB + x * per_xcd + j % n;
        }
    }
};

}  // namespace rf
