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
    // Whole heads dealt one by one (see dealt_head), as long as every XCD gets three or more; the heads that are left
    // over, or all of fewer, in runs of a few blocks.  For launches whose XCDs cannot
    // help each other: a head's class sets how long its items are and is not known here, and heads in a row
    // (ORDER_HEADS) put heads of one class on one XCD.  Heads in a row / dealt, us: 24 heads of 4109 tokens, the first
    // twelve dense, head_dim 96, 214 / 174; 48 of 17776, likewise, 64, 4247 / 3359; 8 of 16384, one of them dense,
    // 64, 599 / 437.  Classes in turn, where a row is even by itself: 128 / 129, 2333 / 2308 and 338 / 374 (runs of
    // blocks: the price of a tile in every L2); 16 of 4109 at 64, 69 / 72.
    ORDER_DEALT = 2
};

// far: the heads in work do not fit the memory-side cache; queued: XCDs with nothing left help the others, which comes
// too late where each has a head or two (8 heads of 16384, one of them dense, head_dim 128, 256 rows: 829 us with heads
// in a row, 686 by eighths; classes in turn 532 and 555; 24 of 17776 and more, either mix: a row 2-5 % faster, up to 8 %
// slower with the first half dense).  From the grid: as long as every workgroup has a CU to itself it does not matter
// which XCD has the longer ones.
inline int item_order(bool far, bool queued, bool dense, int heads, long long items) {
    if (far) return ORDER_EIGHTHS;
    if (dense) return ORDER_HEADS;
    if (queued) return heads < 16 ? ORDER_EIGHTHS : ORDER_HEADS;
    return items <= 256 ? ORDER_HEADS : ORDER_DEALT;
}

// Which of the group-th eight heads XCD x takes.  Classes often alternate from head to head with a period of two, three
// or four, and the same place in every eight would give an XCD heads of one class (period two, four) while any shift by
// a place would (period three).  So the three permutations in turn keep a head's place modulo three and move it by three:
// no XCD has three heads of one parity, and of three heads in turn each has one of each.
RF_BOTH int dealt_head(int group, int x) {
    const int turn = group % 3;
    // octal digits, place of XCD 0 last:  76543210, 10276543 (x -> x + 3), 43210576 (x -> x - 3)
    const unsigned places = turn == 0 ? 076543210u : turn == 1 ? 010276543u : 043210576u;
    return static_cast<int>(places >> (3 * x)) & 7;
}

// MAY_DEAL: the order may be ORDER_DEALT.  The kernels that run from queues never deal, and carry no code for it (it
// costs them registers, and a per cent of time).
template <bool MAY_DEAL>
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
    RF_BOTH bool dealt() const { return MAY_DEAL && order == ORDER_DEALT; }
    RF_BOTH int long_items(int x) const { return (nTB * BH - x + 7) >> 3; }
    // ordinals of each head (ORDER_EIGHTHS), or items of all heads
    RF_BOTH int share(int x) const {
        if (dealt()) {
            const int rest = (BH - 8 * whole) * nVB, run = 1 << shift;
            const int last = (rest & (8 * run - 1)) - x * run;
            return whole * nVB + (rest >> (3 + shift) << shift) + (last < 0 ? 0 : last < run ? last : run);
        }
        const int left = (order == ORDER_HEADS ? nVB * BH : nVB) - x * per_xcd;
        return left < 0 ? 0 : (left < per_xcd ? left : per_xcd);
    }
    // (no queue has more than the first)
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
        } else if (dealt()) {
            if (j < whole * nVB) {
                const int group = j / nVB;
                *bh = 8 * group + dealt_head(group, x);
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

// Keys split four ways: whether each half of a 64-row block can be a workgroup with a CU to itself.  items: of the fullest XCD.
RF_BOTH bool halves_have_cus(int items) {
    constexpr int kCUsPerXCD = 32;  // MI355X
    return 2 * items <= kCUsPerXCD;
}

}  // namespace rf
