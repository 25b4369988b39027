// Block-sparse attention forward for RainFusion's head patterns (Eq. 1-5; Fig. 2a), gfx950.
//
// Work item = one query block (64, 128, 256 or 384 rows) of one head; one workgroup per item in launches of a few
// rounds, otherwise a resident set of workgroups that takes items from per-XCD queues (rf_queues.h says which XCD takes
// which).  For its item a workgroup reads the head's class on the device, walks that class's list of 64-key tiles
// (skipped tiles cost no traffic), loads K and V tiles global -> LDS one tile ahead without staging registers, forms
// the transposed score tile with bf16 MFMA, runs the online softmax in fp32 with exp2, and accumulates O^T = V^T P^T with bf16
// MFMA.  In tiles flagged partial the token-level predicate of the pattern is re-applied to each
// score.
#include <algorithm>
#include <cfloat>
#include <mutex>
#include <type_traits>

#include "rf_band.h"
#include "rf_device.h"
#include "rf_queues.h"

namespace rf {

// How a query block finds its key tiles.
enum : int {
    MODE_ALL = 0,      // every key tile of the sequence in order (dense heads)
    MODE_COMPACT = 1,  // every tile of the compacted key sequence; rows go through the index table (Eq. 5)
    MODE_LISTED = 2,   // the CSR list of the head's pattern; partial tiles re-apply the predicate on a table of key attributes
    MODE_BAND = 3,     // the same for a band over groups of consecutive rows (Spatial; Temporal in position-major
                       // order), where a query keeps one run of key indices (then the text keys): no table
    MODE_BAND_GATHER = 4  // MODE_BAND on rows that go through the index table (position-major order without a copy)
};
constexpr bool gathers(int mode) { return mode == MODE_COMPACT || mode == MODE_BAND_GATHER; }
constexpr bool has_list(int mode) { return mode == MODE_LISTED || mode == MODE_BAND || mode == MODE_BAND_GATHER; }
constexpr bool is_band(int mode) { return mode == MODE_BAND || mode == MODE_BAND_GATHER; }

// Which part of its tile a wavefront works at raised priority.  The wavefronts of a SIMD leave the barrier together; at
// one priority they form their scores together and then want the vector unit together.  One that forms scores going
// before one in its softmax (and one in P V too) staggers them.
enum : int { RAISE_NONE = 0, RAISE_SCORES = 1, RAISE_PRODUCTS = 2, RAISE_SOFTMAX = 3 };
// Measured with classes in turn, us, "before" being the kernels without priorities, but in the softmax of the queued eight
// wavefronts at head_dim 128 (two runs differ by half a per cent).  Taken is the fastest choice that leaves no size slower
// than before by more than that, but one: of 250 drawn sizes 29 heads of 11020, below, where boxes give 0.5 to 1.6 %.
//   keys split four ways: before / none / scores / both products, head_dim 128, 6 heads of 960 21.6 / 21.1 / 20.4 / 20.5, 10 of
//     3584 82.3 / 80.7 / 79.9 / 80.0; head_dim 96, 6 of 960 18.5 / 17.9 / 17.3 / 17.3
//   two ways, head_dim 64: 3 of 34600 with 256 text tokens 660 / 659 / 657 / 678 (all of them Textural 704 / 704 / 703 / 734,
//     Spatial 636 / 631 / 630 / 622), 24 of 4109 89.2 / 87.6 / 87.3 / 88.8, 1 of 52200 466 / 460 / 461 / 447; head_dim 96, 24 of
//     4109 123.3 / 121.3 / 120.6 / 119.8, 34 of 5577 339.9 / 337.2 / 337.2 / 333.1; head_dim 128, 20 of 1890 48.5 / 47.4 /
//     48.3 / 48.9, 32 of 4096 187.3 / 184.9 / 190.7 / 188.6, 14 of 6357 207.9 / 204.2 / 204.8 / 201.7
//   128 rows, head_dim 64, the last with both but in the compacted walk: 48 of 17776 2213 / 2182 / 2182 / 2155 / 2166, 29 of 11020
//     with bands of 0.13, stride 4 and 256 text tokens 389 / 386 / 391 / 395 / 392; head_dim 96: 24 of 4109 161.7 / 160.6 / 163.5
//     / 164.3, 24 of 17776 1569 / 1557 / 1549 / 1546; head_dim 128: 20 of 5278 221.5 / 221.3 / 224.1 / 223.7, 24 of 17776 2008 /
//     1994 / 1986 / 1985
//   256 rows from the grid: head_dim 96, 24 of 4109 168.7 / 169.4 / 162.5 / 163.0; head_dim 128, 48 of 2040 80.9 / 81.1 / 80.5 /
//     80.4
//   256 rows from queues, before / none / scores / both products / softmax: head_dim 64, 24 of 86626 23175 / 22758 / 22712 / 22248
//     / 22943, 6 of 20800 801 / 786 / 766 / 730 / 766; head_dim 96, 32 of 16384 1644 / 1634 / 1647 / 1647 / 1617; head_dim 128, 32 of
//     16384 1958 / 1974 / 1970 / 1964 / 1956, 8 of 119056 25106 / 25206 / 25181 / 25231 / 24980
//   384 rows, before / none / scores / both products / softmax: head_dim 64, 4 of 27375 619 / 601 / 622 / 624 / 604; head_dim 96,
//     12 of 20837 1308 / 1314 / 1279 / 1299 / 1352; head_dim 128, 32 of 16384 2010 / 1992 / 1960 / 1954 / 2029, 8 of 119056 23332 /
//     23076 / 22982 / 23029 / 23869
constexpr int raise_of(int D, int NW, int KS, bool queued, int mode) {
    if (KS == 2) return D == 64 ? RAISE_SCORES : D == 96 ? RAISE_PRODUCTS : RAISE_NONE;
    if (KS == 4) return RAISE_PRODUCTS;
    if (D == 64) return NW == 12 ? RAISE_NONE : !queued && mode == MODE_COMPACT ? RAISE_SCORES : RAISE_PRODUCTS;
    if (NW == 4) return RAISE_NONE;
    return NW == 8 && queued ? RAISE_SOFTMAX : RAISE_SCORES;
}

// K/V tiles kept in flight ahead of the one being consumed.  Two (with a third buffer) measured no
// faster than one at any shape: the loads are not what the wavefronts wait for.
#ifndef RF_TILES_AHEAD
#define RF_TILES_AHEAD 1
#endif

// NW: wavefronts that share a tile.  KS > 1: the workgroup is KS groups of NW wavefronts on the same query
// rows, each with its own tiles (see attend).
template <int D, int NW, int KS = 1, int TILES_AHEAD = RF_TILES_AHEAD>
struct AttnSmem {
    using ST = DirectTile<D, NW>;
    // K/V tiles resident at a time: the one being consumed plus AHEAD on their way
    static constexpr int AHEAD = TILES_AHEAD;
    static constexpr int DEPTH = AHEAD + 1;
    static constexpr int SIDE_SLOTS = DEPTH + 1;  // side data runs one tile further ahead than K/V
    static constexpr int K_OFF = 0;
    static constexpr int V_OFF = DEPTH * ST::K_BYTES;
    static constexpr int TILE_BYTES = V_OFF + DEPTH * ST::V_BYTES;  // of one group
    // KS > 1: at the end every group leaves its rows' references and denominators where its side data was and
    // its share of the output, fp32, where its tiles were (see attend)
    static constexpr int PART_BYTES = NW * D * 32 * 4;
    static constexpr int GROUP_BYTES = KS > 1 && PART_BYTES > TILE_BYTES ? PART_BYTES : TILE_BYTES;
    static constexpr int SIDE_OFF = KS * GROUP_BYTES;  // per group a ring of 64-int slots: key indices or key attributes
    static constexpr int STAT_BYTES = KS > 1 ? NW * 2 * 32 * 4 : 0;
    static constexpr int SIDE_BYTES = SIDE_SLOTS * kTileK * 4 > STAT_BYTES ? SIDE_SLOTS * kTileK * 4 : STAT_BYTES;
    static constexpr int ITEM_OFF = SIDE_OFF + KS * SIDE_BYTES;  // two ints: the work item just taken
    static constexpr int BYTES = ITEM_OFF + 16;
    static_assert(K_OFF % 256 == 0 && V_OFF % 256 == 0 && ST::K_BYTES % 256 == 0 && ST::V_BYTES % 256 == 0,
                  "tile buffers must start at multiples of 256 bytes (see DirectTile::k_address)");
};

struct QueryBlock {
    int bh, qb, cls;
    int list;                    // MODE_LISTED: which of the plan's lists (a class, or Temporal position-major)
    const int32_t* row_token;    // null, or: row of the walked order -> token (queries are gathered, O scattered)
    const unsigned char* kbase;  // K and V rows of the key sequence walked (the head's, or its compacted copy)
    const unsigned char* vbase;
    // tensor row of walked index n = n + (n < Nv ? video_shift : text_shift); both 0 unless the text
    // tokens come first in the tensors, and 0 when kbase/vbase are packed copies (already in walked order)
    int video_shift, text_shift;
    const int32_t* cols;  // MODE_LISTED: this query block's tile entries
    int first;            // entry (tile, for the unlisted walks) the cyclic walk starts at
    int ntiles;           // key tiles to visit
    int* sweep;           // null, or: where this workgroup publishes how far its walk has come (see join_sweep)
    int sweep_tag;        // which key sequence the published tile index refers to
    int keyN;             // length of the key sequence walked (N, or Nc when compacted)
    BandTiles band;       // COMPUTED, banded modes: what cols would say
};

// Workgroups of one XCD share that XCD's L2, so they should walk the same key tiles at the same time.
// Items are handed out one by one as workgroups finish, so a workgroup that starts an item finds the
// others somewhere in the middle of theirs: it joins them.  Every workgroup publishes, every few
// tiles, the tile its walk has reached (with a tag naming the head and the key sequence) in one of
// kSweepSlots words per XCD next to the work-queue counters (an XCD is usually on two or three heads
// at a time: the slot is the head's index modulo kSweepSlots); a starting workgroup whose item walks
// the same sequence begins its cyclic walk at that tile if the tile is in its list.  This only moves
// where the walk starts: every tile of the list is still visited exactly once.
constexpr int kSweepTileBits = 18, kSweepTileMask = (1 << kSweepTileBits) - 1;  // N <= 2^24 tokens: tile indices below 2^18
constexpr int kSweepSlots = 8, kQueueWords = 8 + 8 * kSweepSlots;
static_assert(kQueueWords * 4 <= RF_ATTENTION_MIN_WORKSPACE, "counters and sweep words live in the minimum workspace");
__device__ __forceinline__ int* sweep_word(int* queue, int xcd, int bh) { return queue + 8 + xcd * kSweepSlots + (bh & (kSweepSlots - 1)); }

// exp2 arguments may exceed 0 by at most this much before the running reference is moved: the
// softmax is invariant to the reference, so a stale one only costs range, which fp32/bf16 have.
constexpr float kRescaleSlack = 8.f;

}  // namespace rf

#include "rf_attn_wide.h"

namespace rf {

// QH: 32-query halves a wavefront owns (1, or 2: every K and V slab read from LDS then feeds two MFMAs).
// KS: groups of NW wavefronts that split the walk (group g takes its tiles g, g + KS, ... into LDS of its own
// and keeps a softmax of its own); the groups' results are added up at the end.
template <int D, int NW, int MODE, int QH = 1, int KS = 1, int TILES_AHEAD = RF_TILES_AHEAD, int RAISE = RAISE_NONE, bool COMPUTED = false, bool FEW = false>
__device__ __forceinline__ void attend(const AttnArgs& a, const DevicePlan& pl, const QueryBlock& qk, unsigned char* smem_all) {
    constexpr int BQ = 32 * NW * QH;
    using ST = DirectTile<D, NW>;
    using SM = AttnSmem<D, NW, KS, TILES_AHEAD>;
    constexpr int DEPTH = SM::DEPTH;
    const int group = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / (64 * NW));
    unsigned char* smem = smem_all + group * SM::GROUP_BYTES;
    // how many slabs ahead of their MFMAs the LDS operand reads run: with two halves every slab feeds two
    // MFMAs and the registers are all in use, and two measured best (dense CogVideoX-shaped layer 4.25 ->
    // 3.99 ms against the depths of the one-half loop); twelve wavefronts at head_dim 128 and keys split two ways at 96 (FEW)
    // have 168 registers each, which the loops fit (but for a spill or two off the common path) at depth two
    constexpr bool kTight = (NW == 12 && D == 128) || FEW;
    constexpr int AK = (QH == 2 || kTight) ? 2 : kAheadK, AV = (QH == 2 || kTight) ? 2 : kAheadV;
    const int tid = threadIdx.x - group * (64 * NW), lane = tid & 63, wave = tid >> 6, hf = lane >> 5, m = lane & 31;
    const int N = pl.N, keyN = qk.keyN;
    // opaque, or the loop may load it anew from the arguments, and a scalar load in flight turns its LDS waits into
    // waits for every read
    int Nv = pl.Nv;
    asm volatile("" : "+s"(Nv));
    const int ntiles = KS == 1 ? qk.ntiles : (qk.ntiles - group + KS - 1) / KS;  // of this group
    const int nsteps = (qk.ntiles + KS - 1) / KS;                                // of the longest group
    // per-key side data staged through LDS two tiles ahead: the token index of each key of the
    // compacted sequence, or the pattern attribute (frame / position / kept flag) of each key
    const int32_t* side_src = MODE == MODE_COMPACT ? pl.cidx : (MODE == MODE_BAND_GATHER ? pl.pm_token : (MODE == MODE_LISTED ? pl.attr[qk.list] : nullptr));
    int* side = reinterpret_cast<int*>(smem_all + SM::SIDE_OFF + group * SM::SIDE_BYTES);

    const unsigned char* Kh = qk.kbase;
    const unsigned char* Vh = qk.vbase;
    const uint16_t* Qh = a.Q + static_cast<size_t>(qk.bh) * N * D;

    auto row_of_position_major = [&](int n) {
        return position_major_row(n, pl.group_rows[kListTemporalPM], pl.group_rows[RF_SPATIAL], Nv, pl.video_shift, pl.text_shift);
    };
    // this lane's queries, one per half
    int qrow[QH], qtok[QH];
    bf16x8 qf[QH][D / 16];
    uint32_t q_lo[QH], q_span[QH];
#pragma unroll
    for (int h = 0; h < QH; ++h) {
        qrow[h] = qk.qb * BQ + wave * (32 * QH) + 32 * h + m;  // row of the walked order
        const int qrow_c = min(qrow[h], N - 1);
        qtok[h] = COMPUTED && MODE == MODE_BAND_GATHER ? row_of_position_major(qrow_c) : (has_list(MODE) && qk.row_token) ? qk.row_token[qrow_c]
                                                        : qrow_c + (qrow_c < Nv ? pl.video_shift : pl.text_shift);
        load_q_frags<D>(Qh, qtok[h], hf, qf[h]);
        // a key of attribute x is kept iff x + q_lo <= q_span (unsigned); text queries keep everything
        if (is_band(MODE)) {
            // attribute = key index: the rows of the groups within the radius of the query's
            const int group_rows = pl.group_rows[qk.list], r = pl.radius[qk.list];
            q_lo[h] = qrow_c < Nv ? static_cast<uint32_t>((r - qrow_c / group_rows) * group_rows) : 0x3fffffffu;
            q_span[h] = qrow_c < Nv ? static_cast<uint32_t>((2 * r + 1) * group_rows - 1) : 0x7ffffffeu;
        } else {
            int q_attr = 0, q_rad = 0x3fffffff;
            if (MODE == MODE_LISTED) {
                // Spatial / Temporal compare the query's frame / position with the key's; the Textural
                // table is 0 on kept keys and 1 on dropped ones, compared against 0 with radius 0
                if (qk.cls != RF_TEXTURAL) q_attr = side_src[qrow_c];
                if (qrow_c < Nv) q_rad = pl.radius[qk.list];
            }
            q_lo[h] = static_cast<uint32_t>(q_rad - q_attr);
            q_span[h] = 2u * static_cast<uint32_t>(q_rad);
        }
    }

    f32x16 oacc[QH][D / 32];
#pragma unroll
    for (int h = 0; h < QH; ++h)
#pragma unroll
        for (int db = 0; db < D / 32; ++db) oacc[h][db] = f32x16{0};
    // m_ref: reference subtracted inside exp2, in the units of its argument (score times c); kNoReference until it has
    // been taken from real scores of this row.  c is below 1, so any finite score outgrows that, and what was
    // accumulated relative to it (nothing) is scaled by exp2 of it: 0.  l_run: this lane's share of the softmax denominator
    constexpr float kNoReference = -FLT_MAX;
    float m_ref[QH], l_run[QH];
#pragma unroll
    for (int h = 0; h < QH; ++h) {
        m_ref[h] = kNoReference;
        l_run[h] = 0.f;
    }
    const float c = a.scale_log2;

    ST st;
    st.init(tid);
    int side_reg = 0;

    // FEW: some numbers too many for the registers, which are formed again from the thread's where they are wanted: its place
    // in the wavefront, 8 * hf, its row.
    auto thread_again = [&]() {
        int thread = tid;
        asm volatile("" : "+v"(thread));
        return thread;
    };
    auto lane_of_list = [&]() { return FEW ? thread_again() & 63 : lane; };
    auto half_of_mask = [&]() { return FEW ? (thread_again() & 32) >> 2 : 8 * hf; };
    // Tile entries of a listed query block are read 64 at a time, one per lane, and handed out with
    // v_readlane: no scalar-load latency in the loop.  ent_cur covers [ent_base, ent_base + 64).
    int ent_cur = 0, ent_nxt = 0, ent_base = 0;
    // COMPUTED: no load of a list or a table between the workgroup's start and its first tile
    auto load_entries = [&](int from) {
        const int j = min((from + lane_of_list()) * KS + group, qk.ntiles - 1) + qk.first;  // the walk starts at entry qk.first and wraps
        return COMPUTED && is_band(MODE) ? qk.band.entry(j, keyN, Nv) : qk.cols[j < qk.ntiles ? j : j - qk.ntiles];
    };
    if (has_list(MODE) && ntiles > 0) {
        ent_cur = load_entries(0);
        ent_nxt = load_entries(64);
    }
    // entries must be asked for in increasing t
    auto entry_of = [&](int t) -> int {
        if (has_list(MODE)) {
            if (t >= ent_base + 64) {
                ent_base += 64;
                ent_cur = ent_nxt;
                ent_nxt = load_entries(ent_base + 64);
            }
            return __builtin_amdgcn_readlane(ent_cur, t - ent_base);
        }
        int tile = t * KS + group + qk.first;  // the walk starts at tile qk.first and wraps
        if (tile >= qk.ntiles) tile -= qk.ntiles;
        return tile | ((tile + 1) * kTileK > keyN ? (RF_PLAN_PARTIAL | kTileBoundary) : 0);
    };
    // side data is needed for every gathered tile, and for partial tiles masked by the table
    auto wants_side = [&](int entry) { return gathers(MODE) || (MODE == MODE_LISTED && (entry & RF_PLAN_PARTIAL)); };
    auto load_side = [&](int entry, bool first = false) {
        if (!wants_side(entry)) return;
        const int k0 = (entry & kTileIndexMask) * kTileK;
        if (COMPUTED && first && MODE == MODE_BAND_GATHER) {  // (a load is cheaper than the arithmetic, but for its latency)
            if (tid < kTileK) side_reg = row_of_position_major(min(k0 + tid, keyN - 1));
            return;
        }
        if (tid < kTileK) side_reg = side_src[min(k0 + tid, keyN - 1)];
    };
    auto stash_side = [&](int t, int entry) {
        if (!wants_side(entry)) return;
        if (tid < kTileK) side[(t % SM::SIDE_SLOTS) * kTileK + tid] = side_reg;
    };
    auto k_lds = [&](int t) { return smem + SM::K_OFF + (t % DEPTH) * ST::K_BYTES; };
    auto v_lds = [&](int t) { return smem + SM::V_OFF + (t % DEPTH) * ST::V_BYTES; };
    // three workgroups of four wavefronts per CU at head_dim 96 have 168 registers each, too few for lane offsets of 64 bits
    constexpr bool kNarrow = FEW || (D == 96 && NW == 4 && KS == 1 && MODE == MODE_BAND);
    auto fetch_some = [&](auto with_v, auto with_k, int t, int entry) {
        constexpr bool WV = decltype(with_v)::value, WK = decltype(with_k)::value;
        const int k0 = (entry & kTileIndexMask) * kTileK;
        if (gathers(MODE)) {
            const int* idx = side + (t % SM::SIDE_SLOTS) * kTileK;
            st.template issue<WV, WK, false, FEW>(Kh, Vh, k_lds(t), v_lds(t), [&](int row) { return idx[row]; });
        } else if (k0 + kTileK <= keyN && !(qk.text_shift != 0 && k0 < Nv && k0 + kTileK > Nv)) {
            // full tile of consecutive tensor rows: everything but the tile origin is loop invariant
            const int r0 = k0 + (k0 < Nv ? qk.video_shift : qk.text_shift);
            const size_t origin = static_cast<size_t>(r0) * (2 * D);
            st.template issue_consecutive<WV, WK, kNarrow>(Kh + origin, Vh + origin, k_lds(t), v_lds(t));
        } else {
            st.template issue<WV, WK, true>(Kh, Vh, k_lds(t), v_lds(t), [&](int row) {
                const int n = min(k0 + row, keyN - 1);
                return n + (n < Nv ? qk.video_shift : qk.text_shift);
            });
        }
    };
    auto fetch_tile = [&](int t, int entry) { fetch_some(std::true_type{}, std::true_type{}, t, entry); };

    // S^T of tile t (64 keys x this lane's query of each half), predicate applied where the tile is partial
    auto scores = [&](int t, int entry, bool need_mask, f32x16 (&s)[QH][2]) {
        if (QH == 1) {
            st.template scores<AK>(st.k_address(k_lds(t)), qf[0], s[0]);
        } else {
            // as DirectTile::scores, every K slab feeding one MFMA per half
            constexpr int NQK = 2 * (D / 16);
            const uint32_t ka = st.k_address(k_lds(t));
            bf16x8 frag[NQK];
#pragma unroll
            for (int i = 0; i < AK; ++i) frag[i] = st.k_frag(ka, i & 1, i >> 1);
#pragma unroll
            for (int h = 0; h < QH; ++h) {
                s[h][0] = f32x16{0};
                s[h][1] = f32x16{0};
            }
#pragma unroll
            for (int j = 0; j < NQK; ++j) {
                if (j + AK < NQK) frag[j + AK] = st.k_frag(ka, (j + AK) & 1, (j + AK) >> 1);
#pragma unroll
                for (int h = 0; h < QH; ++h) {
                    s[h][j & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[j], qf[h][j >> 1], s[h][j & 1], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        if (need_mask) {
            const int k0 = (entry & kTileIndexMask) * kTileK;
            const int* al = side + (t % SM::SIDE_SLOTS) * kTileK;
            const bool band_only = has_list(MODE) && !(entry & kTileBoundary);  // all 64 keys are video tokens
            // element (kb2, 8*u + i) of this lane is key  8*hf + c  of the tile,  c = 32*kb2 + 16*u + i
            typedef __attribute__((address_space(3))) const u32x4 lds_u32x4;
#pragma unroll
            for (int h = 0; h < QH; ++h) {
                auto drop = [&](auto keeps) {
#pragma unroll
                    for (int kb2 = 0; kb2 < 2; ++kb2)
#pragma unroll
                        for (int r = 0; r < 16; ++r) {
                            s[h][kb2][r] = keeps(32 * kb2 + 16 * (r >> 3) + (r & 7)) ? s[h][kb2][r] : -INFINITY;
                            if ((r & 3) == 3) __builtin_amdgcn_sched_barrier(0);  // few comparisons' results at a time
                        }
                };
                if (is_band(MODE)) {
                    // keys lo .. hi of the tile (counted from this half's first) are kept.  Where only one end of the
                    // run lies in the tile for every row of the wavefront, one comparison with a constant decides.
                    const int first = half_of_mask();
                    const int lo = -static_cast<int>(q_lo[h]) - k0 - first, hi = lo + static_cast<int>(q_span[h]);
                    if (band_only && __builtin_amdgcn_ballot_w64(hi < kTileK - 1) == 0) drop([&](int c) { return c >= lo; });
                    else if (band_only && __builtin_amdgcn_ballot_w64(lo > 0) == 0) drop([&](int c) { return c <= hi; });
                    else {
                        const int text = band_only ? kTileK : Nv - k0 - first, end = keyN - k0 - first;
                        drop([&](int c) { return (((c >= lo) & (c <= hi)) | (c >= text)) & (c < end); });
                    }
                } else if (MODE != MODE_LISTED) {
                    const int end = keyN - k0 - 8 * hf;
                    drop([&](int c) { return c < end; });
                } else {
#pragma unroll
                    for (int kb2 = 0; kb2 < 2; ++kb2)
#pragma unroll
                        for (int u = 0; u < 2; ++u) {
                            const int base = 32 * kb2 + 16 * u + 8 * hf;
                            uint32_t at[8];
                            const u32x4 a0 = *(lds_u32x4*)(uintptr_t)ST::lds_offset(reinterpret_cast<const unsigned char*>(al + base));
                            const u32x4 a1 = *(lds_u32x4*)(uintptr_t)ST::lds_offset(reinterpret_cast<const unsigned char*>(al + base + 4));
#pragma unroll
                            for (int i = 0; i < 4; ++i) {
                                at[i] = a0[i];
                                at[4 + i] = a1[i];
                            }
#pragma unroll
                            for (int i = 0; i < 8; ++i) {
                                const int kidx = k0 + base + i;
                                bool ok = band_only || kidx < keyN;
                                ok = ok & ((at[i] + q_lo[h] <= q_span[h]) | (!band_only && kidx >= Nv));
                                s[h][kb2][8 * u + i] = ok ? s[h][kb2][8 * u + i] : -INFINITY;
                            }
                        }
                }
            }
        }
    };
    // A partial tile of the block may lie inside or outside the run of keys of this wavefront's rows altogether
    // (the block has many times as many rows): 0 = no score needs the predicate, 1 = it has to be applied,
    // 2 = nothing is kept.
    auto tile_kind = [&](int entry) -> int {
        if (!(entry & RF_PLAN_PARTIAL)) return 0;
        if (!is_band(MODE) || (entry & kTileBoundary)) return 1;
        const int k0 = (entry & kTileIndexMask) * kTileK;
        bool all = true, none = true;
#pragma unroll
        for (int h = 0; h < QH; ++h) {
            const int lo = -static_cast<int>(q_lo[h]) - k0, hi = lo + static_cast<int>(q_span[h]);
            all = all & (lo <= 0) & (hi >= kTileK - 1);
            none = none & ((hi < 0) | (lo >= kTileK));
        }
        return __builtin_amdgcn_ballot_w64(!all) == 0 ? 0 : (__builtin_amdgcn_ballot_w64(!none) == 0 ? 2 : 1);
    };

    // O^T += V^T P^T for tile t, P (bf16) in pf
    bf16x8 pf[QH][4];
    auto accumulate = [&](int t) {
        const uint32_t va = st.v_address(v_lds(t));
        // consecutive MFMAs go to different accumulators (channel blocks, halves): no back-to-back
        // dependence; operand reads kAheadV slabs ahead, order fenced as for the scores
        constexpr int NPV = 4 * (D / 32), NDB = D / 32;
        bf16x8 frag[NPV];
#pragma unroll
        for (int i = 0; i < AV; ++i) frag[i] = ST::v_frag(va, i % NDB, i / NDB);
#pragma unroll
        for (int j = 0; j < NPV; ++j) {
            if (j + AV < NPV) frag[j + AV] = ST::v_frag(va, (j + AV) % NDB, (j + AV) / NDB);
#pragma unroll
            for (int h = 0; h < QH; ++h) {
                oacc[h][j % NDB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[j], pf[h][j / NDB], oacc[h][j % NDB], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    // Software pipeline.  While tile t is consumed, the loads of tiles t+1 .. t+AHEAD are in flight
    // or landed, and the side data of tile t+DEPTH is on its way to its ring slot (one tile further,
    // because the loads of a compacted tile take their row indices from it).  e[i] = entry of tile t+i.
    // AHEAD = 0 (one buffer for K and one for V): K(t+1) is loaded while P V of tile t runs, V(t) while
    // the scores and the softmax of tile t do; each has a barrier that says its buffer is free and the other's full.
    // With one wavefront to a group (kOwnTiles) nobody else reads its tiles, and its own waits say when a buffer is free or
    // full: K(t+1) is asked for as soon as the scores of tile t are formed, V(t+1) after P V, and there is no barrier.  Where
    // rows are gathered they are found once, for K, and kept for V.  The side data of tile t+2 is asked for before K(t+1) and
    // put in its slot before V(t+1) is asked for: the compiler, which does not see the tile loads, waits there for every load,
    // and K(t+1), wanted next, is the only other one.  (Put there after the scores, it waited for V(t) as well.)
    // All heads Temporal, the speed of the loop with barriers = 1: rows found for K and V each 1.077 on the geometric mean of 361
    // drawn sizes and three head_dims, down to 0.96 at head_dim 96 (3 heads of 344 tokens, 10.4 us), now 1.212, none below 0.996.
    constexpr int AHEAD = SM::AHEAD;
    constexpr bool kOwnTiles = NW == 1;
    static_assert(!kOwnTiles || (AHEAD == 0 && ST::EVEN), "the waits of the loop count whole tensors");
    int e[DEPTH + 1 + (kOwnTiles ? 1 : 0)] = {};
    uint32_t row_off[ST::PER_WAVE];  // kOwnTiles, gathered rows: of K(t), then V(t)
    auto fetch_k = [&](int t, int entry) {
        if constexpr (kOwnTiles && gathers(MODE)) {
            const int* idx = side + (t % SM::SIDE_SLOTS) * kTileK;
            st.find_rows(row_off, [&](int row) { return idx[row]; });
            st.template issue_rows<false>(Kh, k_lds(t), row_off);
        } else fetch_some(std::false_type{}, std::true_type{}, t, entry);
    };
    auto fetch_v = [&](int t, int entry) {
        if constexpr (kOwnTiles && gathers(MODE)) st.template issue_rows<true>(Vh, v_lds(t), row_off);
        else fetch_some(std::true_type{}, std::false_type{}, t, entry);
    };
#pragma unroll
    for (int i = 0; i < DEPTH; ++i)
        if (i < ntiles) {
            e[i] = entry_of(i);
            load_side(e[i], true);
            if (AHEAD == 0 && !gathers(MODE)) fetch_k(i, e[i]);
            stash_side(i, e[i]);
        }
    if (AHEAD > 0 || gathers(MODE)) {
        __syncthreads();
        if (AHEAD == 0 && ntiles > 0) fetch_k(0, e[0]);
    }
#pragma unroll
    for (int i = 0; i < AHEAD; ++i)
        if (i < ntiles) fetch_tile(i, e[i]);
    if (kOwnTiles && 1 < ntiles) {
        e[1] = entry_of(1);
        load_side(e[1]);
    }
    ST::template wait_landed<0>();
    __syncthreads();
    // The compiler cannot see the tile loads above, so its own wait for the Q loads, if left inside
    // the loop, would count them out too and wait for the tiles in flight; make it wait here.
#pragma unroll
    for (int h = 0; h < QH; ++h)
#pragma unroll
        for (int cc = 0; cc < D / 16; ++cc) asm volatile("" ::"v"(__builtin_bit_cast(u32x4, qf[h][cc])));

    for (int t = 0; t < nsteps; ++t) {
        // the buffer of tile t+AHEAD held tile t+AHEAD-DEPTH, which every wavefront left before the last barrier
        if (!kOwnTiles && t + DEPTH < ntiles) e[DEPTH] = entry_of(t + DEPTH);
        if constexpr (kOwnTiles) {
            if (t + 1 < ntiles) stash_side(t + 1, e[1]);
            if (t < ntiles) fetch_v(t, e[0]);
        } else if constexpr (AHEAD > 0) {
            if (t + AHEAD < ntiles) fetch_tile(t + AHEAD, e[AHEAD]);
            if (t + DEPTH < ntiles) load_side(e[DEPTH]);
        } else {
            if (t + DEPTH < ntiles) load_side(e[DEPTH]);
            if (t < ntiles) fetch_v(t, e[0]);
        }
        const int e_cur = e[0];
        // every eighth tile, tell the workgroups that start an item on this XCD where this walk is
        if (qk.sweep && (t & 7) == 0 && tid == 0)
            __hip_atomic_store(qk.sweep, (qk.sweep_tag << kSweepTileBits) | (e_cur & kSweepTileMask), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);

        // Online softmax (Eq. 1) in base 2 with 1/sqrt(D) folded into c.  The reference subtracted in
        // the exponent is moved, and the accumulators rescaled, only when a row outgrows it by more
        // than 2^kRescaleSlack (or has none yet): the softmax does not depend on the reference.
        // a group with fewer tiles only keeps step with the others, and so does a wavefront none of whose rows see the tile
        const int kind = KS == 1 || t < ntiles ? tile_kind(e_cur) : 2;
        const bool mine = (KS == 1 && !is_band(MODE)) || kind != 2;
        f32x16 s[QH][2];
        if (kOwnTiles && t < ntiles) ST::wait_all_but_one_tensor();  // K(t) is there, V(t) on its way
        auto form_scores = [&]() {
            if (RAISE == RAISE_SCORES || RAISE == RAISE_PRODUCTS) __builtin_amdgcn_s_setprio(1);
            scores(t, e_cur, is_band(MODE) ? kind == 1 : (e_cur & RF_PLAN_PARTIAL) != 0, s);
            if (RAISE != RAISE_NONE) __builtin_amdgcn_s_setprio(RAISE == RAISE_SOFTMAX ? 1 : 0);
        };
        auto weigh = [&]() {
#pragma unroll
            for (int h = 0; h < QH; ++h) {
                float mt = s[h][0][0];
#pragma unroll
                for (int kb2 = 0; kb2 < 2; ++kb2)
#pragma unroll
                    for (int r = 0; r < 16; ++r) mt = fmaxf(mt, s[h][kb2][r]);
                // the two halves of the wavefront hold different keys of the same 32 queries: their maxima
                // are exchanged only when some lane asks for the reference to move
                if (__builtin_amdgcn_ballot_w64(fmaf(mt, c, -m_ref[h]) > kRescaleSlack) != 0) {
                    mt = fmaxf(mt, other_half(mt));
                    if (mt > -INFINITY) {
                        const float m_new = fmaxf(m_ref[h], mt * c), alpha = fast_exp2(m_ref[h] - m_new);
                        l_run[h] *= alpha;
#pragma unroll
                        for (int db = 0; db < D / 32; ++db)
#pragma unroll
                            for (int r = 0; r < 16; ++r) oacc[h][db][r] *= alpha;
                        m_ref[h] = m_new;
                    }
                }
                // p = exp2(s * c - m_ref) in place
#pragma unroll
                for (int kb2 = 0; kb2 < 2; ++kb2)
#pragma unroll
                    for (int r = 0; r < 16; ++r) s[h][kb2][r] = fast_exp2(fmaf(s[h][kb2][r], c, -m_ref[h]));
                // P is rounded to bf16 for the second MFMA; the denominator sums those same rounded values
                // (two per v_dot2c_f32_bf16), so numerator and denominator of Eq. 2 see identical weights
#pragma unroll
                for (int kb2 = 0; kb2 < 2; ++kb2)
#pragma unroll
                    for (int u2 = 0; u2 < 2; ++u2) {
                        u32x4 w;
                        w.x = pack_bf16(s[h][kb2][8 * u2 + 0], s[h][kb2][8 * u2 + 1]);
                        w.y = pack_bf16(s[h][kb2][8 * u2 + 2], s[h][kb2][8 * u2 + 3]);
                        w.z = pack_bf16(s[h][kb2][8 * u2 + 4], s[h][kb2][8 * u2 + 5]);
                        w.w = pack_bf16(s[h][kb2][8 * u2 + 6], s[h][kb2][8 * u2 + 7]);
                        l_run[h] = add_bf16_pair(add_bf16_pair(add_bf16_pair(add_bf16_pair(l_run[h], w.x), w.y), w.z), w.w);
                        pf[h][2 * kb2 + u2] = as_bf16x8(w);
                    }
            }
            if (RAISE == RAISE_PRODUCTS) __builtin_amdgcn_s_setprio(1);
            else if (RAISE == RAISE_SOFTMAX) __builtin_amdgcn_s_setprio(0);
            if constexpr (AHEAD > 0) accumulate(t);
        };
        if constexpr (kOwnTiles) {
            if (mine) form_scores();
            if (t + 2 < ntiles) {
                e[2] = entry_of(t + 2);
                load_side(e[2]);
            }
            if (t + 1 < ntiles) fetch_k(t + 1, e[1]);
            if (mine) weigh();
            if (t + 1 < ntiles) ST::wait_all_but_one_tensor();  // V(t) is there, K(t + 1) on its way
            else ST::template wait_landed<0>();
            if (mine) accumulate(t);
            e[0] = e[1];
            e[1] = e[2];
            continue;
        }
        if (mine) {  // one block: asked twice, 24 heads of 17776 tokens at head_dim 128 (128 rows) took 2016 us, not 1959
            form_scores();
            weigh();
        }
        if constexpr (AHEAD == 0) {
            ST::template wait_landed<0>();
            if (t + DEPTH < ntiles) stash_side(t + DEPTH, e[DEPTH]);
            __syncthreads();
            if (t + 1 < ntiles) fetch_k(t + 1, e[1]);
            if (mine) accumulate(t);
        }

        // tile t+1 must be in LDS at the barrier; the loads of the tiles after it may stay in flight
        if (AHEAD > 1 && t + AHEAD < ntiles) ST::template wait_landed<AHEAD - 1>();
        else ST::template wait_landed<0>();
        if (AHEAD > 0 && t + DEPTH < ntiles) stash_side(t + DEPTH, e[DEPTH]);
#pragma unroll
        for (int i = 0; i < DEPTH; ++i) e[i] = e[i + 1];
        __syncthreads();
    }
    if (RAISE == RAISE_PRODUCTS) __builtin_amdgcn_s_setprio(0);  // raised for the last tile's P V
    if constexpr (KS > 1) {
        // The groups hold the same rows' results over different keys.  Every group's reference and denominator
        // give the common ones; each group scales its share of the output by them and leaves it in LDS as
        // [chunk of four channels][query], and then adds up 1/KS of the chunks of all groups and stores them.
        static_assert(QH == 1 && (D / 4) % (2 * KS) == 0, "two halves of a wavefront take chunks in turn");
        typedef __attribute__((address_space(3))) float lds_float;
        typedef __attribute__((address_space(3))) f32x4 lds_f32x4;
        auto stat = [&](int g, int which) {
            return (lds_float*)(uintptr_t)(ST::lds_offset(smem_all + SM::SIDE_OFF) + g * SM::SIDE_BYTES + ((wave * 2 + which) * 32 + m) * 4);
        };
        auto part = [&](int g, int chunk) {
            return (lds_f32x4*)(uintptr_t)(ST::lds_offset(smem_all) + g * SM::GROUP_BYTES + wave * (D * 128) + (chunk * 32 + m) * 16);
        };
        const float l_own = l_run[0] + other_half(l_run[0]), m_own = m_ref[0];
        if (hf == 0) {
            *stat(group, 0) = m_own;
            *stat(group, 1) = l_own;
        }
        __syncthreads();
        float m_all = m_own;
#pragma unroll
        for (int g = 0; g < KS; ++g) m_all = fmaxf(m_all, *stat(g, 0));
        float l_all = 0.f;
#pragma unroll
        for (int g = 0; g < KS; ++g) {
            l_all += *stat(g, 1) * fast_exp2(*stat(g, 0) - m_all);
        }
        const float scale = l_all > 0.f ? fast_exp2(m_own - m_all) / l_all : 0.f;
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
                f32x4 w;
#pragma unroll
                for (int r = 0; r < 4; ++r) w[r] = oacc[0][db][4 * rq + r] * scale;
                *part(group, 8 * db + 2 * rq + hf) = w;
            }
        __syncthreads();
        int row = qrow[0], token = qtok[0];
        if (FEW) {  // (gathered rows keep theirs: a load)
            const int thread = thread_again();
            row = qk.qb * BQ + (thread >> 6) * 32 + (thread & 31);
            const int row_c = min(row, N - 1);
            if (!gathers(MODE)) token = has_list(MODE) && qk.row_token ? qk.row_token[row_c] : row_c + (row_c < Nv ? pl.video_shift : pl.text_shift);
        }
        uint16_t* orow = a.O + static_cast<size_t>(qk.bh) * N * D + static_cast<size_t>(token) * D;
#pragma unroll
        for (int i = 0; i < D / 4 / KS / 2; ++i) {
            const int chunk = group * (D / 4 / KS) + 2 * i + hf;
            f32x4 sum = *part(0, chunk);
#pragma unroll
            for (int g = 1; g < KS; ++g) sum += *part(g, chunk);
            u32x2 w;
            w.x = pack_bf16(sum[0], sum[1]);
            w.y = pack_bf16(sum[2], sum[3]);
            if (row < N) *reinterpret_cast<u32x2*>(orow + 4 * chunk) = w;
        }
        return;
    }
    // Eq. 2: divide by the softmax denominator and store.  Lane (hf, m) owns query m and, per
    // 32-channel block, channels 8*(r/4) + 4*hf + r%4.
#pragma unroll
    for (int h = 0; h < QH; ++h) {
        const float l_tot = l_run[h] + other_half(l_run[h]);
        const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
        // formed again from the thread index, which would otherwise cost a register throughout the tile loop
        int thread = tid;
        asm volatile("" : "+v"(thread));
        if (qk.qb * BQ + (thread >> 6) * (32 * QH) + 32 * h + (thread & 31) < N) {
            uint16_t* orow = a.O + static_cast<size_t>(qk.bh) * N * D + static_cast<size_t>(qtok[h]) * D;
#pragma unroll
            for (int db = 0; db < D / 32; ++db)
#pragma unroll
                for (int rq = 0; rq < 4; ++rq) {
                    u32x2 w;
                    w.x = pack_bf16(oacc[h][db][4 * rq + 0] * inv, oacc[h][db][4 * rq + 1] * inv);
                    w.y = pack_bf16(oacc[h][db][4 * rq + 2] * inv, oacc[h][db][4 * rq + 3] * inv);
                    *reinterpret_cast<u32x2*>(orow + 32 * db + 8 * rq + 4 * hf) = w;
                }
        }
    }
}

// Which tile loop a kernel instance runs.
enum : int {
    LOOP_32 = 0,           // wavefronts of 32 query rows (attend)
    LOOP_64_PIPELINED = 1, // wavefronts of 64 rows, one per SIMD, software-pipelined (attend_wide)
    LOOP_ITEM = 3,         // LOOP_32 for one item per workgroup, without a queue; its wavefronts may form groups that split the walk
    LOOP_64 = 2            // wavefronts of 64 rows on the plain loop (attend with two halves): head_dim 64 only, where two fit a SIMD
};
constexpr int rows_per_wave(int LOOP) { return LOOP == LOOP_64_PIPELINED || LOOP == LOOP_64 ? 64 : 32; }
// Workgroups that share a query block of an item kernel of NW-wavefront groups.
constexpr int workgroups_per_block(int NW) { return NW == 1 ? 2 : 1; }
// Which instances walk banded lists by key index (MODE_BAND, MODE_BAND_GATHER) instead of by attribute table
// (MODE_LISTED): two halves, and twelve wavefronts but at head_dim 64, have no registers left for the other masks.
// (Those that do are the ones that need no copies of K and V: AttnForm::copies.)
constexpr bool walks_bands(int D, int NW, int LOOP) { return rows_per_wave(LOOP) == 32 && (NW != 12 || D == 64); }

// Wavefronts per SIMD the register allocation of the queued kernels is held to: three for the twelve-wavefront
// workgroups of 384-row blocks, two otherwise; one for the pipelined 64-row loop, which needs the whole
// register file.
constexpr int attn_waves_per_simd(int NW, int LOOP) {
    return LOOP == LOOP_64_PIPELINED ? 1 : LOOP == LOOP_32 && NW == 12 ? 3 : 2;
}

template <int D, int NW, int LOOP>
using SmemOf = std::conditional_t<LOOP == LOOP_64_PIPELINED, WideSmem<D, NW>, AttnSmem<D, NW>>;

template <bool MAY_DEAL>
__host__ __device__ __forceinline__ Queues<MAY_DEAL> queues_of(const AttnArgs& a) {
    const DevicePlan& p = a.plan[0];
    return Queues<MAY_DEAL>(a.BH, p.first_text_qb, p.nQB - p.first_text_qb, a.item_order);
}

// The next item for a workgroup whose home queue is `home`, or -1 when every queue is empty.
// ctr[x] counts how many items of queue x have been handed out.  A workgroup drains its home queue
// first (its neighbours on the XCD are on the same part of the same head, which is what the L2
// wants) and then helps whichever queue has the most left.  Every path ends: counters only grow, a
// failed take means another workgroup took that item, and once all are taken -1 is returned.
__device__ __forceinline__ int take_item(int* ctr, int home, const Queues<false>& qs, int* queue) {
    auto taken = [&](int x) { return __hip_atomic_load(ctr + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
    int q = home;
    for (;;) {
        if (taken(q) < qs.items(q)) {
            const int j = __hip_atomic_fetch_add(ctr + q, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (j < qs.items(q)) {
                *queue = q;
                return j;
            }
        }
        int best = -1, best_left = 0;
        for (int x = 0; x < 8; ++x) {
            const int left = qs.items(x) - taken(x);
            if (left > best_left) {
                best_left = left;
                best = x;
            }
        }
        if (best < 0) return -1;
        q = best;
    }
}

template <int D, int NW, int LOOP, int KS = 1, int AHEAD = RF_TILES_AHEAD, bool FEW = false>
__device__ __forceinline__ void process_item(const AttnArgs& a, int item, int xcd, int seen, const Queues<LOOP == LOOP_ITEM>& qs, unsigned char* smem, int part = 0);

// Eight queue counters, then the sweep words (-1: nothing published yet).  One workgroup, one thread per word.
constexpr int kResetThreads = 128;
static_assert(kResetThreads >= kQueueWords, "every counter and sweep word is reset");
__global__ void reset_queue_kernel(int* ctr) {
    if (threadIdx.x < kQueueWords) ctr[threadIdx.x] = threadIdx.x < 8 ? 0 : -1;
}

// NW wavefronts of rows_per_wave(LOOP) query rows each.
template <int D, int NW, int LOOP>
__global__ void __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(attn_waves_per_simd(NW, LOOP), attn_waves_per_simd(NW, LOOP)))) attn_kernel(AttnArgs a) {
    extern __shared__ __attribute__((aligned(256))) unsigned char smem[];  // the kernel's only LDS: starts at address 0
    int* item_box = reinterpret_cast<int*>(smem + SmemOf<D, NW, LOOP>::ITEM_OFF);
    // A resident set of workgroups (as many as fit on the chip) works through the (head, query
    // block) items.  Workgroup ids go to the 8 XCDs round-robin; XCD x's queue is one eighth of every
    // head's block order, head after head (neighbours in that order walk nearly the same key tiles,
    // which they share through the XCD's L2), so all XCDs move through the heads together and the
    // K/V of the head in flight (tens of MB) stays resident in the memory-side cache for whatever
    // misses L2.  XCDs differ in speed by several per cent and shares in work; an XCD whose queue is
    // empty takes items from the others.
    const Queues<false> qs = queues_of<false>(a);
    for (;;) {
        if (threadIdx.x == 0) {
            int q = 0;
            item_box[0] = take_item(a.queue, blockIdx.x & 7, qs, &q);
            item_box[1] = q;
            // the sweep word for the item's head on this workgroup's XCD (it serves its own L2, whichever queue
            // the item came from), read ONCE for the whole workgroup: it changes all the time
            const int it = item_box[0];
            int bh = 0, ordinal = 0;
            if (it >= 0) qs.locate(it, q, &bh, &ordinal);
            item_box[2] = (a.join_sweep && it >= 0)
                              ? __hip_atomic_load(sweep_word(a.queue, blockIdx.x & 7, bh), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                              : -1;
        }
        __syncthreads();
        // wavefront-uniform by construction; say so, so that everything derived stays in scalar registers
        const int item = __builtin_amdgcn_readfirstlane(item_box[0]), xcd = __builtin_amdgcn_readfirstlane(item_box[1]);
        const int seen = __builtin_amdgcn_readfirstlane(item_box[2]);
        __syncthreads();
        if (item < 0) break;
        process_item<D, NW, LOOP>(a, item, xcd, seen, qs, smem);
    }
}

// The kernel for launches of few rounds: one workgroup per item and no queue (workgroup ids go to the XCDs
// round-robin, so workgroup i is item i / 8 of queue i mod 8).  Without the queue there is no kernel to reset it,
// no atomic round trip and no second barrier before an item's first load, and workgroups of any size share a CU:
// 48 heads of 2000 tokens at head_dim 128, 128 rows: 109 -> 75 us; 256 rows: 88 -> 81 us.  With the patterns the
// queue's balance between XCDs and its joined walks win from about 17000 tokens on (256 rows, 48 heads of 17776: 3.65
// against 3.72 ms; 24 of 48000: 12.7 against 14.3); dense walks stay even or better from the grid (32 of 16384: 3.73
// against 3.84 ms; 24 of 119056: 147 against 149).
// KS groups of NW wavefronts split the walk of 32 * NW rows.  AHEAD = 0 keeps one buffer for K and one for V, so
// that twice the workgroups fit a CU's LDS.  NW = 1: a block of 64 rows is two workgroups' work, taken while each of them
// has a CU to itself (see launch_items_d).
template <int D, int NW, int KS, int AHEAD, int WAVES>
__global__ void __launch_bounds__(64 * NW * KS) __attribute__((amdgpu_waves_per_eu(WAVES, WAVES))) attn_item_kernel(AttnArgs a) {
    extern __shared__ __attribute__((aligned(256))) unsigned char smem[];  // the kernel's only LDS: starts at address 0
    const Queues<true> qs = queues_of<true>(a);
    constexpr int PARTS = workgroups_per_block(NW);
    const int xcd = blockIdx.x & 7, item = (blockIdx.x >> 3) / PARTS, part = (blockIdx.x >> 3) % PARTS;
    if (item >= qs.items(xcd)) return;
    process_item<D, NW, LOOP_ITEM, KS, AHEAD, D == 96 && KS == 2 && WAVES == 3>(a, item, xcd, -1, qs, smem, part);
}

// One (head, query block) item: item-th of queue xcd.  seen: the sweep word of this workgroup's XCD
// (it serves its own L2, whichever queue the item came from), or -1.
template <int D, int NW, int LOOP, int KS, int AHEAD, bool FEW>
__device__ __forceinline__ void process_item(const AttnArgs& a, int item, int xcd, int seen, const Queues<LOOP == LOOP_ITEM>& qs, unsigned char* smem, int part) {
    // Where few rows leave a launch bound by latency, the tiles of a band are worked out; the others' items are long enough for
    // the loads of the list not to show (15 heads of 4340 tokens, head_dim 128, 256 rows 103.3 / 104.2 us worked out).
    constexpr bool kComputed = LOOP == LOOP_ITEM && KS > 1;
    auto run = [&](auto mode, const DevicePlan& plan, const QueryBlock& block) {
        constexpr int MODE = decltype(mode)::value;
        if constexpr (LOOP == LOOP_64_PIPELINED) attend_wide<D, NW, MODE>(a, plan, block, smem);
        else {
            QueryBlock rows = block;  // the lists are the block's, the rows this workgroup's part of it
            if constexpr (LOOP == LOOP_ITEM && workgroups_per_block(NW) > 1) rows.qb = block.qb * workgroups_per_block(NW) + part;
            attend<D, NW, MODE, rows_per_wave(LOOP) / 32, KS, AHEAD, raise_of(D, NW, KS, LOOP != LOOP_ITEM, MODE), kComputed, FEW>(a, plan, rows, smem);
        }
    };
    int ordinal, bh;  // position in the block order, and the head
    qs.locate(item, xcd, &bh, &ordinal);
    QueryBlock qk;
    qk.bh = bh;
    // per-head bandwidth: the plans differ only in the Spatial / Temporal lists, radii and block order
    int which = 0;
    if (a.head_bw) {
        which = a.head_bw[qk.bh];
        if (static_cast<unsigned>(which) >= static_cast<unsigned>(a.n_plans)) which = 0;
    }
    const DevicePlan& pl = a.plan[which];
    // One item per workgroup: what stands between its start and its first tile are these loads, one after the
    // other, so the list bounds (where they are read: of every pattern) are asked for along with the class, and the blocks
    // keep their order.
    constexpr bool kOneItem = LOOP == LOOP_ITEM;
    int lo[kLists] = {}, hi[kLists] = {};
    if constexpr (kOneItem) {
        qk.qb = ordinal < qs.nTB ? qs.nVB + ordinal : ordinal - qs.nTB;
#pragma unroll
        for (int l = 0; l < kLists; ++l) {
            if (kComputed && l != RF_TEXTURAL) continue;
            lo[l] = pl.row_ptr[l][qk.qb];
            hi[l] = pl.row_ptr[l][qk.qb + 1];
        }
    }
    int cls = a.head_class ? a.head_class[qk.bh] : RF_DENSE;
    if (static_cast<unsigned>(cls) > 3u) cls = RF_DENSE;
    qk.cls = cls;
    // a Temporal head walks its keys in position-major order: a copy of its K and V if the caller gave room for
    // one, else row by row through the index table (or, where that loop does not exist, in token order)
    constexpr bool kBands = walks_bands(D, NW, LOOP);
    const bool temporal_pm = cls == RF_TEMPORAL && (a.packed_k || kBands);
    const int list = temporal_pm ? kListTemporalPM : cls;
    // dense heads: text-holding blocks first, then token order
    if constexpr (!kOneItem) qk.qb = cls == RF_DENSE ? (ordinal < qs.nTB ? qs.nVB + ordinal : ordinal - qs.nTB) : pl.qorder[list][ordinal];
    constexpr int PARTS = kOneItem ? workgroups_per_block(NW) : 1;
    if (PARTS > 1 && (qk.qb * PARTS + part) * (32 * NW) >= pl.N) return;  // the last block ends in its first part
    qk.first = 0;
    qk.cols = nullptr;
    qk.sweep = a.join_sweep ? sweep_word(a.queue, blockIdx.x & 7, bh) : nullptr;
    auto same_sequence = [&]() { return seen >= 0 && (seen >> kSweepTileBits) == qk.sweep_tag; };
    qk.list = cls;
    qk.row_token = nullptr;
    qk.video_shift = pl.video_shift;
    qk.text_shift = pl.text_shift;
    const size_t head_bytes = static_cast<size_t>(qk.bh) * pl.N * D * 2;
    qk.kbase = reinterpret_cast<const unsigned char*>(a.K) + head_bytes;
    qk.vbase = reinterpret_cast<const unsigned char*>(a.V) + head_bytes;
    // tag: the head and which of its key sequences is walked (token order, compacted, position-major)
    const int kTagBits = 31 - kSweepTileBits;
    auto tag_of = [&](int sequence) { return (qk.bh * 4 + sequence) & ((1 << kTagBits) - 1); };
    if (cls == RF_DENSE) {
        qk.ntiles = pl.nKT;
        qk.keyN = pl.N;
        qk.sweep_tag = tag_of(0);
        if (same_sequence() && (seen & kSweepTileMask) < qk.ntiles) qk.first = seen & kSweepTileMask;
        run(std::integral_constant<int, MODE_ALL>{}, pl, qk);
    } else if (cls == RF_TEXTURAL && qk.qb < pl.first_text_qb) {
        // Textural query blocks made only of video tokens see the compacted key sequence (Eq. 5):
        // as a packed copy made by pack_textural_kernel if the caller gave room for one, else
        // gathered row by row through the index table
        qk.ntiles = pl.nCT;
        qk.keyN = pl.Nc;
        qk.sweep_tag = tag_of(1);
        if (same_sequence() && (seen & kSweepTileMask) < qk.ntiles) qk.first = seen & kSweepTileMask;
        if (a.packed_k) {
            const size_t packed_bytes = head_bytes;
            qk.kbase = reinterpret_cast<const unsigned char*>(a.packed_k) + packed_bytes;
            qk.vbase = reinterpret_cast<const unsigned char*>(a.packed_v) + packed_bytes;
            qk.video_shift = qk.text_shift = 0;
            run(std::integral_constant<int, MODE_ALL>{}, pl, qk);
        } else {
            run(std::integral_constant<int, MODE_COMPACT>{}, pl, qk);
        }
    } else {
        qk.list = list;
        if (temporal_pm) {
            qk.row_token = pl.pm_token;
            if (a.packed_k) {
                qk.kbase = reinterpret_cast<const unsigned char*>(a.packed_k) + head_bytes;
                qk.vbase = reinterpret_cast<const unsigned char*>(a.packed_v) + head_bytes;
            }
            qk.video_shift = qk.text_shift = 0;
        }
        if (kComputed && cls != RF_TEXTURAL) {
            qk.band = BandTiles(qk.qb * pl.block, pl.block, pl.group_rows[list], pl.radius[list], pl.N, pl.Nv);
            qk.ntiles = qk.band.tiles;
        } else {
            auto of_list = [&](const int (&v)[kLists]) { return list == 0 ? v[0] : list == 1 ? v[1] : list == 2 ? v[2] : v[3]; };
            const int e0 = kOneItem ? of_list(lo) : pl.row_ptr[list][qk.qb];
            qk.ntiles = (kOneItem ? of_list(hi) : pl.row_ptr[list][qk.qb + 1]) - e0;
            qk.cols = pl.cols[list] + e0;
            if constexpr (!kOneItem) qk.first = pl.first_entry[list][qk.qb];
        }
        qk.keyN = pl.N;
        qk.sweep_tag = tag_of(temporal_pm ? 2 : 0);
        if (same_sequence() && qk.ntiles > 0) {
            // banded lists are one run of consecutive tiles (then the text tiles): the published tile,
            // if it is in the run, sits at entry (tile - first tile of the run)
            const int tile = seen & kSweepTileMask, at = tile - (qk.cols[0] & kTileIndexMask);
            // if it is not (the others are just outside this block's band, which overlaps theirs almost
            // entirely), the start of the run is where they will be next
            qk.first = (at >= 0 && at < qk.ntiles && (qk.cols[at] & kTileIndexMask) == tile) ? at : 0;
        }
        if constexpr (!kBands) run(std::integral_constant<int, MODE_LISTED>{}, pl, qk);
        else if (cls == RF_TEXTURAL) run(std::integral_constant<int, MODE_LISTED>{}, pl, qk);
        else if (temporal_pm && !a.packed_k) run(std::integral_constant<int, MODE_BAND_GATHER>{}, pl, qk);
        else run(std::integral_constant<int, MODE_BAND>{}, pl, qk);
    }
}

// Copies of K and V in the order their head walks them, into the caller's workspace: for a
// Textural head the kept keys' rows, then the text rows (K_C, V_C of Eq. 5 made physical); for a
// Temporal head every row, in position-major order.  One workgroup per (64 copied rows, head).
template <int D>
__global__ void __launch_bounds__(256) pack_textural_kernel(AttnArgs a) {
    const DevicePlan& pl = a.plan[0];
    const int bh = blockIdx.y, cls = a.head_class[bh];
    if (cls != RF_TEXTURAL && cls != RF_TEMPORAL) return;
    const int32_t* token_of = cls == RF_TEXTURAL ? pl.cidx : pl.pm_token;
    const int rows = cls == RF_TEXTURAL ? pl.Nc : pl.N;
    constexpr int CH = D / 8;  // 16-byte chunks per row
    const size_t head = static_cast<size_t>(bh) * pl.N * D;
    for (int i = threadIdx.x; i < kTileK * CH; i += 256) {
        const int c = blockIdx.x * kTileK + i / CH, ch = i % CH;
        if (c >= rows) break;
        const size_t src = head + static_cast<size_t>(token_of[c]) * D + 8 * ch;
        const size_t dst = head + static_cast<size_t>(c) * D + 8 * ch;
        *reinterpret_cast<u32x4*>(a.packed_k + dst) = *reinterpret_cast<const u32x4*>(a.K + src);
        *reinterpret_cast<u32x4*>(a.packed_v + dst) = *reinterpret_cast<const u32x4*>(a.V + src);
    }
}

int launch_pack_textural(const AttnArgs& a, int D, void* stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    const dim3 grid(a.plan[0].nKT, a.BH);
    if (D == 64) hipLaunchKernelGGL(pack_textural_kernel<64>, grid, dim3(256), 0, st, a);
    else if (D == 96) hipLaunchKernelGGL(pack_textural_kernel<96>, grid, dim3(256), 0, st, a);
    else if (D == 128) hipLaunchKernelGGL(pack_textural_kernel<128>, grid, dim3(256), 0, st, a);
    else return static_cast<int>(hipErrorInvalidValue);
    return static_cast<int>(hipGetLastError());
}

template <int D, int NW, int LOOP = LOOP_32>
static int launch_one(const AttnArgs& a, hipStream_t st) {
    constexpr int NT = 64 * NW;
    constexpr int smem = SmemOf<D, NW, LOOP>::BYTES;
    // workgroups each device holds at once, found on first use there (which also raises the kernel's dynamic-LDS limit)
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static int resident_on[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return static_cast<int>(e);
    if (dev < 0 || dev >= kMaxDevices) return static_cast<int>(hipErrorInvalidDevice);
    int resident = 0;
    {
        std::lock_guard<std::mutex> lock(mu);
        if (resident_on[dev] == 0) {
            const void* fn = reinterpret_cast<const void*>(&attn_kernel<D, NW, LOOP>);
            e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, smem);
            if (e != hipSuccess) return static_cast<int>(e);
            int cus = 0, per_cu = 0;
            if ((e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev)) != hipSuccess) return static_cast<int>(e);
            if ((e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, attn_kernel<D, NW, LOOP>, NT, smem)) != hipSuccess)
                return static_cast<int>(e);
            if (cus < 1 || per_cu < 1) return static_cast<int>(hipErrorInvalidValue);
            resident_on[dev] = cus * per_cu;
        }
        resident = resident_on[dev];
    }
    const long long items = static_cast<long long>(a.plan[0].nQB) * a.BH;
    const int grid = static_cast<int>(std::min<long long>(resident, items));
    hipLaunchKernelGGL(reset_queue_kernel, dim3(1), dim3(kResetThreads), 0, st, a.queue);
    e = hipGetLastError();
    if (e != hipSuccess) return static_cast<int>(e);
    hipLaunchKernelGGL((attn_kernel<D, NW, LOOP>), dim3(grid), dim3(NT), smem, st, a);
    return static_cast<int>(hipGetLastError());
}

template <int D, int NW, int KS, int AHEAD, int WAVES>
static int launch_items(const AttnArgs& a, hipStream_t st) {
    constexpr int NT = 64 * NW * KS, smem = AttnSmem<D, NW, KS, AHEAD>::BYTES;
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static bool ready_on[kMaxDevices] = {};  // the kernel's dynamic-LDS limit has been raised there
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return static_cast<int>(e);
    if (dev < 0 || dev >= kMaxDevices) return static_cast<int>(hipErrorInvalidDevice);
    {
        std::lock_guard<std::mutex> lock(mu);
        if (!ready_on[dev]) {
            const void* fn = reinterpret_cast<const void*>(&attn_item_kernel<D, NW, KS, AHEAD, WAVES>);
            if ((e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, smem)) != hipSuccess) return static_cast<int>(e);
            ready_on[dev] = true;
        }
    }
    const int most = queues_of<true>(a).items(0) * workgroups_per_block(NW);
    AttnArgs s = a;
    s.join_sweep = 0;  // its words are not there: nothing resets them
    hipLaunchKernelGGL((attn_item_kernel<D, NW, KS, AHEAD, WAVES>), dim3(8 * most), dim3(NT), smem, st, s);
    return static_cast<int>(hipGetLastError());
}

// The item kernels of one head_dim: 64 rows with the keys split four or two ways, 128 rows, 256 rows (not at
// head_dim 64, where 128 rows measured 6 % faster).  Wavefronts per SIMD: three where the registers allow it.
template <int D>
static int launch_items_d(const AttnArgs& a, hipStream_t st) {
    if (a.plan[0].block == 64 && a.key_groups == 4) {
        // A launch this small is bound by latency: two loads of memory, a barrier and a tile's worth of dependent work one
        // after the other in every step.  As two workgroups of 32 rows a block's steps are half as long and have no barrier, as
        // long as each has a CU to itself; the sums, and so the bits, are the same.  us, 64 rows / 32: 6 heads of 960 tokens, head_dim
        // 128, 20.2 / 17.2 with and 16.6 / 12.5 without text, 64 15.5 / 13.3; 1 of 7936, 128, Spatial 61.9 / 49.2, Temporal 46.5 / 35.0;
        // 2 of 4032, 96, dense 32.9 / 24.8, classes in turn 24.4 / 19.4; 2 of 256, 64, 7.7 / 6.7.  With a CU short (17 or 18 blocks on an
        // XCD): 4 of 2112, 128, dense 24.2 / 37.2, Temporal 19.4 / 26.6, 23 of 380, 96, dense 8.6 / 14.3; at 64, where two fit a CU, 2 of
        // 8192 34.2 / 38.9, 10 of 1600 dense 14.7 / 15.6, classes in turn 15.4 / 13.5.
        if (halves_have_cus(queues_of<true>(a).items(0))) return launch_items<D, 1, 4, 0, 2>(a, st);
        return launch_items<D, 2, 4, 0, 2>(a, st);
    }
    if (a.plan[0].block == 64 && a.key_groups == 2) {
        // at head_dim 96 three leave the loops few registers (FEW in attend): see three_to_a_cu
        if constexpr (D == 96) {
            if (!a.three_to_a_cu) return launch_items<D, 2, 2, 0, 2>(a, st);
        }
        return launch_items<D, 2, 2, 0, D == 128 ? 2 : 3>(a, st);
    }
    if (a.plan[0].block == 128) return launch_items<D, 4, 1, 0, D == 128 ? 2 : 3>(a, st);
    if constexpr (D != 64)
        if (a.plan[0].block == 256) return launch_items<D, 8, 1, 1, 2>(a, st);
    return static_cast<int>(hipErrorInvalidValue);
}

int launch_attention(const AttnArgs& a, int D, void* stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int nw = a.plan[0].block / 32;
    if (a.wide_rows) {  // the pipelined loop for 64-row wavefronts: 256-row blocks as four wavefronts, head_dim 128
        if (D == 128 && nw == 8) return launch_one<128, 4, LOOP_64_PIPELINED>(a, st);
        return static_cast<int>(hipErrorInvalidValue);
    }
    if (D != 64 && D != 96 && D != 128) return static_cast<int>(hipErrorInvalidValue);
    if (!a.queued) return D == 64 ? launch_items_d<64>(a, st) : D == 96 ? launch_items_d<96>(a, st) : launch_items_d<128>(a, st);
    // 256-row blocks at head_dim 64: four wavefronts of 64 rows (two still fit a SIMD; measured 8-15 %
    // faster than eight of 32: half the LDS operand reads and half the per-tile bookkeeping per MFMA)
    if (D == 64 && nw == 8) return launch_one<64, 4, LOOP_64>(a, st);
    if (D == 96 && nw == 8) return launch_one<96, 8>(a, st);
    if (D == 128 && nw == 8) return launch_one<128, 8>(a, st);
    // 384-row blocks: twelve wavefronts, three per SIMD at 168 registers (3-7 % faster than eight on 256
    // rows for every class at head_dim 96 and 128; even with the 64-row wavefronts at head_dim 64)
    if (D == 64 && nw == 12) return launch_one<64, 12>(a, st);
    if (D == 96 && nw == 12) return launch_one<96, 12>(a, st);
    if (D == 128 && nw == 12) return launch_one<128, 12>(a, st);
    return static_cast<int>(hipErrorInvalidValue);
}

}  // namespace rf
