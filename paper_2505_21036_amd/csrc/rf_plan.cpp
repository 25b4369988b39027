// Host-side block lists for RainFusion's three head patterns (Sec. 3.2).
//
// The masks are token-level predicates; this file only decides, for a tiling of the N x N
// score matrix into query blocks of `block` rows and key tiles of 64 columns, which pairs
// contain at least one kept token pair (they are visited) and which of those contain a dropped
// pair or run past the last token (the kernel re-applies the predicate there).  Everything is exact integer interval
// arithmetic on frame indices and in-frame positions.
#include <algorithm>
#include <cmath>
#include <numeric>
#include <utility>

#include "rf_internal.h"
#include "rf_queues.h"

namespace rf {

static int band_radius(float bw, int n) {
    double r = std::floor(static_cast<double>(bw) * static_cast<double>(n));
    if (r < 0) r = 0;
    if (r > n) r = n;
    return static_cast<int>(r);
}

int resolve_geometry(const rf_layout* L, const rf_params* P, Geometry* g) {
    if (!L) return RF_ERR_NULL;
    if (L->T < 1 || L->H < 1 || L->W < 1 || L->text_len < 0) return RF_ERR_LAYOUT;
    const int64_t HW = static_cast<int64_t>(L->H) * L->W;
    const int64_t Nv = HW * L->T;
    const int64_t N = Nv + L->text_len;
    if (N > (int64_t{1} << 24)) return RF_ERR_SHAPE;  // keeps every index and block count in int32
    rf_params def = {0.25f, 0.25f, 2, 0, 0};
    const rf_params* p = P ? P : &def;
    if (!(p->bw_spatial >= 0.f && p->bw_spatial <= 1.f)) return RF_ERR_PARAM;
    if (!(p->bw_temporal >= 0.f && p->bw_temporal <= 1.f)) return RF_ERR_PARAM;
    if (p->tex_stride < 1 || p->sample_interval < 0) return RF_ERR_PARAM;
    if (p->flags & ~(RF_FLAG_TWO_HEAD | RF_FLAG_TEXT_FIRST | RF_FLAG_FORCE_DENSE | RF_FLAG_FIXED_ORDER | RF_FLAG_WIDE_ROWS)) return RF_ERR_PARAM;
    g->T = L->T; g->H = L->H; g->W = L->W; g->text_len = L->text_len;
    g->HW = static_cast<int>(HW); g->Nv = static_cast<int>(Nv); g->N = static_cast<int>(N);
    g->r_spatial = band_radius(p->bw_spatial, L->T);
    g->r_temporal = band_radius(p->bw_temporal, g->HW);
    g->tau = p->tex_stride;
    g->omega = p->sample_interval > 0 ? p->sample_interval : L->T;
    g->two_head = (p->flags & RF_FLAG_TWO_HEAD) ? 1 : 0;
    g->text_first = (p->flags & RF_FLAG_TEXT_FIRST) && L->text_len > 0 ? 1 : 0;
    return RF_OK;
}

namespace {

struct Span { int lo, hi; };  // inclusive

// In-frame positions covered by video tokens [s, e): one span per frame touched.
void position_spans(int s, int e, int HW, std::vector<Span>* out) {
    out->clear();
    if (s >= e) return;
    const int fs = s / HW, fe = (e - 1) / HW;
    for (int f = fs; f <= fe; ++f) {
        Span sp{f == fs ? s % HW : 0, f == fe ? (e - 1) % HW : HW - 1};
        out->push_back(sp);
        if (sp.lo == 0 && sp.hi == HW - 1) { out->assign(1, sp); return; }  // a whole frame covers all
    }
}

inline int span_gap(Span a, Span b) { return std::max(0, std::max(b.lo - a.hi, a.lo - b.hi)); }
inline int span_reach(Span a, Span b) { return std::max(b.hi - a.lo, a.hi - b.lo); }

}  // namespace

// How a head's query blocks are handed to workgroups.  The attention kernel runs one queue of
// (head, query block) items per XCD (each XCD has its own L2) and a workgroup takes items from other
// XCDs' queues once its own is empty, so the queues need not hold equal work.  Two things matter:
//  - The blocks that hold text rows are the long items (text queries see every key, so such a block
//    walks the whole sequence under every pattern).  They come first in the order, and the kernel
//    hands them out, for all heads, before anything else: the launch must not end waiting for one.
//  - The other blocks follow in a locality order, of which XCD x owns the x-th eighth, head after
//    head: blocks that run together (an XCD has about kConcurrentRows query rows in flight, a
//    generation) should walk the same key tiles at the same time, so that a tile is fetched into
//    the XCD's L2 once.  That order is token order (under the Temporal pattern in token order,
//    whose lists depend only on the in-frame position: grouped by position across frames); and in
//    the banded lists (Spatial; Temporal in position-major order), where a block's tiles are one
//    contiguous range that slides with the block, the blocks of a generation all start their walk
//    at the same tile, the first tile of the generation's last block, and wrap around: they then
//    sweep the same tiles in step instead of each trailing its neighbour by the slide.
static void order_query_blocks(HostPlan* plan) {
    HostPlan& P = *plan;
    const int nQB = P.nQB, block = P.block, HW = P.g.HW;
    const int nVB = P.first_text_qb, nTB = nQB - nVB;  // video-only blocks, text-holding blocks
    const int per_share = (nVB + 7) / 8;
    constexpr int kConcurrentRows = 8192;  // 32 CUs x 256 rows
    const int generation = std::max(1, kConcurrentRows / block);
    for (int cls = 0; cls < kLists; ++cls) {
        std::vector<int32_t>& ord = P.qorder[cls];
        ord.resize(nQB);
        for (int i = 0; i < nTB; ++i) ord[i] = nVB + i;
        for (int qb = 0; qb < nVB; ++qb) ord[nTB + qb] = qb;
        if (cls == RF_TEMPORAL) {
            auto key = [&](int qb) { return (static_cast<int64_t>(qb) * block % HW) / block; };
            std::stable_sort(ord.begin() + nTB, ord.end(), [&](int a, int b) { return key(a) < key(b); });
        }
        std::vector<int32_t>& fe = P.first_entry[cls];
        fe.assign(nQB, 0);
        if (cls != RF_SPATIAL && cls != kListTemporalPM) continue;
        auto tile_of = [&](int e) { return P.cols[cls][e] & kTileIndexMask; };
        for (int s0 = 0; s0 < nVB; s0 += per_share)
            for (int g0 = s0; g0 < std::min(s0 + per_share, nVB); g0 += generation) {
                const int g1 = std::min({g0 + generation, s0 + per_share, nVB});
                int start_tile = 0;
                for (int o = g0; o < g1; ++o) {
                    const int qb = ord[nTB + o];
                    if (P.row_ptr[cls][qb] < P.row_ptr[cls][qb + 1]) start_tile = std::max(start_tile, tile_of(P.row_ptr[cls][qb]));
                }
                for (int o = g0; o < g1; ++o) {
                    const int qb = ord[nTB + o], e0 = P.row_ptr[cls][qb], e1 = P.row_ptr[cls][qb + 1];
                    int e = e0;
                    while (e < e1 && tile_of(e) < start_tile) ++e;
                    fe[qb] = e < e1 ? e - e0 : 0;
                }
            }
    }
}

void build_tables(const Geometry& g, TokenTables* tables) {
    TokenTables& T = *tables;
    const int N = g.N, Nv = g.Nv, HW = g.HW;
    for (auto& a : T.attr) a.assign(N, 0);
    T.pm_token.resize(N);
    for (int p = 0; p < HW; ++p)  // position-major row p*T + f
        for (int f = 0; f < g.T; ++f) {
            T.pm_token[p * g.T + f] = g.row_of(f * HW + p);
            T.attr[kListTemporalPM][p * g.T + f] = p;
        }
    for (int n = Nv; n < N; ++n) T.pm_token[n] = g.row_of(n);
    T.cidx.clear();
    for (int f = 0, n = 0; f < g.T; ++f)
        for (int y = 0, p = 0; y < g.H; ++y)
            for (int x = 0; x < g.W; ++x, ++p, ++n) {
                T.attr[RF_SPATIAL][n] = f;
                T.attr[RF_TEMPORAL][n] = p;
                const bool kept = ((y - x) % g.tau) == 0;
                T.attr[RF_TEXTURAL][n] = kept ? 0 : 1;
                if (kept) T.cidx.push_back(g.row_of(n));
            }
    for (int n = Nv; n < N; ++n) T.cidx.push_back(g.row_of(n));
}

void build_plan(const Geometry& g, int block, HostPlan* plan) {
    TokenTables tables;
    build_tables(g, &tables);
    build_plan(g, tables, block, true, plan);
}

void build_plan(const Geometry& g, const TokenTables& tables, int block, bool token_order_temporal, HostPlan* plan, bool with_banded) {
    HostPlan& P = *plan;
    P.g = g;
    P.block = block;
    const int N = g.N, Nv = g.Nv, HW = g.HW;
    P.nQB = (N + block - 1) / block;
    P.nKT = (N + kTileK - 1) / kTileK;
    P.first_text_qb = g.text_len > 0 ? Nv / block : P.nQB;
    P.Nc = static_cast<int>(tables.cidx.size());
    P.nCT = (P.Nc + kTileK - 1) / kTileK;
    const int first_text_tile = g.text_len > 0 ? Nv / kTileK : P.nKT;

    std::vector<Span> qs, ks, tile(P.nKT);
    std::vector<char> every_kept(P.nKT), some_kept(P.nKT);
    for (int cls = 0; cls < kLists; ++cls) {
        // a band over groups of consecutive rows: frames of HW tokens (Spatial), positions of T tokens
        // (Temporal in position-major order)
        const bool banded = cls == RF_SPATIAL || cls == kListTemporalPM;
        const int group = cls == RF_SPATIAL ? HW : g.T, group_radius = cls == RF_SPATIAL ? g.r_spatial : g.r_temporal;
        auto& rp = P.row_ptr[cls];
        auto& co = P.cols[cls];
        rp.assign(P.nQB + 1, 0);
        co.clear();
        if ((cls == RF_TEMPORAL && !token_order_temporal) || (banded && !with_banded)) continue;
        // of the video keys of every tile: the groups they lie in, or which of them the Textural pattern keeps
        for (int kb = 0; kb < P.nKT; ++kb) {
            const int k0 = kb * kTileK, kv1 = std::min(k0 + kTileK, Nv);
            if (k0 >= Nv) break;
            if (banded) tile[kb] = Span{k0 / group, (kv1 - 1) / group};
            if (cls == RF_TEXTURAL && P.first_text_qb < P.nQB) {
                int kept = 0;
                for (int j = k0; j < kv1; ++j) kept += tables.attr[RF_TEXTURAL][j] == 0;
                every_kept[kb] = kept == kv1 - k0;
                some_kept[kb] = kept > 0;
            }
        }
        for (int qb = 0; qb < P.nQB; ++qb) {
            const int q0 = qb * block, q1 = std::min(N, q0 + block);
            const int qv1 = std::min(q1, Nv);  // video part [q0, qv1)
            const bool q_text = q1 > Nv, q_video = q0 < Nv;
            if (cls == RF_TEXTURAL && !q_text) { rp[qb + 1] = static_cast<int32_t>(co.size()); continue; }
            if (cls == RF_TEMPORAL && q_video) position_spans(q0, qv1, HW, &qs);
            auto add = [&](int kb, bool all) {
                const bool tail = (kb + 1) * kTileK > N, k_text = (kb + 1) * kTileK > Nv, k_video = kb * kTileK < Nv;
                // a tile of text keys only is never partial; one that mixes text and video keys, or
                // runs past N, needs the position checks as well as the pattern's band check
                const bool boundary = tail || (k_text && k_video && !all);
                co.push_back(kb | ((!all || tail) ? RF_PLAN_PARTIAL : 0) | (boundary ? kTileBoundary : 0));
            };
            if (banded && q_video && !q_text) {
                // the tiles with a key of a group within reach (their video keys are the tokens below Nv), then those with text keys
                const int lo = q0 / group, hi = (qv1 - 1) / group;
                const int run0 = std::max(lo - group_radius, 0) * group / kTileK;
                const int run1 = static_cast<int>((std::min<int64_t>(Nv, static_cast<int64_t>(hi + group_radius + 1) * group) + kTileK - 1) / kTileK);
                // full tiles of video keys, nearly all there are, without the other cases' tests
                const int whole = std::min(run1, Nv / kTileK);
                const size_t at = co.size();
                co.resize(at + std::max(whole - run0, 0));
                for (int kb = run0; kb < whole; ++kb)
                    co[at + kb - run0] = kb | (span_reach(Span{lo, hi}, tile[kb]) <= group_radius ? 0 : RF_PLAN_PARTIAL);
                for (int kb = std::max(run0, whole); kb < run1; ++kb) add(kb, span_reach(Span{lo, hi}, tile[kb]) <= group_radius);
                for (int kb = std::max(run1, first_text_tile); kb < P.nKT; ++kb)
                    add(kb, kb * kTileK >= Nv || span_reach(Span{lo, hi}, tile[kb]) <= group_radius);
                rp[qb + 1] = static_cast<int32_t>(co.size());
                continue;
            }
            for (int kb = 0; kb < P.nKT; ++kb) {
                const int k0 = kb * kTileK, k1 = std::min(N, k0 + kTileK);
                const int kv1 = std::min(k1, Nv);
                bool any = q_text || k1 > Nv, all = true;
                if (q_video && k0 < Nv) {
                    if (banded) {
                        all = span_reach(Span{q0 / group, (qv1 - 1) / group}, tile[kb]) <= group_radius;
                    } else if (cls == RF_TEMPORAL) {
                        position_spans(k0, kv1, HW, &ks);
                        for (Span a : qs)
                            for (Span b : ks) {
                                any = any || span_gap(a, b) <= g.r_temporal;
                                all = all && span_reach(a, b) <= g.r_temporal;
                            }
                    } else {  // Textural rows of a block that also holds text rows
                        any = any || some_kept[kb];
                        all = every_kept[kb];
                    }
                }
                if (any) add(kb, all);
            }
            rp[qb + 1] = static_cast<int32_t>(co.size());
        }
    }
    order_query_blocks(plan);
}

namespace {

// What a launch takes in each form, us: the model by which the form is chosen.  The numbers are fitted to the times
// that the kernels without wave priorities had at 107 sizes (256 to 119056 tokens, 1 to 160 heads), dense and with the
// three patterns in turn at bandwidth 1/4 and stride 2, and at 58 of them at bandwidths 1/8 to 1/2 and strides 1 to 4.
// They were not fitted again, but for the two kernels that changed most (kThreeToACu, and choose_form for few blocks); over the
// present kernels' times at the same sizes (profiles/forms_sweep.txt) the form they pick is, on the geometric mean, 0.2 % from the best
// where all heads are dense (1.2 % at head_dim 64) and 1.3 to 2.2 % with the patterns; the worst are 7 to 33 %, mostly a few heads of short
// layouts with text.  Few rows: keys split four ways, then two ways (16 heads of 960 tokens, head_dim 128: 21 us, 25 and with 128 rows 39;
// 24 heads of 4109: 175, 147 and 168).  Many: the forms with the most rows do the least per row and tile (48 heads of
// 17776: 4.7, 4.4 and 3.8 ms for these, 3.62 and 3.60 with 256 rows from the grid and from queues, 3.58 with 384; 24 of 48000, dense:
// 26.4 ms with 128 rows, 24.5 with 256, 23.4 with 384).  Between them what counts is how full the last round of
// workgroups is, on the fullest XCD where the XCDs cannot help each other.
//
// At head_dim 64 the model has 256 rows from queues slower than they are with the priorities (48 heads of 17776 tokens, patterns
// in turn: 2316 us when it was fitted, 2062 since, against 2102 with 128 rows), so some sizes with room for copies stay with 128
// rows, in whose launches every block starts at a fixed tile: their O is the same bits in every call.
//
// copies: up to 256 rows, rows gathered through an index table cost nothing that can be measured, so no copies are
// made (17776 tokens, 24 heads, head_dim 128, 128 rows: 1.92 ms either way); twelve wavefronts at head_dim 96 and
// 128 and the 64-row wavefronts at 64 have no registers for the loop that gathers Temporal heads (3.79 ms in token
// order against 1.85 ms with copies at 384 rows).
struct Kernel {
    AttnForm form;
    int per_cu;           // workgroups a CU holds
    double tile_us;       // per 64-key tile of a listed walk, where every CU holds that many
    double item_us;       // to start and finish a workgroup
    double spread;        // share of its time that a workgroup saves as its CU's only one of very many
    double dense;         // times tile_us where no list is walked
    double text;          // times tile_us in a block that holds text rows, which walks every tile, most of them masked
    double text_tile_us;  // per tile of such a block where nothing else is left to run: no launch ends before it
};
struct Chip {
    double start_us;             // of a launch
    double smooth, smoother;     // how far the last, partial round is spread over the chip: after one round, more with every further one
    double smooth_dense;         // likewise for dense walks, which are all of one length
    double queue_us;             // the reset and the atomics of a launch from queues
    double copy_us;              // per MB read and written for copies of K and V
    double far, far_dense;       // times tile_us where eight heads' K and V do not fit the memory-side cache (workgroups from the grid: nothing keeps them in step)
    double alone;                // share of text_tile_us on a nearly empty chip
    double many, many_dense;     // gain, resp. loss if negative, of a launch of very many rounds
};
constexpr int kForms = 6;  // of one head_dim, at most
const Kernel kKernels[3][kForms] = {{{{64, 4, false, false}, 1, 0.478, 5.0, 0, 0.750, 2.00, 0.59},  // head_dim 64
                                     {{64, 2, false, false}, 3, 1.175, 6.1, 0.72, 0.754, 1.58, 1.09},
                                     {{128, 1, false, false}, 3, 2.130, 4.7, 0.72, 0.765, 1.02, 2.15},
                                     {{256, 1, true, true}, 2, 2.675, 3.9, 0.74, 0.779, 0.50, 3.46},
                                     {{384, 1, true, false}, 1, 2.022, 1.7, 0, 0.774, 1.10, 3.00},
                                     {{0, 0, false, false}, 0, 0, 0, 0, 0, 0, 0}},
                                    {{{64, 4, false, false}, 1, 0.630, 6.0, 0, 0.704, 2.00, 0.72},  // head_dim 96
                                     {{64, 2, false, false}, 2, 1.156, 7.2, 0.66, 0.696, 1.49, 1.13},
                                     {{128, 1, false, false}, 3, 2.844, 7.4, 0.77, 0.725, 1.14, 2.38},
                                     {{256, 1, false, false}, 1, 1.923, 4.7, 0, 0.692, 1.40, 2.53},
                                     {{256, 1, true, false}, 1, 1.901, 6.2, 0, 0.735, 1.19, 2.65},
                                     {{384, 1, true, true}, 1, 2.505, 3.2, 0, 0.768, 1.22, 3.29}},
                                    {{{64, 4, false, false}, 1, 0.753, 7.6, 0, 0.714, 2.00, 0.87},  // head_dim 128
                                     {{64, 2, false, false}, 2, 1.409, 8.5, 0.69, 0.715, 1.30, 1.33},
                                     {{128, 1, false, false}, 2, 2.430, 7.5, 0.73, 0.728, 1.20, 2.44},
                                     {{256, 1, false, false}, 1, 2.250, 7.1, 0, 0.707, 1.23, 2.70},
                                     {{256, 1, true, false}, 1, 2.196, 6.8, 0, 0.762, 1.07, 2.85},
                                     {{384, 1, true, true}, 1, 3.043, 6.3, 0, 0.775, 1.22, 3.70}}};
// 64 rows, keys split two ways, at head_dim 96 where three workgroups to a CU make one round (three_to_a_cu).  Fitted to the sizes of the
// sweep at which three are taken.  With the numbers of two the model is 1.31 too long there: 160 heads of 256 tokens took 256 rows, 18.9
// us, not 13.4, 24 of 1536 33.5, not 24.9.  From three rounds on the numbers of two stay: there 128 rows are even (us, keys split / 128
// rows: 120 heads of 960 50.4 / 51.9, 160 63.5 / 62.0, 72 of 2000 100 / 95).
const Kernel kThreeToACu = {{64, 2, false, false}, 3, 1.525, 6.0, 0.81, 0.70, 1.20, 1.34};
const Chip kChips[3] = {{4.4, 0.51, 0.05, 0.15, 6.1, 0.46, 1.11, 1.02, 0.40, 0.112, -0.048},
                        {3.2, 0.50, 0.13, 0.08, 4.9, 0.30, 1.08, 1.03, 0.52, 0.103, -0.090},
                        {2.6, 0.53, 0.10, 0.08, 6.6, 0.24, 1.07, 1.03, 0.51, 0.087, -0.112}};
int index_of(int D) { return D == 64 ? 0 : D == 96 ? 1 : 2; }
const Kernel* kernels_of(int D) { return kKernels[index_of(D)]; }

}  // namespace

bool find_form(int D, int rows, int key_groups, bool queued, AttnForm* form) {
    const Kernel* of_d = kernels_of(D);
    for (int i = 0; i < kForms; ++i) {
        const AttnForm& f = of_d[i].form;
        if (of_d[i].per_cu > 0 && f.rows == rows && f.key_groups == key_groups && f.queued == queued) {
            *form = f;
            return true;
        }
    }
    return false;
}

namespace {

// Tiles of 64 keys of the compacted sequence that Textural heads walk.
double textural_tiles(const Geometry& g) {
    // rows y and columns x with (y - x) mod tau == 0, by residue
    const int64_t tau = g.tau;
    int64_t kept = 0;
    for (int64_t c = 0; c < std::min<int64_t>(tau, std::min(g.W, g.H)); ++c)
        kept += (g.W - c + tau - 1) / tau * ((g.H - c + tau - 1) / tau);
    return (static_cast<double>(kept) * g.T + g.text_len) / kTileK;
}

// Tiles of 64 keys that a block of `rows` rows visits under each pattern.
struct PatternTiles { double spatial, temporal, textural; };
PatternTiles pattern_tiles(const Geometry& g, int rows, double textural) {
    const double tiles = (g.N + kTileK - 1) / kTileK;
    // a band of radius r over n groups of `group` rows: its share of the pairs, and what blocks and tiles that are not
    // aligned with the groups take in beside it
    auto band = [&](int n, int r, int group) {
        if (r >= n - 1) return tiles;
        const double share = (static_cast<double>(n) * (2 * r + 1) - static_cast<double>(r) * (r + 1)) / (static_cast<double>(n) * n);
        const double beside = rows - std::gcd(rows, group) + kTileK - std::gcd(kTileK, group);
        return std::min(tiles, (share * g.Nv + beside + g.text_len) / kTileK);
    };
    return {band(g.T, g.r_spatial, g.HW), band(g.HW, g.r_temporal, g.T), textural};
}
// The same on the average over the three.
double mean_tiles(const Geometry& g, int rows, double textural) {
    const PatternTiles p = pattern_tiles(g, rows, textural);
    return (p.spatial + p.temporal + p.textural) / 3;
}

// Items of the fullest XCD of a launch from the grid whose heads are nVB + nTB blocks each.
int most_items(const Geometry& g, int BH, int D, bool dense, int nVB, int nTB) {
    return Queues<true>(BH, nVB, nTB, item_order(!whole_heads_fit(g, D), false, dense, BH, static_cast<long long>(nVB + nTB) * BH)).items(0);
}

// Time of a launch in form k, us; HUGE_VAL if the form is not to be taken at this size.  textural: textural_tiles(g).
double launch_us(const Kernel& of_form, const Geometry& g, int BH, int D, bool dense, double textural) {
    constexpr int kCUs = 256;  // MI355X
    const bool one_round_of_three = D == 96 && of_form.form.key_groups == 2 && three_to_a_cu(g, BH, dense) &&
                                    static_cast<long long>((g.N + 63) / 64) * BH <= 3 * kCUs;
    const Kernel& k = one_round_of_three ? kThreeToACu : of_form;
    const Chip& chip = kChips[index_of(D)];
    const int rows = k.form.rows;
    if (rows < 256 && g.N > kSmallBlockTokens) return HUGE_VAL;
    if (rows >= 2 * std::max(g.N, kTileK)) return HUGE_VAL;  // half of the block would have no rows
    const int nQB = (g.N + rows - 1) / rows, nTB = g.text_len > 0 ? nQB - g.Nv / rows : 0, nVB = nQB - nTB;
    const bool far = !whole_heads_fit(g, D);
    const double tiles = (g.N + kTileK - 1) / kTileK, slots = static_cast<double>(kCUs) * k.per_cu;
    const double items = static_cast<double>(nQB) * BH, longs = dense ? 0 : static_cast<double>(nTB) * BH;
    const double tile_us = k.tile_us * (dense ? k.dense : 1) * (!far || k.form.queued ? 1 : dense ? chip.far_dense : chip.far);
    const double item = (dense ? tiles : mean_tiles(g, rows, textural)) * tile_us + k.item_us;
    const double text_item = tiles * tile_us * k.text + k.item_us;
    double rounds = items / slots;
    if (!k.form.queued) {  // what the fullest XCD has to do; beyond some thousand heads all are equally full
        const int heads = std::min(BH, 4096);
        rounds = 8.0 * most_items(g, heads, D, dense, nVB, nTB) * (static_cast<double>(BH) / heads) / slots;
    }
    rounds *= 1 + longs / items * (text_item / item - 1);
    // how long an item takes where n workgroups share the chip, relative to a full one
    auto shared = [&](double n) { return 1 - k.spread * (1 - std::min<double>(k.per_cu, std::ceil(n / kCUs)) / k.per_cu); };
    const double full = std::floor(rounds), rest = rounds - full;
    double length = full > 0 ? full : shared(rest * slots);
    if (full > 0 && rest > 0) {
        const double even = dense ? chip.smooth_dense : std::min(1.0, chip.smooth + chip.smoother * (full - 1));
        length += shared(rest * slots) * (1 - even) + rest * even;
    }
    double us = item * length * (1 - (dense ? chip.many_dense : chip.many) * (1 - 1 / std::max(1.0, rounds)));
    if (longs > 0) us = std::max(us, k.text_tile_us * tiles * (chip.alone + (1 - chip.alone) * std::min(1.0, items / slots)) + k.item_us);
    us += chip.start_us + (k.form.queued ? chip.queue_us : 0);
    if (k.form.copies && !dense) us += 3 + chip.copy_us * (2. / 3) * 8e-6 * BH * g.N * D;  // two patterns in three walk copies
    return us;
}

// The form of least cost(form) among those of head_dim D, copies: with those that walk copies of K and V.
template <typename F>
AttnForm cheapest(int D, bool copies, F cost) {
    const Kernel* of_d = kernels_of(D);
    const Kernel* best = nullptr;
    double least = 0;
    for (int i = 0; i < kForms; ++i) {
        const Kernel& k = of_d[i];
        if (k.per_cu == 0 || (k.form.copies && !copies)) continue;
        const double c = cost(k);
        if (!best || c < least) {
            best = &k;
            least = c;
        }
    }
    return best->form;
}

}  // namespace

// A call whose heads have classes on the device may be all dense (a program that runs the first tenth of its steps dense
// may say so through the classes), so a tenth of the weight goes to the dense walk.  It decides between forms that are
// nearly even for the patterns; head_dim 64 has the widest gap, 48 heads of 17776 tokens: 128 rows 2163 us with the
// patterns in turn and 4269 dense, 384 2214 and 4052.
static double mixed_cost(const Kernel& k, const Geometry& g, int BH, int D, double textural) {
    const double sparse = launch_us(k, g, BH, D, false, textural), cube = sparse * sparse * sparse;
    return cube * cube * cube * launch_us(k, g, BH, D, true, textural);  // tenth power of the weighted geometric mean
}

// A third workgroup on a CU hides more, but each is slower by itself.  Measured both ways at 5962 drawn sizes (150 to 60000 tokens, 1 to 120
// heads, bandwidths 0.13 to 1/2), each with the classes in turn and with all heads of one (one in ten: profiles/two_or_three_to_a_cu.txt);
// the lines were drawn from 3662 of them, and the other 2300 agree.  Three pay
//   - where they make one round of what two would start a second for, 512 to 768 blocks: without text 1.20 of the speed of two, from 8
//     heads on (below, down to 0.89); with text from 32 heads on, 1.17, with all heads Textural 1.01 (0.90 to 1.2).  With fewer the launch
//     waits for the walks of its text blocks, which visit every tile and take 1.1 times as long with three (Textural 0.94, down to 0.89);
//   - in many rounds: from three on if a text block's tiles are at most 0.9 of what a slot has to visit if all heads are of the shortest
//     pattern (1.08; beyond, down to 0.87), and where 24 heads or more give the text blocks company, from 2.25 on (1.10).
// Between those, 1.5 to 2 rounds: 0.97 to 1.02.  With the classes in turn 1.13 on the mean of the 1830 sizes that take three, the worst
// 0.93, 14 of them below 0.97.  Dense calls: 0.99 below one round, too few of them in this form beyond.
bool three_to_a_cu(const Geometry& g, int BH, bool dense) {
    constexpr int kCUs = 256;  // MI355X
    const double tiles = (g.N + kTileK - 1) / kTileK, items = tiles * BH;  // a block has as many rows as a tile has keys
    if (dense || items <= 2 * kCUs) return false;
    if (items <= 3 * kCUs) return BH >= (g.text_len > 0 ? 32 : 8);
    if (items < 6 * kCUs) return BH >= 24 && items >= 4.5 * kCUs;
    if (BH >= 24 || g.text_len == 0) return true;
    const PatternTiles p = pattern_tiles(g, kTileK, textural_tiles(g));
    return tiles <= 0.9 * items / (2 * kCUs) * std::min({p.spatial, p.temporal, p.textural});
}

AttnForm choose_form(const Geometry& g, int BH, int D, bool dense, bool room) {
    // Few blocks: two workgroups to each, whose wavefronts have tiles of their own (launch_items_d).  The model does not know
    // them, and need not: on this side of the line they are the fastest at all 111 sizes of the sweep, by up to 1.5 (2 heads of 1536
    // tokens at head_dim 64, 9.7 us against 14.4 with the keys split two ways), and 1.00-1.33 times as fast as what the model takes at
    // 180 drawn ones; with one or two tiles, which leave groups idle, 0.92 at worst.
    const int nQB = (g.N + kTileK - 1) / kTileK, nTB = g.text_len > 0 ? nQB - g.Nv / kTileK : 0;
    AttnForm few;
    if (nQB >= 3 && static_cast<long long>(nQB) * BH <= 8 * 16 && halves_have_cus(most_items(g, BH, D, dense, nQB - nTB, nTB)) && find_form(D, 64, 4, false, &few)) return few;
    const double textural = textural_tiles(g);
    // without room a form with copies would walk Temporal heads in token order: up to twice the time
    return cheapest(D, room || dense, [&](const Kernel& k) { return dense ? launch_us(k, g, BH, D, true, textural) : mixed_cost(k, g, BH, D, textural); });
}

AttnForm choose_fixed_form(const Geometry& g, int D) {
    const double textural = textural_tiles(g);
    return cheapest(D, false, [&](const Kernel& k) {
        double product = 1;  // of numbers below 1e10 ^ 10 each at any size that runs
        for (int heads : {12, 24, 48}) product *= std::pow(mixed_cost(k, g, heads, D, textural), 0.1);
        return product;
    });
}

// cls in the public numbering: a head class, or RF_LIST_TEMPORAL_POSITION_MAJOR
void flatten_class(const HostPlan& P, int cls, std::vector<int32_t>* row_ptr, std::vector<int32_t>* cols) {
    const int list = cls == RF_LIST_TEMPORAL_POSITION_MAJOR ? kListTemporalPM : cls;
    row_ptr->assign(P.nQB + 1, 0);
    cols->clear();
    for (int qb = 0; qb < P.nQB; ++qb) {
        if (cls == RF_DENSE || (cls == RF_TEXTURAL && qb < P.first_text_qb)) {
            const int nt = cls == RF_DENSE ? P.nKT : P.nCT;
            const int len = cls == RF_DENSE ? P.g.N : P.Nc;
            for (int kt = 0; kt < nt; ++kt)
                cols->push_back(kt | ((kt + 1) * kTileK > len ? RF_PLAN_PARTIAL : 0));
        } else {
            for (int e = P.row_ptr[list][qb]; e < P.row_ptr[list][qb + 1]; ++e)
                cols->push_back(P.cols[list][e] & ~kTileBoundary);
        }
        (*row_ptr)[qb + 1] = static_cast<int32_t>(cols->size());
    }
}

}  // namespace rf
