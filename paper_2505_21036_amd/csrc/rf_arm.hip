// ARM head classifier (Sec. 3.3, Eq. 6, Alg. 1) on gfx950.
//
// Pass 0 measures the recall of the Temporal mask (R-hat), pass 1 that of the Spatial mask
// (R-tilde).  A pass is described by its sample (sample a is token a * stride), an integer
// attribute per sample (in-frame position, resp. frame index) and a radius: the mask keeps
// |attr[a] - attr[b]| <= radius.  The scores Q'K'^T / sqrt(D) are formed tile by tile with
// bf16 MFMA and never stored; the sampled K' rows go global -> LDS one tile ahead, gathered by
// index arithmetic (no copy of Q', K' is made).  Per sampled query the kernel keeps a reference for
// the exponent, the softmax denominator over all sampled keys (M_init) and the part of it on kept
// keys (M').  The masks are bands on the attribute, so for most (32 queries, 64 keys) pairs every
// entry is kept or every entry is dropped; the kernel tells from the attribute ranges of the two
// sides and applies the mask entry by entry only where the band's edge crosses the pair.
// A sample's attribute (in-frame position or frame) follows from its index by arithmetic; no table of
// samples exists anywhere.  The recalls' sums over 32 rows go to scratch and are reduced in a fixed order by
// arm_finish_kernel, which also applies the decision rule.
//
// Bound by vector issue (about eight vector instructions per MFMA; each score costs a maximum, an exponent and a
// sum, and three more per pass where a band's edge crosses its tile: the Temporal band does in every tile at equal
// intervals).  Measured, recall and finish, us:
//   24 heads of 3600 samples at head_dim 128, equal intervals 257 with the mask applied to every score, 161 with the edges told
//   apart, 151 with three instructions there instead of four, 149.5 with the scores at raised priority too, 133 with all reads of
//   the table of attributes asked for before the first is used (each was waited for by itself), positions carried from tile to
//   tile instead of divided out, and the radius of a call with one bandwidth in a register; first frame 249, 215, 213, 213 and
//   200 (a pass of its own needs no table at all)
//   three candidates 252 -> 197; head_dim 96, 24 heads of 3600, equal 141 -> 120, first 188 -> 169; head_dim 64, 48 of 1350, 54.9 -> 44.7
//   and 62.1 -> 51.4; 24 of 448 at head_dim 96 39.9, 13.8 and 11.9 now, first 29.0, 16.2 and 13.5; 40 heads of 2800 at head_dim 64,
//   four candidates, 282 -> 199
// Also tried: the products of the next tile dealt out between the sums of this one, 1.0-1.03 at head_dim 64 and 96 and 0.96 at 128 of
// the same time, where the second set of scores spills; the differences of the attributes from the matrix unit, 1.00.
#include <cfloat>
#include <mutex>
#include <type_traits>

#include "rf_device.h"

namespace rf {

// A workgroup is KS groups of R wavefronts, 32 sampled queries each; the groups hold the same queries and split
// the sampled keys.  Large samples: one group of four (eight measured 1-17 % slower, two at once on a CU leave
// coarser steps).  Small ones, which would leave most CUs with one workgroup or none: four groups of two.
constexpr int kArmWaves = 4, kArmSplitWaves = 2, kArmSplit = 4;
// Up to this many workgroups of the first kind (128 queries of one head, and of one pass unless both share the
// sample) the second kind is taken: 96 workgroups with both passes 23.0 -> 14.6 us, 256: 41.2 -> 35.7, 528: 60 ->
// 100; one pass each, 120: 19.5 -> 14.2, 192: 16.6 -> 20.2.
constexpr int kArmSplitItemsBoth = 256, kArmSplitItemsApart = 128;
// as in the attention kernel: the reference in the exponent moves only when a row outgrows it by this
constexpr float kArmRescaleSlack = 8.f;

// Wavefronts per SIMD the register allocation is held to: what the tile loop fits without spills (head_dim 96, one pass,
// several candidates: four with a few registers spilled outside the loop; head_dim 128: four for one pass with one
// bandwidth, 198.7 -> 196.4 us for 24 heads of 3600 samples).
constexpr int arm_waves_per_simd(int D, bool both, int KS, int NB) { return KS > 1 ? 2 : (both ? (D == 64 ? 4 : 3) : (D == 128 && NB > 1 ? 3 : 4)); }

template <int D, int R, int KS>
struct ArmSmem {
    using ST = DirectTile<D, R>;
    // per group: two K' tiles, then per tile and pass the 64 samples' attributes (float)
    static constexpr int ATTR_SLOT = kTileK;
    static constexpr int ATTR_OFF = 2 * ST::K_BYTES;
    static constexpr int GROUP_BYTES = (ATTR_OFF + 2 * 2 * ATTR_SLOT * 4 + 255) / 256 * 256;
    static constexpr int BYTES = KS * GROUP_BYTES;
    // at the end the groups exchange, per query, reference, denominator and kept sums where the tiles were
    static constexpr int PART = 2 + 2 * kMaxBw;
    static_assert(R * PART * 32 * 4 <= 2 * ST::K_BYTES, "the exchange fits the tile buffers");
    static_assert(ST::K_BYTES % 256 == 0, "tile buffers must start at multiples of 256 bytes (see DirectTile::k_address)");
};

// BOTH: the two passes use the same sample (equal-interval sampling), so one workgroup forms each
// score tile once and keeps the kept-key sums of both masks; the arithmetic per pass, and so every
// recall, is the same as when the passes run apart.
// NB: candidate bandwidths there is room for (1 or kMaxBw).
template <int D, bool BOTH, int R, int KS, int NB>
__global__ void __launch_bounds__(64 * R * KS) __attribute__((amdgpu_waves_per_eu(arm_waves_per_simd(D, BOTH, KS, NB), arm_waves_per_simd(D, BOTH, KS, NB)))) arm_recall_kernel(ArmArgs a, int nQB) {
    constexpr int BQ = 32 * R, NP = BOTH ? 2 : 1;
    using SM = ArmSmem<D, R, KS>;
    using ST = typename SM::ST;
    typedef __attribute__((address_space(3))) float lds_float;
    typedef __attribute__((address_space(3))) const f32x4 lds_f32x4;
    extern __shared__ __attribute__((aligned(256))) unsigned char smem_all[];  // the kernel's only LDS: starts at address 0
    const int group = KS == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / (64 * R));
    unsigned char* smem = smem_all + group * SM::GROUP_BYTES;
    int* abuf = reinterpret_cast<int*>(smem + SM::ATTR_OFF);

    const int item = xcd_contiguous_item(blockIdx.x, nQB * (2 / NP) * a.BH);
    if (item < 0) return;
    const int qb = item % nQB, pass0 = BOTH ? 0 : (item / nQB) & 1, bh = item / ((2 / NP) * nQB);
    ArmPass ps[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) ps[i] = a.pass[pass0 + i];
    const int n = ps[0].n, stride = ps[0].stride;  // BOTH: the same in the two passes (the host checks)
    if (qb * BQ >= n) return;
    const int tid = threadIdx.x - group * (64 * R), lane = tid & 63, wave = tid >> 6, hf = lane >> 5, m = lane & 31;

    // samples are video tokens; first_video_row is where those start in the tensors
    const size_t head_off = (static_cast<size_t>(bh) * a.N + a.first_video_row) * D;
    const uint16_t* Qh = a.Q + head_off;
    const unsigned char* Kh = reinterpret_cast<const unsigned char*>(a.K + head_off);

    const int qs = qb * BQ + wave * 32 + m;  // this lane's sampled query
    const int qsc = min(qs, n - 1);
    bf16x8 qf[D / 16];
    load_q_frags<D>(Qh, qsc * stride, hf, qf);
    auto attr_of = [&](int i, int sample) {
        const int token = sample * stride;
        return ps[i].by_frame ? token / ps[i].HW : token % ps[i].HW;
    };
    // With one candidate bandwidth, a query's kept samples are one run of sample indices if the attribute rises with
    // the index: frames always, positions where the passes have samples of their own (pass 0 then the first frame's).
    // Then lo .. hi, and no table is needed.  Otherwise the attributes of a tile's samples are compared with the query's.
    constexpr auto is_run = [](int i) { return NB == 1 && (!BOTH || i == 1); };
    const int n_bw = NB == 1 ? 1 : a.n_bw;
    int q_attr[NP], lo[NP], hi[NP];
    // range of the attribute over the wavefront's 32 queries (both halves hold the same queries)
    int q_min[NP], q_max[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        q_attr[i] = attr_of(i, qsc);
        int low = q_attr[i], high = q_attr[i];
#pragma unroll
        for (int w = 1; w < 32; w <<= 1) {
            low = min(low, __shfl_xor(low, w, 64));
            high = max(high, __shfl_xor(high, w, 64));
        }
        q_min[i] = __builtin_amdgcn_readfirstlane(low);
        q_max[i] = __builtin_amdgcn_readfirstlane(high);
        const int r = ps[i].radius[0];
        if (ps[i].by_frame) {  // samples whose token lies in frames q_attr - r .. q_attr + r
            lo[i] = static_cast<int>((static_cast<long long>(max(q_attr[i] - r, 0)) * ps[i].HW + stride - 1) / stride);
            hi[i] = static_cast<int>((static_cast<long long>(q_attr[i] + r + 1) * ps[i].HW - 1) / stride);
        } else {
            lo[i] = q_attr[i] - r;
            hi[i] = q_attr[i] + r;
        }
    }

    // m_ref: reference subtracted inside exp2, in the units of its argument (score times c, which is below 1);
    // kNoReference, which any finite score outgrows, until it has been taken from one; l_all / l_kept: this lane's share of
    // the denominator over all sampled keys and over the kept ones, both relative to m_ref
    constexpr float kNoReference = -FLT_MAX;
    float m_ref = kNoReference, l_all = 0.f, l_kept[NP][NB];
#pragma unroll
    for (int i = 0; i < NP; ++i)
#pragma unroll
        for (int b = 0; b < NB; ++b) l_kept[i][b] = 0.f;
    const float c = a.scale_log2;
    const int all_tiles = (n + kTileK - 1) / kTileK;
    const int ntiles = (all_tiles - group + KS - 1) / KS, nsteps = (all_tiles + KS - 1) / KS;  // this group's; the longest's

    ST st;
    st.init(tid);
    auto first_of = [&](int t) { return (t * KS + group) * kTileK; };  // the group's t-th tile starts at this sample
    auto k_lds = [&](int t) { return smem + (t & 1) * ST::K_BYTES; };
    auto attr_slot = [&](int t, int i) { return abuf + ((t & 1) * 2 + i) * SM::ATTR_SLOT; };
    auto fetch_tile = [&](int t) {
        const int k0 = first_of(t);
        if (stride == 1 && k0 + kTileK <= n)
            st.template issue_consecutive<false>(Kh + static_cast<size_t>(k0) * (2 * D), nullptr, k_lds(t), nullptr);
        else
            st.template issue<false>(Kh, nullptr, k_lds(t), nullptr, [&](int r) { return min(k0 + r, n - 1) * stride; });
    };
    // Where samples are told apart by a table: frame and in-frame position of sample first_of(t) + lane of the tile t last
    // stashed, and of the tile worked on its first sample's, both moved on from tile to tile without a division.  Samples
    // past the last one go on in the same way: their weights are 0, and bounds that take them in are only too wide.
    // (A stride beyond the last token leaves one sample, and the products below 2^32.)
    const unsigned HW = ps[0].HW, hop = min(stride, a.N), step = kTileK * KS * hop;
    const int span = (kTileK - 1) * hop, span_frames = span / HW, span_rest = span % HW, step_frames = step / HW, step_rest = step % HW;
    auto advance = [&](int& frame, int& at) {
        at += step_rest;
        frame += step_frames;
        if (at >= static_cast<int>(HW)) {
            at -= HW;
            ++frame;
        }
    };
    int own_frame = (first_of(0) + lane) * hop / HW, own_at = (first_of(0) + lane) * hop % HW;
    int tile_frame = first_of(0) * hop / HW, tile_at = first_of(0) * hop % HW;
    auto stash_attr = [&](int t) {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            if (is_run(i)) continue;
            if (tid < kTileK) attr_slot(t, i)[tid] = __float_as_int(static_cast<float>(ps[i].by_frame ? own_frame : own_at));
        }
        advance(own_frame, own_at);
    };
    if (ntiles > 0) {
        fetch_tile(0);
        stash_attr(0);
    }
    ST::template wait_landed<0>();
    __syncthreads();
    // the compiler cannot see the tile loads; make its own wait for the Q loads happen here, not in the loop
#pragma unroll
    for (int cc = 0; cc < D / 16; ++cc) asm volatile("" ::"v"(__builtin_bit_cast(u32x4, qf[cc])));

    for (int t = 0; t < nsteps; ++t) {
        if (t + 1 < ntiles) fetch_tile(t + 1);
        if (KS == 1 || t < ntiles) {
            const int k0 = first_of(t);

            f32x16 s[2];
            // the wavefronts of a SIMD leave the barrier together: one that forms scores goes before one in its sums, so
            // that the matrix pipe works while others use the vector unit
            __builtin_amdgcn_s_setprio(1);
            st.template scores<kAheadK>(st.k_address(k_lds(t)), qf, s);
            __builtin_amdgcn_s_setprio(0);
            if (k0 + kTileK > n) {  // ragged last tile: samples past the end do not exist
                int end = n - k0 - 8 * hf;
#pragma unroll
                for (int kb2 = 0; kb2 < 2; ++kb2)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        if (32 * kb2 + key_of_reg(r, 0) >= end) s[kb2][r] = -INFINITY;
                        if ((r & 3) == 3) asm volatile("" : "+v"(end));  // few comparisons' results at a time
                    }
            }
            float mt = s[0][0];
#pragma unroll
            for (int kb2 = 0; kb2 < 2; ++kb2)
#pragma unroll
                for (int r = 0; r < 16; ++r) mt = fmaxf(mt, s[kb2][r]);
            // the two halves of the wavefront hold different keys of the same 32 queries: their maxima are
            // exchanged, and the sums rescaled, only when some lane asks for the reference to move
            if (__builtin_amdgcn_ballot_w64(fmaf(mt, c, -m_ref) > kArmRescaleSlack) != 0) {
                mt = fmaxf(mt, other_half(mt));
                if (mt > -INFINITY) {
                    const float m_new = fmaxf(m_ref, mt * c), alpha = fast_exp2(m_ref - m_new);
                    l_all *= alpha;
#pragma unroll
                    for (int i = 0; i < NP; ++i)
#pragma unroll
                        for (int b = 0; b < NB; ++b) l_kept[i][b] *= alpha;
                    m_ref = m_new;
                }
            }
            // the tile's terms of the denominator, summed in the same order whatever the masks need: four chains,
            // so that an addition need not wait for the one before it
            float part[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kb2 = 0; kb2 < 2; ++kb2)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    s[kb2][r] = fast_exp2(fmaf(s[kb2][r], c, -m_ref));
                    part[r & 3] += s[kb2][r];
                    if ((r & 7) == 7) __builtin_amdgcn_sched_barrier(0);  // keeps the temporaries few
                }
            const float sum_all = (part[0] + part[1]) + (part[2] + part[3]);
            l_all += sum_all;
            // sum of the terms whose place in the tile, counted from this half's first, is from .. to, of which only the ends
            // asked for are looked at; the ends are opaque, or all comparisons are made first and their results kept
            auto sum_of_run = [&](auto look_from, int from, auto look_to, int to) {
                constexpr bool FROM = decltype(look_from)::value, TO = decltype(look_to)::value;
                float k4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kb2 = 0; kb2 < 2; ++kb2)
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        if ((r & 3) == 0) asm volatile("" : "+v"(from), "+v"(to));
                        const int at = 32 * kb2 + key_of_reg(r, 0);
                        k4[r & 3] += (!FROM | (at >= from)) & (!TO | (at <= to)) ? s[kb2][r] : 0.f;
                        if ((r & 3) == 3) asm volatile("" : "+v"(k4[0]), "+v"(k4[1]), "+v"(k4[2]), "+v"(k4[3]));
                    }
                return (k4[0] + k4[1]) + (k4[2] + k4[3]);
            };
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                if (is_run(i)) {
                    // entry (kb2, r) of this lane is sample  k0 + 8*hf + 32*kb2 + 16*(r/8) + r%8
                    const bool all = lo[i] <= k0 && hi[i] >= min(k0 + kTileK, n) - 1, none = hi[i] < k0 || lo[i] >= k0 + kTileK;
                    if (__builtin_amdgcn_ballot_w64(!all) == 0) {
                        l_kept[i][0] += sum_all;
                    } else if (__builtin_amdgcn_ballot_w64(!none) != 0) {
                        const int from = lo[i] - k0 - 8 * hf, to = hi[i] - k0 - 8 * hf;
                        // usually one end of the run lies in the tile for the 32 queries: one comparison each
                        constexpr std::true_type look{};
                        constexpr std::false_type skip{};
                        if (__builtin_amdgcn_ballot_w64(hi[i] < k0 + kTileK - 1) == 0) l_kept[i][0] += sum_of_run(look, from, skip, to);
                        else if (__builtin_amdgcn_ballot_w64(lo[i] > k0) == 0) l_kept[i][0] += sum_of_run(skip, from, look, to);
                        else l_kept[i][0] += sum_of_run(look, from, look, to);
                    }
                    continue;
                }
                // Where does the band's edge fall for this (wavefront, tile) pair?  inside: bit b set if every
                // pair is within radius b; mixed: some candidate has both kept and dropped pairs here.
                // Frames never decrease from sample to sample, and positions do not either inside one frame; a tile that
                // crosses into another frame gets the widest bounds (it is then masked entry by entry, which is exact).
                const int end = tile_at + span_rest >= static_cast<int>(HW) ? 1 : 0;  // of the frame, once more than span_frames times
                const bool crosses = span_frames + end > 0;
                const int k_min = ps[i].by_frame ? tile_frame : crosses ? 0 : tile_at;
                const int k_max = ps[i].by_frame ? tile_frame + span_frames + end : crosses ? static_cast<int>(HW) - 1 : tile_at + span;
                const int reach = max(k_max - q_min[i], q_max[i] - k_min), gap = max(k_min - q_max[i], q_min[i] - k_max);
                int inside = 0;
                bool mixed = false;
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    if (b >= n_bw) break;
                    if (reach <= ps[i].radius[b]) inside |= 1 << b;
                    else if (gap <= ps[i].radius[b]) mixed = true;
                }
                if (!mixed) {
#pragma unroll
                    for (int b = 0; b < NB; ++b) l_kept[i][b] += ((inside >> b) & 1) ? sum_all : 0.f;
                    continue;
                }
                // The attributes are whole numbers below 2^24, exact as floats:  radius + 1 - |difference|, held between 0
                // and 1, is 1 on kept entries and 0 on the others, and the product with it is added exactly as a kept
                // entry would be: three full-rate instructions, two for every further candidate.  All reads of the table are
                // asked for before the first is used.
                const float own = static_cast<float>(q_attr[i]);
                f32x4 apart[8];  // of entries 4 * k to 4 * k + 3
                const uint32_t table = ST::lds_offset(reinterpret_cast<const unsigned char*>(attr_slot(t, i))) + 32 * hf;
#pragma unroll
                for (int k = 0; k < 8; ++k) apart[k] = *(lds_f32x4*)(uintptr_t)(table + 4 * (32 * (k >> 2) + key_of_reg(4 * (k & 3), 0)));
                __builtin_amdgcn_sched_barrier(0);
                if (NB > 1) {
#pragma unroll
                    for (int k = 0; k < 8; ++k)
#pragma unroll
                        for (int j = 0; j < 4; ++j) apart[k][j] -= own;
                }
                auto sum_within = [&](int radius) {
                    const float edge = static_cast<float>(radius + 1);
                    float k4[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int k = 0; k < 8; ++k)
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const float d = NB > 1 ? apart[k][j] : apart[k][j] - own;
                            k4[j] = fmaf(s[k >> 2][4 * (k & 3) + j], __builtin_amdgcn_fmed3f(edge - fabsf(d), 0.f, 1.f), k4[j]);
                        }
                    return (k4[0] + k4[1]) + (k4[2] + k4[3]);
                };
                if constexpr (NB == 1) {
                    l_kept[i][0] += sum_within(ps[i].radius[0]);
                } else {
#pragma clang loop unroll(disable)  // unrolled, more registers
                    for (int b = 0; b < n_bw; ++b) {
                        const float kept = sum_within(a.pass[pass0 + i].radius[b]);
#pragma unroll
                        for (int k = 0; k < NB; ++k) l_kept[i][k] += k == b ? kept : 0.f;
                    }
                }
            }
            advance(tile_frame, tile_at);
        }
        if (t + 1 < ntiles) stash_attr(t + 1);
        ST::template wait_landed<0>();
        __syncthreads();
    }
    // one value per query, in both halves
    l_all += other_half(l_all);
#pragma unroll
    for (int i = 0; i < NP; ++i)
#pragma unroll
        for (int b = 0; b < NB; ++b)
            if (b < n_bw) l_kept[i][b] += other_half(l_kept[i][b]);
    if constexpr (KS > 1) {
        // the first group adds up what the groups found, at the largest of their references
        auto slot = [&](int g, int which) {
            return (lds_float*)(uintptr_t)(ST::lds_offset(smem_all) + g * SM::GROUP_BYTES + ((wave * SM::PART + which) * 32 + m) * 4);
        };
        if (hf == 0) {
            *slot(group, 0) = m_ref;
            *slot(group, 1) = l_all;
#pragma unroll
            for (int i = 0; i < NP; ++i)
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    if (b < n_bw) *slot(group, 2 + i * kMaxBw + b) = l_kept[i][b];
        }
        __syncthreads();
        if (group != 0) return;
        float top = kNoReference;
#pragma unroll
        for (int g = 0; g < KS; ++g) top = fmaxf(top, *slot(g, 0));
        l_all = 0.f;
#pragma unroll
        for (int i = 0; i < NP; ++i)
#pragma unroll
            for (int b = 0; b < NB; ++b) l_kept[i][b] = 0.f;
#pragma unroll
        for (int g = 0; g < KS; ++g) {
            const float w = fast_exp2(*slot(g, 0) - top);
            l_all += w * *slot(g, 1);
#pragma unroll
            for (int i = 0; i < NP; ++i)
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    if (b < n_bw) l_kept[i][b] += w * *slot(g, 2 + i * kMaxBw + b);
        }
    }
    // Eq. 6: one recall per query; the wavefront's 32 are summed in a fixed order and leave as one number
#pragma unroll
    for (int i = 0; i < NP; ++i)
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            if (b >= n_bw) break;
            float sum = qs < n ? l_kept[i][b] / l_all : 0.f;
#pragma unroll
            for (int w = 16; w > 0; w >>= 1) sum += __shfl_xor(sum, w, 64);
            const int at = qb * R + wave;
            if (lane == 0 && at * 32 < n)
                a.row_recall[((static_cast<size_t>(bh) * 2 + pass0 + i) * n_bw + b) * a.max_n + at] = sum;
        }
}

// Mean of the recalls from the wavefronts' sums, in a fixed order, one wavefront per pass and candidate; then
// Alg. 1's rule (with several candidate bandwidths: the narrowest one that holds the threshold, Temporal before
// Spatial).
__global__ void __launch_bounds__(64 * 2 * kMaxBw) arm_finish_kernel(ArmArgs a) {
    __shared__ float rec[2][kMaxBw];
    const int bh = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n_bw = a.n_bw;
    const int pass = wave / kMaxBw, b = wave % kMaxBw;
    if (b < n_bw) {
        const int n = a.pass[pass].n, sums = (n + 31) / 32;
        const float* rr = a.row_recall + ((static_cast<size_t>(bh) * 2 + pass) * n_bw + b) * a.max_n;
        float acc = 0.f;
        for (int i = lane; i < sums; i += 64) acc += rr[i];
#pragma unroll
        for (int w = 32; w > 0; w >>= 1) acc += __shfl_xor(acc, w, 64);
        if (lane == 0) {
            const float mean = acc / static_cast<float>(n);
            rec[pass][b] = mean;
            if (a.recalls) a.recalls[(bh * 2 + pass) * n_bw + b] = mean;
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        int cls = a.fallback_class, chosen = -1;
        for (int p = 0; p < 2 && chosen < 0; ++p)  // Temporal (pass 0) has priority
            for (int i = 0; i < n_bw && chosen < 0; ++i) {
                const int k = a.by_width[i];
                if (rec[p][k] >= a.threshold) {
                    chosen = k;
                    cls = p == 0 ? RF_TEMPORAL : RF_SPATIAL;
                }
            }
        a.head_class[bh] = cls;
        if (a.head_bw) a.head_bw[bh] = chosen;
    }
}

template <int D, bool BOTH, int R, int KS, int NB>
static int launch_recall_nb(const ArmArgs& a, hipStream_t st) {
    const int nQB = (a.max_n + 32 * R - 1) / (32 * R), total = nQB * (BOTH ? 1 : 2) * a.BH;
    constexpr int smem = ArmSmem<D, R, KS>::BYTES;
    if (smem > 64 * 1024) {  // above what a kernel may have by itself: once per device
        constexpr int kMaxDevices = 64;
        static std::mutex mu;
        static bool ready_on[kMaxDevices] = {};
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return static_cast<int>(e);
        if (dev < 0 || dev >= kMaxDevices) return static_cast<int>(hipErrorInvalidDevice);
        std::lock_guard<std::mutex> lock(mu);
        if (!ready_on[dev]) {
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(&arm_recall_kernel<D, BOTH, R, KS, NB>), hipFuncAttributeMaxDynamicSharedMemorySize, smem);
            if (e != hipSuccess) return static_cast<int>(e);
            ready_on[dev] = true;
        }
    }
    hipLaunchKernelGGL((arm_recall_kernel<D, BOTH, R, KS, NB>), dim3(8 * ((total + 7) / 8)), dim3(64 * R * KS), smem, st, a, nQB);
    return static_cast<int>(hipGetLastError());
}

template <int D, bool BOTH, int R, int KS>
static int launch_recall(const ArmArgs& a, hipStream_t st) {
    return a.n_bw == 1 ? launch_recall_nb<D, BOTH, R, KS, 1>(a, st) : launch_recall_nb<D, BOTH, R, KS, kMaxBw>(a, st);
}

template <int D>
static int launch_arm_d(const ArmArgs& a, hipStream_t st) {
    const bool both = a.pass[0].n == a.pass[1].n && a.pass[0].stride == a.pass[1].stride;  // one sample for the two passes
    const long long items = static_cast<long long>((a.max_n + 32 * kArmWaves - 1) / (32 * kArmWaves)) * a.BH * (both ? 1 : 2);
    const bool split = items <= (both ? kArmSplitItemsBoth : kArmSplitItemsApart);
    int e;
    if (split)
        e = both ? launch_recall<D, true, kArmSplitWaves, kArmSplit>(a, st) : launch_recall<D, false, kArmSplitWaves, kArmSplit>(a, st);
    else
        e = both ? launch_recall<D, true, kArmWaves, 1>(a, st) : launch_recall<D, false, kArmWaves, 1>(a, st);
    if (e != 0) return e;
    hipLaunchKernelGGL(arm_finish_kernel, dim3(a.BH), dim3(64 * 2 * kMaxBw), 0, st, a);
    return static_cast<int>(hipGetLastError());
}

// Scratch for callers that cannot allocate (rf_arm_classify_noalloc): lives in the library's image on
// every GPU the library runs on, at an address that differs from device to device.
static __device__ __align__(256) unsigned char scratch[kArmStaticScratchBytes];

int arm_static_scratch(void** ptr, size_t* bytes) {
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void* address[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return static_cast<int>(e);
    if (dev < 0 || dev >= kMaxDevices) return static_cast<int>(hipErrorInvalidDevice);
    std::lock_guard<std::mutex> lock(mu);
    if (!address[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));  // with device `dev` current: that device's copy
        if (e != hipSuccess) return static_cast<int>(e);
        address[dev] = p;
    }
    *ptr = address[dev];
    *bytes = kArmStaticScratchBytes;
    return 0;
}

int launch_arm(const ArmArgs& a, int D, void* stream) {
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (D == 64) return launch_arm_d<64>(a, st);
    if (D == 96) return launch_arm_d<96>(a, st);
    if (D == 128) return launch_arm_d<128>(a, st);
    return static_cast<int>(hipErrorInvalidValue);
}

}  // namespace rf
