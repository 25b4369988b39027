// Internal declarations shared by the host side (argument checks, block lists) and the
// HIP kernels of the RainFusion library.  Not part of the public ABI.
#pragma once
#include <cstddef>
#include <cstdint>
#include <vector>

#include "rainfusion.h"

namespace rf {

constexpr int kTileK = 64;  // keys per LDS tile of the attention and ARM kernels
constexpr int kMaxBw = RF_MAX_BANDWIDTHS;  // candidate bandwidths of the per-head bandwidth variant

// Flags on a key-tile entry of a block list (RF_PLAN_PARTIAL is public).
constexpr int32_t kTileBoundary = 0x20000000;  // tile holds text keys or runs past the last key
constexpr int32_t kTileIndexMask = 0x1fffffff;

// Resolved, validated problem description.
struct Geometry {
    int T, H, W, text_len;
    int HW, Nv, N;
    int r_spatial, r_temporal;  // band half-widths in frames / in-frame positions
    int tau;                    // checkerboard stride (Eq. 4)
    int omega;                  // global sampling interval (Sec. 3.3)
    int two_head;               // ARM fallback class is DENSE instead of TEXTURAL
    int text_first;             // text tokens are the first rows of the tensors instead of the last

    // Lists, attributes and orders are all built on the WALKED order: video tokens 0 .. Nv-1, then
    // text.  row_of() gives the tensor row of a walked index (the identity unless text_first).
    int video_shift() const { return text_first ? text_len : 0; }  // added to a walked video index
    int text_shift() const { return text_first ? -Nv : 0; }        // added to a walked text index
    int row_of(int n) const { return n + (n < Nv ? video_shift() : text_shift()); }
};

// Lists: 0/1/2 = Spatial / Temporal / Textural in token order; 3 = Temporal in POSITION-MAJOR
// order (video token (frame f, position p) sits at p*T + f, text tokens stay last), where the
// Temporal band |p_i - p_j| <= r is one contiguous run of keys per query block.
constexpr int kLists = 4;
constexpr int kListTemporalPM = 3;

// What the attention kernel needs of a layout whatever the block size: one entry per token.
struct TokenTables {
    // per row of the list's order: frame index / in-frame index / 0 if kept by Eq. 4 else 1 / in-frame index
    std::vector<int32_t> attr[kLists];
    std::vector<int32_t> cidx;      // compacted position -> tensor row (Textural): kept video keys, then text keys
    std::vector<int32_t> pm_token;  // position-major row -> tensor row
};

// Host copy of the block lists of one block size.
struct HostPlan {
    Geometry g;
    int block;     // query rows per block = rows one workgroup owns
    int nQB;       // ceil(N / block)
    int nKT;       // ceil(N / kTileK): key tiles of the token sequence
    int Nc;        // compacted key count of the Textural pattern: kept video keys + text keys
    int nCT;       // ceil(Nc / kTileK): key tiles of the compacted sequence
    int first_text_qb;  // first query block holding a text row (nQB if there is none)
    // CSR lists of key tiles per query block; Textural: text-holding query blocks only
    std::vector<int32_t> row_ptr[kLists], cols[kLists];
    // Scheduling of a head's query blocks (affects cache behaviour only, never the result), per list:
    // qorder = the order in which blocks are handed out (a permutation; XCD x takes ordinals
    // [x * ceil(nQB/8), (x+1) * ceil(nQB/8)) of it), first_entry = the entry of its list a block starts
    // its (cyclic) walk at.
    std::vector<int32_t> qorder[kLists];
    std::vector<int32_t> first_entry[kLists];
};

// Fills g from layout/params (params may be null -> paper defaults). Returns an rf_status.
int resolve_geometry(const rf_layout* layout, const rf_params* params, Geometry* g);

// Builds the token tables and the block lists. Pure host code.  token_order_temporal: also the Temporal list in token
// order, the longest to build, which only RF_FLAG_WIDE_ROWS walks; banded: the Spatial list and the Temporal one in
// position-major order.  Without them those lists are empty.
void build_tables(const Geometry& g, TokenTables* tables);
void build_plan(const Geometry& g, const TokenTables& tables, int block, bool token_order_temporal, HostPlan* plan, bool banded = true);
void build_plan(const Geometry& g, int block, HostPlan* plan);  // tables of its own, every list

// How an attention call runs: query rows a workgroup takes at a time (64, 128, 256 or 384), groups of its
// wavefronts that split the keys (4, 2 or 1), whether a resident set of workgroups takes items from queues or every
// item has a workgroup, and whether the kernel profits from copies of K and V.
struct AttnForm {
    int rows, key_groups;
    bool queued, copies;
};
// Whole heads to an XCD (every L2 then fetches a head's K and V once) as long as the eight heads in work fit the
// memory-side cache with room to spare: 1-20 % up to 17776 tokens; beyond, all XCDs on one head at a time.
inline bool whole_heads_fit(const Geometry& g, int D) { return 8 * 2 * static_cast<size_t>(g.N) * D * sizeof(uint16_t) <= (size_t{128} << 20); }

// Forms of fewer than 256 rows are taken up to here (beyond, one head fills the chip with larger blocks), so that the
// lists of 64- and 128-row blocks, which grow with the square of the length, need not exist for longer sequences.
constexpr int kSmallBlockTokens = 1 << 17;
// The form with the shortest launch at this size.  dense: every head is known to be dense; room: there is a
// workspace for the copies.
AttnForm choose_form(const Geometry& g, int BH, int D, bool dense, bool room);
// The same from the layout and head_dim alone, for RF_FLAG_FIXED_ORDER: a form decides the order in which a row's tiles
// are summed up, so a head's bits are the same in any batch, on any share of the heads and with any workspace only if
// none of these decides the form.  Without copies, and best on the (geometric) mean of 12, 24 and 48 heads.
AttnForm choose_fixed_form(const Geometry& g, int D);
// Keys split two ways at head_dim 96: whether three workgroups to a CU (three wavefronts a SIMD) are faster than two.
bool three_to_a_cu(const Geometry& g, int BH, bool dense);
// The form with these numbers, if head_dim D has one.
bool find_form(int D, int rows, int key_groups, bool queued, AttnForm* form);

// Block list of one class as the kernel walks it (see rf_plan_host in rainfusion.h).
void flatten_class(const HostPlan& plan, int cls, std::vector<int32_t>* row_ptr, std::vector<int32_t>* cols);

// Device-resident plan: raw device pointers into one allocation.
struct DevicePlan {
    const int32_t* row_ptr[kLists];
    const int32_t* cols[kLists];
    const int32_t* attr[kLists];
    const int32_t* qorder[kLists];
    const int32_t* first_entry[kLists];
    const int32_t* cidx;
    const int32_t* pm_token;
    int radius[kLists];
    int group_rows[kLists];  // rows per frame (Spatial), per position (Temporal in position-major order)
    int video_shift, text_shift;  // tensor row = walked index + (index < Nv ? video_shift : text_shift)
    int N, Nv, Nc;
    int block, nQB, nKT, nCT, first_text_qb;
};

// All plans of one call share the layout and the checkerboard; they differ in the band widths.
struct AttnArgs {
    const uint16_t* Q;
    const uint16_t* K;
    const uint16_t* V;
    uint16_t* O;
    const int32_t* head_class;  // null: every head dense
    int BH;            // B * nH
    float scale_log2;  // log2(e) / sqrt(D)
    // optional: packed copies of K and V, [BH][N][D] each: the kept rows of Textural heads (first Nc rows),
    // all rows of Temporal heads in position-major order; null: no packing
    uint16_t* packed_k;
    uint16_t* packed_v;
    const int32_t* head_bw;  // optional per-head index into plan[]; null or out of range: plan[0]
    int* queue;              // 8 work-queue counters (one per XCD) and 64 sweep words (8 per XCD) at the start of the caller's workspace, reset by the launcher
    int item_order;          // ORDER_*: which items an XCD takes, and when (rf_queues.h)
    int queued;              // see AttnForm
    int key_groups;          // see AttnForm
    int three_to_a_cu;       // keys split two ways at head_dim 96: see the function of that name
    int wide_rows;           // 1: wavefronts of 64 query rows (256-row blocks only)
    int join_sweep;          // 1: a starting item joins the tile walk of the workgroups already running on its XCD; 0: fixed start
    int n_plans;
    DevicePlan plan[kMaxBw];
};

// One ARM pass = one (sampling, mask) pair: sample a -> video token a * stride, whose attribute is its
// in-frame position (token mod HW) or its frame (token div HW); the mask keeps |attr[a] - attr[b]| <= radius.
struct ArmPass {
    int by_frame;         // 0: attribute = in-frame position (Temporal mask), 1: attribute = frame (Spatial mask)
    int n;                // number of samples
    int stride;           // token stride between samples
    int HW;               // tokens per frame
    int radius[kMaxBw];   // one band half-width per candidate bandwidth
};

struct ArmArgs {
    const uint16_t* Q;
    const uint16_t* K;
    int BH, N;
    int first_video_row;  // tensor row of video token 0
    float scale_log2;
    ArmPass pass[2];   // 0: Temporal mask (R_hat), 1: Spatial mask (R_tilde)
    int n_bw;          // candidate bandwidths (1 for plain Alg. 1)
    int by_width[kMaxBw];  // candidate indices from the narrowest bandwidth to the widest
    float* row_recall; // device [BH][2][n_bw][max_n]: the first ceil(n / 32) of each max_n hold the sums over 32 sampled rows
    int max_n;
    float threshold;
    int fallback_class;   // class of a head that matches neither mask
    int32_t* head_class;  // device [BH]
    int32_t* head_bw;     // device [BH] or null: chosen candidate index, -1 for Textural heads
    float* recalls;       // device [BH][2][n_bw] or null
};

// Kernel launchers (defined in the .hip files). Return a hipError_t as int.
int launch_attention(const AttnArgs& a, int D, void* stream);
int launch_pack_textural(const AttnArgs& a, int D, void* stream);
int launch_arm(const ArmArgs& a, int D, void* stream);
// Device address and size of the library's static scratch array on the current device (rf_arm.hip).
int arm_static_scratch(void** ptr, size_t* bytes);
constexpr size_t kArmStaticScratchBytes = RF_ARM_STATIC_SCRATCH_BYTES;

}  // namespace rf

// rf_sparse_attention_plus (or, with bandwidths and head_bw null, rf_sparse_attention) in the form named instead of
// the one choose_form picks: for tests and measurements, which have to reach every kernel at small sizes.
// RF_ERR_PARAM if the head_dim has no such form, RF_ERR_WORKSPACE if the form walks copies of K and V and the
// workspace has no room for them (and the call is not RF_FLAG_FORCE_DENSE).
extern "C" int rf_internal_attention_as(int rows, int key_groups, int queued, const void* Q, const void* K, const void* V,
                                        const int32_t* head_class, const int32_t* head_bw, const float* bandwidths, int n_bw,
                                        int B, int nH, int D, const rf_layout* layout, const rf_params* params, void* O,
                                        void* workspace, size_t workspace_bytes, void* stream);

// The form a call of rf_sparse_attention with these arguments takes: form[0..3] = query rows per workgroup, groups that
// split the keys, whether from queues, whether K and V are copied.  For tests and measurements.
extern "C" int rf_internal_attention_form(int B, int nH, int D, const rf_layout* layout, const rf_params* params, int block,
                                          size_t workspace_bytes, int32_t* form);
