// C ABI of the RainFusion library: argument checks, the cache of device-resident block
// lists, and the two entry points.  All checks run before the first HIP call, so they can
// be exercised on a machine without a GPU.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <vector>

#include "rf_internal.h"
#include "rf_queues.h"

namespace rf {
namespace {

// The lists of one (layout, params): of every block size, so that whichever form a later call takes (it depends on the
// number of heads, the head_dim, the workspace and the dense flag) finds its lists there.  A call captured into a graph
// may not build any.
constexpr int kBlocks[] = {64, 128, 256, 384};
constexpr int kBlockSizes = 4;
struct CachedPlan {
    Geometry g;       // with the fields the lists do not depend on zeroed (see list_key)
    bool wide;        // for RF_FLAG_WIDE_ROWS: 256-row blocks only, and the Temporal list in token order
    int device;
    unsigned long long last_use = 0;
    void* blob = nullptr;
    DevicePlan dev[kBlockSizes] = {};
};

std::mutex g_mu;
std::vector<std::unique_ptr<CachedPlan>> g_plans;
unsigned long long g_use_counter = 0;
constexpr size_t kMaxCachedPlans = 16;  // per process; the least recently used one makes room

// The block lists depend on the layout, the band widths, the checkerboard stride and the placement
// of the text tokens, not on the ARM's sampling interval or its fallback class.
Geometry list_key(Geometry g) {
    g.omega = 0;
    g.two_head = 0;
    return g;
}

bool same_geometry(const Geometry& a, const Geometry& b) { return std::memcmp(&a, &b, sizeof(Geometry)) == 0; }

CachedPlan* find_plan(const Geometry& g, bool wide, int device) {
    for (auto& p : g_plans)
        if (p->wide == wide && p->device == device && same_geometry(p->g, g)) return p.get();
    return nullptr;
}

// Lays vectors out in one device allocation, each at a multiple of 256 bytes.
struct BlobBuilder {
    struct Part { const std::vector<int32_t>* v; size_t at; };
    std::vector<Part> parts;
    size_t words = 0;
    size_t add(const std::vector<int32_t>& v) {  // v must stay as it is until upload()
        const size_t at = words;
        parts.push_back({&v, at});
        words += std::max<size_t>(v.size(), 1);
        words = (words + 63) / 64 * 64;
        return at;
    }
    int upload(void** blob) const {
        std::unique_ptr<int32_t[]> staged(new int32_t[words]);
        for (const Part& p : parts)
            if (!p.v->empty()) std::memcpy(staged.get() + p.at, p.v->data(), p.v->size() * sizeof(int32_t));
        if (hipMalloc(blob, words * sizeof(int32_t)) != hipSuccess) return RF_ERR_HIP;
        if (hipMemcpy(*blob, staged.get(), words * sizeof(int32_t), hipMemcpyHostToDevice) != hipSuccess) {
            (void)hipFree(*blob);
            *blob = nullptr;
            return RF_ERR_HIP;
        }
        return RF_OK;
    }
};

int build_and_upload(const Geometry& g, bool wide, CachedPlan* p) {
    TokenTables tables;
    build_tables(g, &tables);
    HostPlan plans[kBlockSizes];
    BlobBuilder bb;
    struct Offsets { size_t row_ptr[kLists], cols[kLists], qorder[kLists], first_entry[kLists]; } off[kBlockSizes];
    size_t off_attr[kLists];
    for (int c = 0; c < kLists; ++c) off_attr[c] = bb.add(tables.attr[c]);
    const size_t off_cidx = bb.add(tables.cidx), off_pm = bb.add(tables.pm_token);
    auto wanted = [&](int i) { return wide ? kBlocks[i] == 256 : kBlocks[i] >= 256 || g.N <= kSmallBlockTokens; };
    for (int i = 0; i < kBlockSizes; ++i) {
        if (!wanted(i)) continue;
        // the kernels on blocks of 64 rows all split the keys, and those work out the tiles of a band (rf_band.h): without these
        // lists the plans of 119056 tokens, 256 of text, are 14.3 MB in 9 ms, with them 26.7 in 17-22
        build_plan(g, tables, kBlocks[i], wide, &plans[i], kBlocks[i] != 64);
        for (int c = 0; c < kLists; ++c) {
            off[i].row_ptr[c] = bb.add(plans[i].row_ptr[c]);
            off[i].cols[c] = bb.add(plans[i].cols[c]);
            off[i].qorder[c] = bb.add(plans[i].qorder[c]);
            off[i].first_entry[c] = bb.add(plans[i].first_entry[c]);
        }
    }
    const int st = bb.upload(&p->blob);
    if (st != RF_OK) return st;
    const int32_t* base = static_cast<const int32_t*>(p->blob);
    for (int i = 0; i < kBlockSizes; ++i) {
        if (!wanted(i)) continue;
        const HostPlan& hp = plans[i];
        DevicePlan& d = p->dev[i];
        for (int c = 0; c < kLists; ++c) {
            d.row_ptr[c] = base + off[i].row_ptr[c];
            d.cols[c] = base + off[i].cols[c];
            d.attr[c] = base + off_attr[c];
            d.qorder[c] = base + off[i].qorder[c];
            d.first_entry[c] = base + off[i].first_entry[c];
        }
        d.cidx = base + off_cidx;
        d.pm_token = base + off_pm;
        d.radius[RF_SPATIAL] = g.r_spatial;
        d.radius[RF_TEMPORAL] = g.r_temporal;
        d.radius[RF_TEXTURAL] = 0;
        d.radius[kListTemporalPM] = g.r_temporal;
        d.group_rows[RF_SPATIAL] = g.HW;
        d.group_rows[kListTemporalPM] = g.T;
        d.video_shift = g.video_shift();
        d.text_shift = g.text_shift();
        d.N = g.N; d.Nv = g.Nv; d.Nc = hp.Nc;
        d.block = hp.block; d.nQB = hp.nQB; d.nKT = hp.nKT; d.nCT = hp.nCT;
        d.first_text_qb = hp.first_text_qb;
    }
    return RF_OK;
}

// out receives a COPY of the plan: the cache entry may be evicted by a later call (its device memory
// is only freed after the device has drained, so kernels already launched keep reading valid lists).
int get_attention_plan(const Geometry& geometry, int block, bool wide, DevicePlan* out) {
    int device = 0;
    if (hipGetDevice(&device) != hipSuccess) return RF_ERR_HIP;
    const Geometry g = list_key(geometry);
    std::lock_guard<std::mutex> lock(g_mu);
    CachedPlan* cp = find_plan(g, wide, device);
    if (!cp) {
        if (g_plans.size() >= kMaxCachedPlans) {
            size_t oldest = 0;
            for (size_t i = 1; i < g_plans.size(); ++i)
                if (g_plans[i]->last_use < g_plans[oldest]->last_use) oldest = i;
            if (hipDeviceSynchronize() != hipSuccess) return RF_ERR_HIP;
            if (g_plans[oldest]->blob && hipFree(g_plans[oldest]->blob) != hipSuccess) return RF_ERR_HIP;
            g_plans.erase(g_plans.begin() + static_cast<std::ptrdiff_t>(oldest));
        }
        auto p = std::make_unique<CachedPlan>();
        p->g = g;
        p->wide = wide;
        p->device = device;
        int st = RF_ERR_HIP;
        try {
            st = build_and_upload(g, wide, p.get());
        } catch (const std::bad_alloc&) {  // host memory for the lists, before any device memory is taken
        }
        if (st != RF_OK) return st;
        cp = p.get();
        g_plans.push_back(std::move(p));
    }
    cp->last_use = ++g_use_counter;
    *out = cp->dev[std::find(kBlocks, kBlocks + kBlockSizes, block) - kBlocks];
    return RF_OK;
}

int global_sample_count(const Geometry& g) { return (g.Nv + g.omega - 1) / g.omega; }

bool valid_block(int block) { return std::find(kBlocks, kBlocks + kBlockSizes, block) != kBlocks + kBlockSizes; }  // query rows per block

// (token counts that overflow int32 indices were already refused by resolve_geometry)
int check_shape(int B, int nH, int D) {
    if (B < 1 || nH < 1) return RF_ERR_SHAPE;
    if (D != 64 && D != 96 && D != 128) return RF_ERR_SHAPE;
    if (static_cast<int64_t>(B) * nH > (1 << 20)) return RF_ERR_SHAPE;
    return RF_OK;
}

// The kernels read and write the tensors 16 bytes at a time.
bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

size_t arm_rows(const Geometry& g) { return static_cast<size_t>(std::max(g.HW, global_sample_count(g))); }

}  // namespace
}  // namespace rf

using namespace rf;

extern "C" {

int rf_version(void) { return 100; }

const char* rf_status_string(int status) {
    switch (status) {
        case RF_OK: return "ok";
        case RF_ERR_NULL: return "null pointer";
        case RF_ERR_SHAPE: return "bad tensor shape";
        case RF_ERR_LAYOUT: return "bad video layout";
        case RF_ERR_PARAM: return "bad parameter";
        case RF_ERR_BLOCK: return "block must be 64, 128, 256 or 384";
        case RF_ERR_WORKSPACE: return "workspace missing or too small";
        case RF_ERR_HIP: return "HIP runtime error";
        case RF_ERR_ALIGN: return "tensor or workspace pointer misaligned";
        default: return "unknown status";
    }
}

size_t rf_arm_workspace_bytes(int B, int nH, const rf_layout* layout, const rf_params* params) {
    Geometry g;
    if (resolve_geometry(layout, params, &g) != RF_OK || B < 1 || nH < 1) return 0;
    return static_cast<size_t>(B) * nH * 2 * arm_rows(g) * sizeof(float);
}

// Geometry of `params` with both band widths replaced by bw.
static int geometry_with_bandwidth(const rf_layout* layout, const rf_params* params, float bw, Geometry* g) {
    rf_params p = params ? *params : rf_params{0.25f, 0.25f, 2, 0, 0};
    p.bw_spatial = bw;
    p.bw_temporal = bw;
    return resolve_geometry(layout, &p, g);
}

static int check_bandwidths(const float* bandwidths, int n_bw) {
    if (!bandwidths) return RF_ERR_NULL;
    if (n_bw < 1 || n_bw > RF_MAX_BANDWIDTHS) return RF_ERR_PARAM;
    for (int k = 0; k < n_bw; ++k)
        if (!(bandwidths[k] >= 0.f && bandwidths[k] <= 1.f)) return RF_ERR_PARAM;
    return RF_OK;
}

// Shared by rf_arm_classify (bandwidths == null: the widths of params) and rf_arm_classify_plus.
static int arm_classify_impl(const void* Q, const void* K, int B, int nH, int D, const rf_layout* layout,
                             const rf_params* params, int sample_mode, float threshold, const float* bandwidths,
                             int n_bw, int32_t* head_class, int32_t* head_bw, float* recalls, void* workspace,
                             size_t workspace_bytes, void* stream) {
    if (!Q || !K || !head_class || !layout) return RF_ERR_NULL;
    Geometry g;
    int st = resolve_geometry(layout, params, &g);
    if (st != RF_OK) return st;
    st = check_shape(B, nH, D);
    if (st != RF_OK) return st;
    if (!aligned16(Q) || !aligned16(K)) return RF_ERR_ALIGN;
    if (sample_mode != RF_SAMPLE_FIRST_FRAME && sample_mode != RF_SAMPLE_EQUAL_INTERVAL) return RF_ERR_PARAM;
    if (!(threshold >= 0.f && threshold <= 1.f)) return RF_ERR_PARAM;
    if (bandwidths) {
        st = check_bandwidths(bandwidths, n_bw);
        if (st != RF_OK) return st;
    }
    if (!workspace || workspace_bytes < n_bw * rf_arm_workspace_bytes(B, nH, layout, params)) return RF_ERR_WORKSPACE;

    int r_temporal[kMaxBw] = {g.r_temporal}, r_spatial[kMaxBw] = {g.r_spatial};
    ArmArgs a{};
    a.n_bw = n_bw;
    for (int k = 0; k < n_bw; ++k) a.by_width[k] = k;
    if (bandwidths) {
        for (int k = 0; k < n_bw; ++k) {
            Geometry gk;
            st = geometry_with_bandwidth(layout, params, bandwidths[k], &gk);
            if (st != RF_OK) return st;
            r_temporal[k] = gk.r_temporal;
            r_spatial[k] = gk.r_spatial;
        }
        std::stable_sort(a.by_width, a.by_width + n_bw, [&](int x, int y) { return bandwidths[x] < bandwidths[y]; });
    }

    a.Q = static_cast<const uint16_t*>(Q);
    a.K = static_cast<const uint16_t*>(K);
    a.BH = B * nH;
    a.N = g.N;
    a.first_video_row = g.video_shift();
    a.scale_log2 = static_cast<float>(1.4426950408889634 / std::sqrt(static_cast<double>(D)));
    const int nG = global_sample_count(g);
    if (sample_mode == RF_SAMPLE_FIRST_FRAME) a.pass[0] = ArmPass{0, g.HW, 1, g.HW, {0}};
    else a.pass[0] = ArmPass{0, nG, g.omega, g.HW, {0}};
    a.pass[1] = ArmPass{1, nG, g.omega, g.HW, {0}};
    for (int k = 0; k < n_bw; ++k) {
        a.pass[0].radius[k] = r_temporal[k];
        a.pass[1].radius[k] = r_spatial[k];
    }
    a.row_recall = static_cast<float*>(workspace);
    a.max_n = static_cast<int>(arm_rows(g));
    a.threshold = threshold;
    a.fallback_class = g.two_head ? RF_DENSE : RF_TEXTURAL;
    a.head_class = head_class;
    a.head_bw = head_bw;
    a.recalls = recalls;
    return launch_arm(a, D, stream) == 0 ? RF_OK : RF_ERR_HIP;
}

int rf_arm_classify(const void* Q, const void* K, int B, int nH, int D, const rf_layout* layout,
                    const rf_params* params, int sample_mode, float threshold, int32_t* head_class,
                    float* recalls, void* workspace, size_t workspace_bytes, void* stream) {
    return arm_classify_impl(Q, K, B, nH, D, layout, params, sample_mode, threshold, nullptr, 1, head_class, nullptr,
                             recalls, workspace, workspace_bytes, stream);
}

int rf_arm_classify_noalloc(const void* Q, const void* K, int B, int nH, int D, const rf_layout* layout,
                            const rf_params* params, int sample_mode, float threshold, int32_t* head_class,
                            float* recalls, void* stream) {
    // every argument check, and the size limit, before any HIP call
    if (!Q || !K || !head_class || !layout) return RF_ERR_NULL;
    Geometry g;
    int st = resolve_geometry(layout, params, &g);
    if (st != RF_OK) return st;
    st = check_shape(B, nH, D);
    if (st != RF_OK) return st;
    if (!aligned16(Q) || !aligned16(K)) return RF_ERR_ALIGN;
    if (sample_mode != RF_SAMPLE_FIRST_FRAME && sample_mode != RF_SAMPLE_EQUAL_INTERVAL) return RF_ERR_PARAM;
    if (!(threshold >= 0.f && threshold <= 1.f)) return RF_ERR_PARAM;
    if (rf_arm_workspace_bytes(B, nH, layout, params) > kArmStaticScratchBytes) return RF_ERR_WORKSPACE;
    void* scratch = nullptr;
    size_t scratch_bytes = 0;
    if (arm_static_scratch(&scratch, &scratch_bytes) != 0) return RF_ERR_HIP;
    return arm_classify_impl(Q, K, B, nH, D, layout, params, sample_mode, threshold, nullptr, 1, head_class, nullptr,
                             recalls, scratch, scratch_bytes, stream);
}

int rf_arm_classify_plus(const void* Q, const void* K, int B, int nH, int D, const rf_layout* layout,
                         const rf_params* params, int sample_mode, float threshold, const float* bandwidths,
                         int n_bw, int32_t* head_class, int32_t* head_bw, float* recalls, void* workspace,
                         size_t workspace_bytes, void* stream) {
    if (!head_bw) return RF_ERR_NULL;
    const int st = check_bandwidths(bandwidths, n_bw);
    if (st != RF_OK) return st;
    return arm_classify_impl(Q, K, B, nH, D, layout, params, sample_mode, threshold, bandwidths, n_bw, head_class,
                             head_bw, recalls, workspace, workspace_bytes, stream);
}

size_t rf_attention_workspace_bytes(int B, int nH, int D, const rf_layout* layout, const rf_params* params) {
    Geometry g;
    if (resolve_geometry(layout, params, &g) != RF_OK || check_shape(B, nH, D) != RF_OK) return 0;
    return RF_ATTENTION_MIN_WORKSPACE + 2 * static_cast<size_t>(B) * nH * g.N * D * sizeof(uint16_t);
}

static AttnForm form_of_call(const Geometry& g, int BH, int D, const rf_params* params, int block, bool room) {
    const int flags = params ? params->flags : 0;
    if (flags & RF_FLAG_WIDE_ROWS) return AttnForm{block, 1, true, true};
    if (flags & RF_FLAG_FIXED_ORDER) return choose_fixed_form(g, D);
    return choose_form(g, BH, D, (flags & RF_FLAG_FORCE_DENSE) != 0, room);
}

static int sparse_attention_impl(const void* Q, const void* K, const void* V, const int32_t* head_class,
                                 const int32_t* head_bw, const float* bandwidths, int n_bw, int B, int nH, int D,
                                 const rf_layout* layout, const rf_params* params, int block, void* O, void* workspace,
                                 size_t workspace_bytes, void* stream, const AttnForm* named = nullptr) {
    if (!Q || !K || !V || !O || !layout) return RF_ERR_NULL;
    const bool force_dense = params && (params->flags & RF_FLAG_FORCE_DENSE);
    if (!head_class && !force_dense) return RF_ERR_NULL;
    Geometry g;
    int st = resolve_geometry(layout, params, &g);
    if (st != RF_OK) return st;
    st = check_shape(B, nH, D);
    if (st != RF_OK) return st;
    if (!valid_block(block)) return RF_ERR_BLOCK;
    if (params && (params->flags & RF_FLAG_WIDE_ROWS) && (block != 256 || D != 128)) return RF_ERR_PARAM;
    if (!aligned16(Q) || !aligned16(K) || !aligned16(V) || !aligned16(O)) return RF_ERR_ALIGN;
    // the work-queue counters live in the first RF_ATTENTION_MIN_WORKSPACE bytes; a workspace of the
    // full size also has room for the packed copies of K and V
    if (!workspace || workspace_bytes < RF_ATTENTION_MIN_WORKSPACE) return RF_ERR_WORKSPACE;
    if (reinterpret_cast<uintptr_t>(workspace) & 255) return RF_ERR_ALIGN;
    const bool room_to_pack = workspace_bytes >= rf_attention_workspace_bytes(B, nH, D, layout, params);

    AttnArgs a{};
    a.wide_rows = (params && (params->flags & RF_FLAG_WIDE_ROWS)) ? 1 : 0;
    const AttnForm form = named ? *named : form_of_call(g, B * nH, D, params, block, room_to_pack);
    // a kernel that walks copies cannot gather: without them it would look for a Temporal list that is not built
    if (form.copies && !a.wide_rows && !room_to_pack && !force_dense) return RF_ERR_WORKSPACE;
    if (named && named->rows < 256 && g.N > kSmallBlockTokens) return RF_ERR_PARAM;  // no such lists
    a.queued = form.queued ? 1 : 0;
    a.key_groups = form.key_groups;
    a.three_to_a_cu = form.key_groups == 2 && D == 96 ? 1 : 0;
    a.n_plans = bandwidths ? n_bw : 1;
    for (int k = 0; k < a.n_plans; ++k) {
        Geometry gk = g;
        if (bandwidths) {
            st = geometry_with_bandwidth(layout, params, bandwidths[k], &gk);
            if (st != RF_OK) return st;
        }
        if (a.three_to_a_cu && !three_to_a_cu(gk, B * nH, force_dense)) a.three_to_a_cu = 0;  // by the narrowest bandwidth
        st = get_attention_plan(gk, form.rows, a.wide_rows != 0, &a.plan[k]);
        if (st != RF_OK) return st;
    }
    a.Q = static_cast<const uint16_t*>(Q);
    a.K = static_cast<const uint16_t*>(K);
    a.V = static_cast<const uint16_t*>(V);
    a.O = static_cast<uint16_t*>(O);
    a.queue = static_cast<int*>(workspace);
    a.join_sweep = (params && (params->flags & RF_FLAG_FIXED_ORDER)) ? 0 : 1;
    a.BH = B * nH;
    a.item_order = item_order(!whole_heads_fit(g, D), form.queued, force_dense, a.BH, static_cast<long long>(a.plan[0].nQB) * a.BH);
    a.head_class = force_dense ? nullptr : head_class;
    a.head_bw = bandwidths ? head_bw : nullptr;
    a.scale_log2 = static_cast<float>(1.4426950408889634 / std::sqrt(static_cast<double>(D)));
    if (room_to_pack && !force_dense && form.copies) {
        a.packed_k = reinterpret_cast<uint16_t*>(static_cast<unsigned char*>(workspace) + RF_ATTENTION_MIN_WORKSPACE);
        a.packed_v = a.packed_k + static_cast<size_t>(B) * nH * g.N * D;
        if (launch_pack_textural(a, D, stream) != 0) return RF_ERR_HIP;
    }
    return launch_attention(a, D, stream) == 0 ? RF_OK : RF_ERR_HIP;
}

int rf_sparse_attention(const void* Q, const void* K, const void* V, const int32_t* head_class, int B, int nH,
                        int D, const rf_layout* layout, const rf_params* params, int block, void* O,
                        void* workspace, size_t workspace_bytes, void* stream) {
    return sparse_attention_impl(Q, K, V, head_class, nullptr, nullptr, 1, B, nH, D, layout, params, block, O,
                                 workspace, workspace_bytes, stream);
}

int rf_sparse_attention_plus(const void* Q, const void* K, const void* V, const int32_t* head_class,
                             const int32_t* head_bw, const float* bandwidths, int n_bw, int B, int nH, int D,
                             const rf_layout* layout, const rf_params* params, int block, void* O, void* workspace,
                             size_t workspace_bytes, void* stream) {
    if (!head_bw) return RF_ERR_NULL;
    const int st = check_bandwidths(bandwidths, n_bw);
    if (st != RF_OK) return st;
    return sparse_attention_impl(Q, K, V, head_class, head_bw, bandwidths, n_bw, B, nH, D, layout, params, block, O,
                                 workspace, workspace_bytes, stream);
}

int rf_internal_attention_as(int rows, int key_groups, int queued, const void* Q, const void* K, const void* V,
                             const int32_t* head_class, const int32_t* head_bw, const float* bandwidths, int n_bw, int B,
                             int nH, int D, const rf_layout* layout, const rf_params* params, void* O, void* workspace,
                             size_t workspace_bytes, void* stream) {
    AttnForm form;
    if ((D != 64 && D != 96 && D != 128) || !find_form(D, rows, key_groups, queued != 0, &form)) return RF_ERR_PARAM;
    if (params && (params->flags & RF_FLAG_WIDE_ROWS)) return RF_ERR_PARAM;
    if (bandwidths) {
        if (!head_bw) return RF_ERR_NULL;
        const int st = check_bandwidths(bandwidths, n_bw);
        if (st != RF_OK) return st;
    }
    return sparse_attention_impl(Q, K, V, head_class, head_bw, bandwidths, n_bw, B, nH, D, layout, params, rows, O, workspace,
                                 workspace_bytes, stream, &form);
}

int rf_internal_attention_form(int B, int nH, int D, const rf_layout* layout, const rf_params* params, int block,
                               size_t workspace_bytes, int32_t* form) {
    Geometry g;
    int st = resolve_geometry(layout, params, &g);
    if (st != RF_OK || (st = check_shape(B, nH, D)) != RF_OK) return st;
    const bool room = workspace_bytes >= rf_attention_workspace_bytes(B, nH, D, layout, params);
    const AttnForm f = form_of_call(g, B * nH, D, params, block, room);
    form[0] = f.rows;
    form[1] = f.key_groups;
    form[2] = f.queued;
    form[3] = f.copies && room && !(params && (params->flags & RF_FLAG_FORCE_DENSE));
    return RF_OK;
}

int rf_plan_host(const rf_layout* layout, const rf_params* params, int block, int cls, int32_t* row_ptr,
                 int32_t* cols, size_t cap, size_t* needed) {
    if (!layout || !needed) return RF_ERR_NULL;
    Geometry g;
    const int st = resolve_geometry(layout, params, &g);
    if (st != RF_OK) return st;
    if (!valid_block(block)) return RF_ERR_BLOCK;
    if (cls < RF_SPATIAL || cls > RF_LIST_TEMPORAL_POSITION_MAJOR) return RF_ERR_PARAM;
    HostPlan hp;
    build_plan(g, block, &hp);
    std::vector<int32_t> rp, co;
    flatten_class(hp, cls, &rp, &co);
    *needed = co.size();
    if (row_ptr) std::memcpy(row_ptr, rp.data(), rp.size() * sizeof(int32_t));
    if (cols) {
        if (cap < co.size()) return RF_ERR_WORKSPACE;
        std::memcpy(cols, co.data(), co.size() * sizeof(int32_t));
    }
    return RF_OK;
}

int rf_plan_order(const rf_layout* layout, const rf_params* params, int block, int cls, int32_t* order,
                  int32_t* first_entry) {
    if (!layout || !order) return RF_ERR_NULL;
    Geometry g;
    const int st = resolve_geometry(layout, params, &g);
    if (st != RF_OK) return st;
    if (!valid_block(block)) return RF_ERR_BLOCK;
    if (cls < RF_SPATIAL || cls > RF_LIST_TEMPORAL_POSITION_MAJOR) return RF_ERR_PARAM;
    HostPlan hp;
    build_plan(g, block, &hp);
    const int list = cls == RF_LIST_TEMPORAL_POSITION_MAJOR ? kListTemporalPM : cls;
    // dense heads: the same scheme with plain token order for the blocks without text rows
    for (int i = 0; i < hp.nQB; ++i) order[i] = hp.qorder[cls == RF_DENSE ? RF_SPATIAL : list][i];
    if (first_entry)
        for (int i = 0; i < hp.nQB; ++i) first_entry[i] = cls == RF_DENSE ? 0 : hp.first_entry[list][i];
    return RF_OK;
}

int rf_plan_position_major(const rf_layout* layout, const rf_params* params, int32_t* token_of) {
    if (!layout || !token_of) return RF_ERR_NULL;
    Geometry g;
    const int st = resolve_geometry(layout, params, &g);
    if (st != RF_OK) return st;
    for (int n = 0; n < g.Nv; ++n) token_of[n] = g.row_of((n % g.T) * g.HW + n / g.T);
    for (int n = g.Nv; n < g.N; ++n) token_of[n] = g.row_of(n);
    return RF_OK;
}

int rf_plan_clear(void) {
    std::lock_guard<std::mutex> lock(g_mu);
    if (g_plans.empty()) return RF_OK;
    int st = RF_OK;
    if (hipDeviceSynchronize() != hipSuccess) st = RF_ERR_HIP;
    for (auto& p : g_plans)
        if (p->blob && hipFree(p->blob) != hipSuccess) st = RF_ERR_HIP;
    g_plans.clear();
    return st;
}

}  // extern "C"
