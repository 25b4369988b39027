// The library's host side (rf_api.cpp, rf_plan.cpp) without a GPU: the HIP calls it makes are replaced by ones on host
// memory that are counted, and the launches by ones that record their arguments.  For every line
//   T H W text  bandwidth stride flags  block B nH D full_workspace
// on standard input one call of rf_sparse_attention; prints
//   status  allocations so far  rows key_groups queued item_order copies  hash of the lists the launch walks
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "rf_internal.h"

static int g_allocations = 0;
static rf::AttnArgs g_args;

extern "C" {
hipError_t hipGetDevice(int* device) { *device = 0; return hipSuccess; }
hipError_t hipMalloc(void** p, size_t bytes) { ++g_allocations; *p = std::malloc(bytes); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipMemcpy(void* to, const void* from, size_t bytes, hipMemcpyKind) { std::memcpy(to, from, bytes); return hipSuccess; }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
}

namespace rf {
int launch_attention(const AttnArgs& a, int, void*) { g_args = a; return 0; }
int launch_pack_textural(const AttnArgs&, int, void*) { return 0; }
int launch_arm(const ArmArgs&, int, void*) { return 0; }
int arm_static_scratch(void**, size_t*) { return 1; }
}  // namespace rf

// a walk reads all of these; a list that is not there would be null
static unsigned long long lists_hash(const rf::DevicePlan& p) {
    unsigned long long h = 1469598103934665603ull;
    auto add = [&](const int32_t* v, long long n) { for (long long i = 0; i < n; ++i) h = (h ^ static_cast<unsigned>(v[i])) * 1099511628211ull; };
    for (int l = 0; l < rf::kLists; ++l) {
        add(p.row_ptr[l], p.nQB + 1);
        add(p.cols[l], p.row_ptr[l][p.nQB]);
        add(p.attr[l], p.N);
        add(p.qorder[l], p.nQB);
        add(p.first_entry[l], p.nQB);
    }
    add(p.cidx, p.Nc);
    add(p.pm_token, p.N);
    return h;
}

int main() {
    alignas(256) static char tensor[256], workspace[256];  // never read: nothing is launched
    static int32_t classes[1];
    int T, H, W, text, stride, flags, block, B, nH, D, full;
    float bw;
    while (std::scanf("%d %d %d %d %f %d %d %d %d %d %d %d", &T, &H, &W, &text, &bw, &stride, &flags, &block, &B, &nH, &D, &full) == 12) {
        const rf_layout layout = {T, H, W, text};
        const rf_params params = {bw, bw, stride, 0, flags};
        const size_t bytes = full ? rf_attention_workspace_bytes(B, nH, D, &layout, &params) : RF_ATTENTION_MIN_WORKSPACE;
        const int st = rf_sparse_attention(tensor, tensor, tensor, classes, B, nH, D, &layout, &params, block, tensor, workspace, bytes, nullptr);
        std::printf("%d %d", st, g_allocations);
        if (st == RF_OK)
            std::printf(" %d %d %d %d %d %llx", g_args.plan[0].block, g_args.key_groups, g_args.queued, g_args.item_order,
                        g_args.packed_k != nullptr, lists_hash(g_args.plan[0]));
        std::printf("\n");
    }
    rf_plan_clear();
    return 0;
}
