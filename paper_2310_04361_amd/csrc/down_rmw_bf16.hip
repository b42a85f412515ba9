// The pair-proportional down-projection (down_rmw.h) as a kernel of its own: for sizes whose H or packed
// weights are beyond the 32-bit buffer offsets of the kernels that sum inside the matrix cores.
#include "down_rmw.h"

namespace dmoe {

namespace {

template <int KS, int RN>
__global__ __launch_bounds__(kDownWaves * 64) void down_rmw_bf16_kernel(
    const __bf16* __restrict__ w2f, const __bf16* __restrict__ b_down, const int32_t* __restrict__ item_start,
    const int32_t* __restrict__ group_off, const int32_t* __restrict__ alist, const __bf16* __restrict__ Hf,
    __bf16* __restrict__ y, int T, int d, int E, int NG, int rows_per_item) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    // The slices of one chunk share its H rows and token lists: keep them on one XCD (workgroups
    // are dealt round-robin to the 8 XCDs) and next to each other in launch order.
    const int NS = d / kDownCols;
    const int k_in_xcd = blockIdx.x >> 3;
    const int chunk = (k_in_xcd / NS) * 8 + (blockIdx.x & 7), slice = k_in_xcd % NS;
    if (chunk * kChunk >= T) return;  // the grid is rounded up to whole groups of 8 chunks
#include "down_rmw_walk.inc"
}

template <int KS, int RN>
void launch_down_rmw_t(const dmoe_layer& L, const PackedLayout& P, int T, const int32_t* item_start,
                       const int32_t* group_off, const int32_t* alist, const void* H, void* y, hipStream_t s) {
    const int NG = div_up(T, kGroup), NC = div_up(T, kChunk), NS = L.d_model / kDownCols;
    static std::once_flag attr_once;  // kernel attributes: once per process, thread-safe
    std::call_once(attr_once, [&] {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&down_rmw_bf16_kernel<KS, RN>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)kDownLds);
    });
    const char* pk = static_cast<const char*>(L.packed);
    launch_kernel(down_rmw_bf16_kernel<KS, RN>, round_up(NC, 8) * NS, kDownWaves * 64, kDownLds, s, 
        (const __bf16*)(pk + P.w2f), (const __bf16*)L.b_down, item_start, group_off, alist,
        (const __bf16*)H, (__bf16*)y, T, L.d_model, L.n_experts, NG, up_rows_bf16(L));
}

}  // namespace

void launch_down_rmw_bf16(const dmoe_layer& L, int T, const int32_t* item_start,
                          const int32_t* group_off, const int32_t* alist, const void* H, void* y, hipStream_t s) {
    LaunchTimer tm(kSlotDownRmw, s);
    const PackedLayout P = packed_layout(L);
#define DMOE_RMW(KS_, RN_) launch_down_rmw_t<KS_, RN_>(L, P, T, item_start, group_off, alist, H, y, s)
    switch (h_row_neurons(L)) {
    case 8: DMOE_RMW(1, 8); break;
    case 16: DMOE_RMW(1, 16); break;
    case 32: DMOE_RMW(1, 32); break;
    case 64: DMOE_RMW(2, 64); break;
    default: DMOE_RMW(4, 128); break;
    }
#undef DMOE_RMW
}

}  // namespace dmoe
