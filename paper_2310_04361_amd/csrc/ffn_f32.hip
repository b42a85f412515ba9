// fp32 expert execution and merge (Sec. 3.2, Appendix G): token-major, straight from the mask.
// One workgroup per token; a token's selected experts are merged in ascending order by one chain of
// fused multiply-adds per output column, so the result is deterministic.  Meant for the small fp32
// exactness configuration.
//
// What bounds it there is latency: with one expert after the other, two barriers and two memory round
// trips each, the 64-wide layer of 16 experts of 16 took 42 us at 128 tokens.  Now the hidden values
// of all the selected experts (as many as LDS holds at a time) are computed side by side, four rows per
// wavefront in flight, and the merge requests its next sixteen weights while it uses the last sixteen:
// 20 us, with the same bits.
#include "dmoe_internal.h"
#include "mfma.h"

namespace dmoe {

namespace {

constexpr int kF32Threads = 512, kF32Waves = kF32Threads / 64;

// batch: experts whose hidden values hs holds at a time
__global__ __launch_bounds__(kF32Threads) void ffn_f32_kernel(
    const float* __restrict__ x, const float* __restrict__ w_up, const float* __restrict__ w_gate,
    const float* __restrict__ b_up, const float* __restrict__ w_down,
    const float* __restrict__ b_down, const uint64_t* __restrict__ mask, float* __restrict__ y,
    int d, int E, int m, int W, int act, int batch) {
    extern __shared__ float smem[];
    float* xs = smem;          // [d]
    float* ys = smem + d;      // [d]
    float* hs = smem + 2 * d;  // [batch][m]
    int* list = reinterpret_cast<int*>(hs + (size_t)batch * m);  // [batch] the selected ones, ascending
    int* row_id = list + batch;                                  // [batch][m] their rows of w_up / w_down
    __shared__ int s_n;
    const int t = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int k = threadIdx.x; k < d; k += kF32Threads) {
        xs[k] = x[(size_t)t * d + k];
        ys[k] = b_down ? b_down[k] : 0.0f;
    }
    for (int e0 = 0; e0 < E; e0 += batch) {
        const int e1 = min(E, e0 + batch);
        if (wave == 0) {
            int n = 0;
            for (int eb = e0; eb < e1; eb += 64) {
                const int e = eb + lane;
                const bool keep = e < e1 && ((mask[(size_t)t * W + (e >> 6)] >> (e & 63)) & 1ull);
                const uint64_t bal = __ballot(keep);
                if (keep) list[n + __popcll(bal & ((1ull << lane) - 1ull))] = e;
                n += __popcll(bal);
            }
            if (lane == 0) s_n = n;
        }
        __syncthreads();
        const int rows = s_n * m;
        for (int r = threadIdx.x; r < rows; r += kF32Threads) row_id[r] = list[r / m] * m + r % m;
        __syncthreads();
        for (int r0 = 4 * wave; r0 < rows; r0 += 4 * kF32Waves) {
            float a[4] = {0.f, 0.f, 0.f, 0.f}, g[4] = {0.f, 0.f, 0.f, 0.f};
            size_t row[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) row[u] = (size_t)row_id[min(r0 + u, rows - 1)] * d;
            for (int k = lane; k < d; k += 64) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    a[u] = fmaf(w_up[row[u] + k], xs[k], a[u]);
                    if (w_gate) g[u] = fmaf(w_gate[row[u] + k], xs[k], g[u]);
                }
            }
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    a[u] += __shfl_xor(a[u], off, 64);
                    g[u] += __shfl_xor(g[u], off, 64);
                }
            }
            const int r = r0 + lane;
            if (lane < 4 && r < rows) {  // lane u finishes row u
                const float up = lane == 0 ? a[0] : lane == 1 ? a[1] : lane == 2 ? a[2] : a[3];
                const float gate = lane == 0 ? g[0] : lane == 1 ? g[1] : lane == 2 ? g[2] : g[3];
                if (w_gate) hs[r] = activate(act, gate) * up;
                else hs[r] = activate(act, up + (b_up ? b_up[row_id[r]] : 0.0f));
            }
        }
        __syncthreads();
        for (int c = threadIdx.x; c < d; c += kF32Threads) {
            float acc = ys[c];
            float v[2][16];
            // hidden rows r0 .. r0 + 15 (past the end: the last one again)
            auto load = [&](int r0, float (&o)[16]) {
#pragma unroll
                for (int u = 0; u < 16; ++u) o[u] = w_down[(size_t)row_id[min(r0 + u, rows - 1)] * d + c];
            };
            auto use = [&](int r0, const float (&o)[16]) {
#pragma unroll
                for (int u = 0; u < 16; ++u)
                    if (r0 + u < rows) acc = fmaf(hs[r0 + u], o[u], acc);
            };
            if (rows > 0) load(0, v[0]);
            for (int r0 = 0; r0 < rows; r0 += 32) {
                load(r0 + 16, v[1]);
                use(r0, v[0]);
                load(r0 + 32, v[0]);
                use(r0 + 16, v[1]);
            }
            ys[c] = acc;
        }
        __syncthreads();
    }
    for (int c = threadIdx.x; c < d; c += kF32Threads) y[(size_t)t * d + c] = ys[c];
}

}  // namespace

void launch_ffn_f32(const dmoe_layer& L, const float* x, int T, const uint64_t* mask, float* y,
                    hipStream_t s) {
    LaunchTimer tm(kSlotFfnF32, s);
    const int W = div_up(L.n_experts, 64), m = L.expert_size;
    // up to 2048 hidden values at a time, fewer where x and y leave less of 64 KB (one expert at least:
    // x, y and one expert's values take up to 64 KB, its row numbers come on top)
    const int room = std::min(4096, 16000 - 2 * L.d_model);
    const int batch = std::max(1, std::min(L.n_experts, room / (2 * m + 1)));
    const size_t lds = sizeof(float) * (2 * (size_t)L.d_model + (size_t)batch * (2 * m + 1));
    static std::once_flag attr_once;  // kernel attributes: once per process, thread-safe
    std::call_once(attr_once, [] {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&ffn_f32_kernel),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, 152 * 1024);
    });
    launch_kernel(ffn_f32_kernel, T, kF32Threads, lds, s, x, (const float*)L.w_up,
                                       L.gated ? (const float*)L.w_gate : nullptr,
                                       (const float*)L.b_up, (const float*)L.w_down,
                                       (const float*)L.b_down, mask, y, L.d_model, L.n_experts,
                                       m, W, L.act, batch);
}

}  // namespace dmoe
