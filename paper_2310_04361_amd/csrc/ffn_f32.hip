// fp32 layers (Sec. 3.2 - 3.4, Appendix G).  First the experts and merge of wide layers: token-major, straight
// from the mask; below, the whole layer in one launch.
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

// Sums over the wavefront of N values at a time (every lane gets them): the lanes 32, 16, 8, 4, 2 and 1
// apart added in turn, in registers.  After a step all lanes that far apart hold the same value, so the
// rotations by 8 and 4 within a row of 16 lanes bring the partner's.
template <int CTRL>
__device__ __forceinline__ float plus_dpp(float v) {
    return v + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int N>
__device__ __forceinline__ void wave_sums(float (&a)[N]) {
#pragma unroll
    for (int u = 0; u < N; ++u) {
        const auto h = __builtin_amdgcn_permlane32_swap(__float_as_int(a[u]), __float_as_int(a[u]), false, false);
        a[u] = __int_as_float(h[0]) + __int_as_float(h[1]);
    }
#pragma unroll
    for (int u = 0; u < N; ++u) {
        const auto h = __builtin_amdgcn_permlane16_swap(__float_as_int(a[u]), __float_as_int(a[u]), false, false);
        a[u] = __int_as_float(h[0]) + __int_as_float(h[1]);
    }
#pragma unroll
    for (int u = 0; u < N; ++u) a[u] = plus_dpp<0x128>(a[u]);  // row_ror:8
#pragma unroll
    for (int u = 0; u < N; ++u) a[u] = plus_dpp<0x124>(a[u]);  // row_ror:4
#pragma unroll
    for (int u = 0; u < N; ++u) a[u] = plus_dpp<0x4e>(a[u]);   // quad_perm [2,3,0,1]
#pragma unroll
    for (int u = 0; u < N; ++u) a[u] = plus_dpp<0xb1>(a[u]);   // quad_perm [1,0,3,2]
}

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

// ---- the whole layer in one launch (d <= kF32FusedMaxD, router_hidden and E as LDS holds them) ---------
// One workgroup per token.  What bounds such a layer is latency, so the token's router, gate and experts
// are one chain of memory round trips without a launch between them: x with the router's rows, then the
// rows of w_up, w_gate and w_down of the selected experts.  A wavefront owns whole rows of the expert
// matrices: x and its share of y live in its registers (column lane + 64 c), the hidden value of a row
// is a wavefront sum that every lane then has, and the row of w_down was requested together with the
// row of w_up -- so up- and down-projection need no barrier and no second round trip.  The wavefronts'
// shares of y meet in LDS, in wavefront order.  Scores and hidden values have the bits of
// router_f32_kernel and ffn_f32_kernel; y sums the rows of a wavefront first.
// 128 tokens of the 64-wide layer of 16 experts of 16: 28.7 us as three launches, 8.9 as one (16 wavefronts,
// 4 rows in flight each; 8 wavefronts 9.9; with sums through LDS instead of in registers 10.3).
// GATE: router and gate inside; otherwise the selection comes from mask.  DC = ceil(d / 64).
constexpr int kLayerThreads = 1024, kLayerWaves = kLayerThreads / 64;

template <int DC, bool GATE>
__global__ __launch_bounds__(kLayerThreads) void layer_f32_kernel(
    const float* __restrict__ x, const float* __restrict__ r_w1, const float* __restrict__ r_b1,
    const float* __restrict__ r_w2, const float* __restrict__ r_b2, const float* __restrict__ w_up,
    const float* __restrict__ w_gate, const float* __restrict__ b_up, const float* __restrict__ w_down,
    const float* __restrict__ b_down, uint64_t* __restrict__ mask, float* __restrict__ scores_out,
    float* __restrict__ y, int d, int dh, int E, int m, int W, int act, float tau) {
    constexpr int RU = DC <= 2 ? 4 : DC <= 4 ? 2 : 1;  // rows in flight per wavefront
    constexpr int RR = DC <= 4 ? 2 : 1;                // ... of the router's matrices
    extern __shared__ float smem[];
    float* shares = smem;                                     // [kLayerWaves][d]
    int* list = reinterpret_cast<int*>(smem + kLayerWaves * d); // [E] selected experts, ascending
    float* sc = smem + kLayerWaves * d + E;                     // [E] scores (GATE)
    float* hid = sc + E;                                      // [dh]       (GATE)
    __shared__ int s_n;
    const int t = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    float xv[DC];
#pragma unroll
    for (int c = 0; c < DC; ++c) xv[c] = lane + 64 * c < d ? x[(size_t)t * d + min(lane + 64 * c, d - 1)] : 0.0f;
    // element lane + 64 c of a row; columns beyond d meet xv = 0 (and are never stored)
    int col[DC];
#pragma unroll
    for (int c = 0; c < DC; ++c) col[c] = min(lane + 64 * c, d - 1);
    if (GATE) {
        float w2[RR];  // first 64 columns of this wavefront's first rows of the second product
#pragma unroll
        for (int u = 0; u < RR; ++u)
            w2[u] = r_w2[(size_t)min(wave + u * kLayerWaves, E - 1) * dh + min(lane, dh - 1)];
        for (int j0 = wave; j0 < dh; j0 += RR * kLayerWaves) {
            float w[RR][DC], a[RR];
#pragma unroll
            for (int u = 0; u < RR; ++u)
#pragma unroll
                for (int c = 0; c < DC; ++c) w[u][c] = r_w1[(size_t)min(j0 + u * kLayerWaves, dh - 1) * d + col[c]];
#pragma unroll
            for (int u = 0; u < RR; ++u) {
                a[u] = 0.0f;
#pragma unroll
                for (int c = 0; c < DC; ++c) a[u] = lane + 64 * c < d ? fmaf(w[u][c], xv[c], a[u]) : a[u];
            }
            wave_sums(a);
#pragma unroll
            for (int u = 0; u < RR; ++u) {
                const int j = j0 + u * kLayerWaves;
                if (lane == 0 && j < dh) hid[j] = fmaxf(a[u] + (r_b1 ? r_b1[j] : 0.0f), 0.0f);
            }
        }
        __syncthreads();
        for (int i0 = wave; i0 < E; i0 += RR * kLayerWaves) {
            float a[RR];
#pragma unroll
            for (int u = 0; u < RR; ++u) a[u] = 0.0f;
            for (int k = lane; k < dh; k += 64) {
                const float hv = hid[k];
#pragma unroll
                for (int u = 0; u < RR; ++u)
                    a[u] = fmaf(i0 == wave && k == lane ? w2[u] : r_w2[(size_t)min(i0 + u * kLayerWaves, E - 1) * dh + k], hv, a[u]);
            }
            wave_sums(a);
#pragma unroll
            for (int u = 0; u < RR; ++u) {
                const int i = i0 + u * kLayerWaves;
                if (lane == 0 && i < E) {
                    sc[i] = fabsf(a[u] + (r_b2 ? r_b2[i] : 0.0f));
                    if (scores_out) scores_out[(size_t)t * E + i] = sc[i];
                }
            }
        }
        __syncthreads();
    }
    if (wave == 0) {
        float mx = -INFINITY;
        if (GATE) {
            for (int e = lane; e < E; e += 64) mx = fmaxf(mx, sc[e]);
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
        }
        const double thr = (double)tau * (double)mx;  // exact: at most 48 significant bits
        int n = 0;
        for (int w = 0; w < W; ++w) {
            const int e = 64 * w + lane;
            const bool keep = GATE ? e < E && (tau == 0.0f || (double)sc[min(e, E - 1)] >= thr)
                                   : e < E && ((mask[(size_t)t * W + w] >> lane) & 1ull);
            const uint64_t bal = __ballot(keep);
            if (keep) list[n + __popcll(bal & ((1ull << lane) - 1ull))] = e;
            n += __popcll(bal);
            if (GATE && mask && lane == 0) mask[(size_t)t * W + w] = bal;
        }
        if (lane == 0) s_n = n;
    }
    __syncthreads();
    const int rows = s_n * m;
    float acc[DC];
#pragma unroll
    for (int c = 0; c < DC; ++c) acc[c] = 0.0f;
    for (int r0 = wave * RU; r0 < rows; r0 += RU * kLayerWaves) {
        int i = r0 / m, n = r0 - i * m;  // row r0 + u: neuron n of the i-th selected expert
        float wu[RU][DC], wg[RU][DC], wd[RU][DC], a[RU], g[RU], bu[RU];
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            const size_t id = (size_t)__builtin_amdgcn_readfirstlane(list[i]) * m + n, row = id * d;
            if (r0 + u + 1 < rows && ++n == m) n = 0, ++i;  // (past the end: the last row again)
            bu[u] = b_up ? b_up[id] : 0.0f;
#pragma unroll
            for (int c = 0; c < DC; ++c) {
                wu[u][c] = w_up[row + col[c]];
                if (w_gate) wg[u][c] = w_gate[row + col[c]];
                wd[u][c] = w_down[row + col[c]];
            }
        }
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            a[u] = g[u] = 0.0f;
#pragma unroll
            for (int c = 0; c < DC; ++c) {
                if (lane + 64 * c < d) {
                    a[u] = fmaf(wu[u][c], xv[c], a[u]);
                    if (w_gate) g[u] = fmaf(wg[u][c], xv[c], g[u]);
                }
            }
        }
        wave_sums(a);
        if (w_gate) wave_sums(g);
#pragma unroll
        for (int u = 0; u < RU; ++u) {
            const float h = w_gate ? activate(act, g[u]) * a[u] : activate(act, a[u] + bu[u]);
            if (r0 + u < rows) {
#pragma unroll
                for (int c = 0; c < DC; ++c) acc[c] = fmaf(h, wd[u][c], acc[c]);
            }
        }
    }
#pragma unroll
    for (int c = 0; c < DC; ++c)
        if (lane + 64 * c < d) shares[wave * d + lane + 64 * c] = acc[c];
    __syncthreads();
    for (int c = threadIdx.x; c < d; c += kLayerThreads) {
        float v = b_down ? b_down[c] : 0.0f;
#pragma unroll
        for (int w = 0; w < kLayerWaves; ++w) v += shares[w * d + c];
        y[(size_t)t * d + c] = v;
    }
}

// Where it is taken: rows of up to 1024 values (x, a share of y and a row of each matrix in registers), and
// the wavefronts' shares with the scores in the 64 KB of LDS that need no attribute, which ends it somewhat earlier:
// 16 d + 2 E + d_h <= 16384 with the gate inside, 16 d + E <= 16384 without.  Wider layers keep the kernels that hold
// x and y in LDS.  Three launches / one, us: d = 960, 16 experts of 16, 1 / 128 / 2048 tokens 45 / 64 / 157 and 12 / 20 /
// 115, 64 of 32 135 / 296 / 788 and 40 / 69 / 594; d = 512, 128 of 8 86 / 130 / 245 and 20 / 27 / 110; d = 768, 16 of 16, 2048
// tokens 135 and 120, the closest of 45.  Experts alone (top-k, given lists), 512 tokens: d = 960, 128 of 8, 4 of them per
// token 182 and 176, the closest of 45; 64 of 32, 30 % 319 and 200.
constexpr int kF32FusedMaxD = 1024;

size_t layer_f32_lds(const dmoe_layer& L, bool gate) {
    return sizeof(float) * ((size_t)kLayerWaves * L.d_model + L.n_experts + (gate ? L.n_experts + L.router_hidden : 0));
}

void launch_layer_f32_any(const dmoe_layer& L, const float* x, int T, bool gate, float tau, uint64_t* mask,
                          float* scores_out, float* y, hipStream_t s) {
    LaunchTimer tm(kSlotFfnF32, s);
    const size_t lds = layer_f32_lds(L, gate);
    // (a launch holds fewer than 2^32 threads: beyond, the runtime takes their number modulo 2^32)
    constexpr int kSlice = 1 << 21;  // tokens
    auto go = [&](auto kernel) {
        const int E = L.n_experts, W = div_up(E, 64);
        for (int t0 = 0; t0 < T; t0 += std::min(kSlice, T - t0)) {
            launch_kernel(kernel, std::min(kSlice, T - t0), kLayerThreads, lds, s, x + (size_t)t0 * L.d_model,
                          (const float*)L.r_w1, (const float*)L.r_b1, (const float*)L.r_w2, (const float*)L.r_b2,
                          (const float*)L.w_up, L.gated ? (const float*)L.w_gate : nullptr, (const float*)L.b_up,
                          (const float*)L.w_down, (const float*)L.b_down, mask ? mask + (size_t)t0 * W : nullptr,
                          scores_out ? scores_out + (size_t)t0 * E : nullptr, y + (size_t)t0 * L.d_model, L.d_model,
                          L.router_hidden, E, L.expert_size, W, L.act, tau);
        }
    };
    const int dc = div_up(L.d_model, 64);
#define DMOE_F32(DC_) (gate ? go(layer_f32_kernel<DC_, true>) : go(layer_f32_kernel<DC_, false>))
    if (dc <= 1) DMOE_F32(1);
    else if (dc <= 2) DMOE_F32(2);
    else if (dc <= 4) DMOE_F32(4);
    else if (dc <= 8) DMOE_F32(8);
    else DMOE_F32(16);
#undef DMOE_F32
}

}  // namespace

bool layer_f32_fused(const dmoe_layer& L) {
    return L.dtype == DMOE_F32 && L.d_model <= kF32FusedMaxD && layer_f32_lds(L, true) <= 64 * 1024;
}

void launch_layer_f32(const dmoe_layer& L, const float* x, int T, float tau, uint64_t* mask, float* scores_out,
                      float* y, hipStream_t s) {
    launch_layer_f32_any(L, x, T, true, tau, mask, scores_out, y, s);
}

void launch_ffn_f32(const dmoe_layer& L, const float* x, int T, const uint64_t* mask, float* y,
                    hipStream_t s) {
    if (L.d_model <= kF32FusedMaxD && layer_f32_lds(L, false) <= 64 * 1024) {
        launch_layer_f32_any(L, x, T, false, 0.0f, const_cast<uint64_t*>(mask), nullptr, y, s);
        return;
    }
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
