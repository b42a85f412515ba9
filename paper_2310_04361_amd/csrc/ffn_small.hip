// Small batches (decode): up to 64 tokens ride in one to four MFMA column tiles (TT tiles of 16), so
// the work is reading every touched expert's weights exactly once -- a weight-bandwidth-bound stream
// -- and what is not the stream is launches and latency.  A forward is two launches:
//
//   small_up    router, gate and up-projection.  The first workgroups compute the router's hidden rows
//               (one tile of 16 hidden units x 16 tokens each), one more per token tile collects
//               them for the second router product and the gate and announces the token sets.  The
//               other workgroups each own one or two neuron tiles of an expert: all wavefronts
//               split K, the slices are added up through LDS and h goes out as H fragments.  They
//               either wait for the announcement and drop the experts that nobody selected, or,
//               where most experts will be touched or the weights are small, do not wait at all
//               (see launch_up_t): the stream then runs while the router works.
//   small_down  workgroup = (16 to 64 output columns, group of experts), its wavefronts split the
//               touched experts and add up through LDS; with several expert groups the fp32 shares go
//               to memory, and the last workgroup of a column group to finish adds them up in order.
//               It masks the hidden rows with the token sets and reads only the touched experts, so what
//               was computed for nobody adds nothing.
//
// What workgroups of one launch exchange goes through agent-scope accesses, which pass by the per-XCD
// L2s (a release fence would write the whole L2 back: measured ten times slower).  The flags behind
// the hidden rows and the announced token sets (16 bits of payload, 48 of tag) carry the call's own
// number, so nothing in the workspace needs to start at zero; small_down clears them for the replay
// of a recorded graph, whose calls keep their number.  All waits are bounded: a gate that has not
// seen all hidden rows for a while computes them itself.  An up-projection workgroup that has not seen all
// announcements for much longer does not know which work items the others leave to it (they are numbered
// by the list of the touched experts), so it computes them all.
//
// Measured, whole call (five launches before, of which the prefill kernels took the sizes above 16
// tokens), weights in the last-level cache: three layers of 32 experts of 24, d = 768, 16 tokens 20.7 -> 13.6 us;
// 256 gated experts of 64, d = 2048: 1 token 28.9 -> 19.5, 16 tokens 57.3 -> 45.3, 48 tokens of e4m3
// weights 289 -> 43.3 us.  At 16 tokens, with weights from HBM, the two streams (134 MB of up and gate, 64 MB
// of down weights) run at about 5 and 4.4 TB/s; the rest is the router's chain of two products (16 us with the
// stream beside it) and the two launches.
#include <atomic>
#include <chrono>
#include <cmath>
#include <type_traits>

#include "dmoe_internal.h"
#include "mfma.h"
#include "small_gate.h"

namespace dmoe {

namespace {

// Polls of a workgroup that waits, each a round trip past the L2s of about half a microsecond: for the hidden
// rows some 0.1 ms (they take a few us), and for the announcements some 2 ms, several times what a gate
// takes that computes the hidden rows of 512 units itself.  give_up: see dmoe_small_give_up.
constexpr int kHiddenPolls = 200, kSetPolls = 4000;
__device__ __forceinline__ int wait_budget(int polls, int give_up) {
    return give_up > 0 && blockIdx.x % give_up == 0 ? 0 : polls;
}


// Exchange area of one layer of a call: flags of the hidden tiles [token tile][32], tagged token sets
// [token tile][E].
constexpr int kMaxHidTiles = 32;  // d_h <= 512
__device__ __forceinline__ uint64_t* flag_words(const SmallMod& M) { return reinterpret_cast<uint64_t*>(M.sync); }
__device__ __forceinline__ uint64_t* set_words(const SmallMod& M) { return flag_words(M) + kSmallMaxTiles * kMaxHidTiles; }
__device__ __forceinline__ uint32_t* tickets_of(const SmallMod& M) { return reinterpret_cast<uint32_t*>(M.tickets); }
// tag: the call's number in the upper 48 bits
__device__ __forceinline__ bool has_tag(uint64_t word, uint64_t tag) { return (word >> 16) == (tag >> 16); }

template <typename V>
__device__ __forceinline__ void store_agent(V* p, V v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename V>
__device__ __forceinline__ V load_agent(const V* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The two sides of an exchange.  Writer: its stores are out (vmcnt) before it announces them.  Reader: once
// it has seen the announcement, and branched on it, its loads are issued, and an agent-scope load finds
// no older value in a cache.  The fences forbid the compiler to move an access to the other side; at wavefront scope
// they are no instruction (an agent-scope acquire would invalidate the L2 under the weight stream).
__device__ __forceinline__ void stores_are_out() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    wait_vmem();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}
__device__ __forceinline__ void announcement_seen() { __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront"); }

// ---- router and gate ------------------------------------------------------------------------------
// Hidden units 16 h .. + 15 of the tokens of tile tt: KQ wavefronts split K and add up through LDS
// (red[KQ][64]), kB k-steps per request.  Returns, in wavefront 0, lane (q, c): hidden units
// 16 h + 4 q + r of token c.
template <int KQ, int kB>
__device__ __forceinline__ bf16x4 small_hidden_tile(const SmallMod& M, const __bf16* __restrict__ x, int h, int tt,
                                                    int T, int d, f32x4* red) {
    const int tid = threadIdx.x, lane = tid & 63, q = lane >> 4, c = lane & 15;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int NK32 = d / 32, per = NK32 / KQ;
    const __bf16* af = M.r1f + (((size_t)h * NK32 + w * per) * 64 + lane) * 8;
    const __bf16* xr = x + (size_t)min(16 * tt + c, T - 1) * d + 8 * q + 32 * w * per;
    bf16x4 b1 = {};
    if (M.r_b1) {
#pragma unroll
        for (int r = 0; r < 4; ++r) b1[r] = M.r_b1[16 * h + 4 * q + r];
    }
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 a[2][kB], b[2][kB];
    auto load = [&](int kb, int set) {
#pragma unroll
        for (int i = 0; i < kB; ++i)
            if (kb + i < per) {  // uniform
                a[set][i] = load8(af + (size_t)(kb + i) * 512);
                b[set][i] = load8(xr + 32 * (kb + i));
            }
    };
    auto multiply = [&](int kb, int set) {
#pragma unroll
        for (int i = 0; i < kB; ++i)
            if (kb + i < per) acc = mfma16(a[set][i], b[set][i], acc);
    };
    load(0, 0);
    for (int kb = 0; kb < per; kb += 2 * kB) {
        load(kb + kB, 1);
        multiply(kb, 0);
        if (kb + 2 * kB < per) load(kb + 2 * kB, 0);
        multiply(kb + kB, 1);
    }
    red[w * 64 + lane] = acc;
    __syncthreads();
    bf16x4 hv = {};
    if (w == 0) {
        f32x4 sum = red[lane];
#pragma unroll
        for (int k = 1; k < KQ; ++k) sum += red[k * 64 + lane];
#pragma unroll
        for (int r = 0; r < 4; ++r) hv[r] = (__bf16)fmaxf(sum[r] + (float)b1[r], 0.0f);
    }
    return hv;
}

template <int KQ>
__device__ __forceinline__ void small_hidden_wg(const SmallMod& M, const __bf16* __restrict__ x, int h, int tt, int T, int d,
                                int dh, uint64_t tag, char* smem) {
    const bf16x4 hv = small_hidden_tile<KQ, 8>(M, x, h, tt, T, d, reinterpret_cast<f32x4*>(smem));
    const int lane = threadIdx.x & 63, q = lane >> 4, c = lane & 15;
    if (threadIdx.x < 64) {
        store_agent(reinterpret_cast<uint64_t*>(M.hid + (size_t)(16 * tt + c) * dh + 16 * h + 4 * q),
                    __builtin_bit_cast(uint64_t, hv));
        stores_are_out();
        if (lane == 0) store_agent(flag_words(M) + tt * kMaxHidTiles + h, tag);
    }
}

// Second router product and gate of token tile tt; KS2 = d_h / 32.  The scores stay in registers: lane (q, c)
// of expert tile et holds the experts 16 et + 4 q + r of token c, so the ballot over "kept" of one r is the
// token sets of four experts, and only the row maxima go through LDS.  The mask words, which nobody in
// this launch waits for, are assembled after the announcement.
template <int KQ, int KS2>
__device__ __forceinline__ void small_gate_wg(const SmallMod& M, const __bf16* __restrict__ x, int tt, int T, int d,
                                              int E, uint64_t tag, int budget, char* smem) {
    constexpr int dh = 32 * KS2, NH = dh / 16, kHRow = 2 * dh + 16;  // (bytes per hidden row, bank skew)
    constexpr int kThreads = 64 * KQ, kTiles = KS2 >= 8 ? (KS2 == 8 ? 4 : 2) : 8;  // R2 tiles requested ahead
    constexpr int kMost = kSmallGateMaxE / 16 / KQ;                // tiles per wavefront
    const int tid = threadIdx.x, lane = tid & 63, q = lane >> 4, c = lane & 15;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int W = (E + 63) >> 6, NE = (E + 15) >> 4;
    char* hid = smem;                                              // [16][kHRow]
    float* pmax = reinterpret_cast<float*>(smem + 16 * kHRow);     // [KQ][16]
    int* s_missing = reinterpret_cast<int*>(pmax + 16 * KQ);
    f32x4* red = reinterpret_cast<f32x4*>(smem);                   // (fallback) [KQ][64]

    // this wavefront's expert tiles w, w + KQ, ...: the first ones' fragments are requested now
    bf16x8 r2[kTiles][KS2];
    auto load_r2 = [&](int j, bf16x8 (&a)[KS2]) {
        const int et = min(w + KQ * j, NE - 1);
#pragma unroll
        for (int ks = 0; ks < KS2; ++ks) a[ks] = load8(M.r2f + (((size_t)et * KS2 + ks) * 64 + lane) * 8);
    };
#pragma unroll
    for (int j = 0; j < kTiles; ++j)
        if (w + KQ * j < NE) load_r2(j, r2[j]);  // uniform
    // wait for the hidden rows
    const uint64_t* flags = flag_words(M) + tt * kMaxHidTiles;
    bool missing = true;
    for (int poll = 0; poll < budget && missing; ++poll) {
        const bool here = lane >= NH || load_agent(flags + min(lane, NH - 1)) == tag;
        missing = __ballot(!here) != 0ull;
        if (missing) __builtin_amdgcn_s_sleep(1);
    }
    const uint64_t* hsrc = reinterpret_cast<const uint64_t*>(M.hid + (size_t)16 * tt * dh);
    constexpr int kWords = 16 * dh / 4 / kThreads;                 // 8-byte words per thread
    static_assert(kWords >= 1, "hidden rows");
    uint64_t hw[kWords];
    auto load_hidden = [&]() {
#pragma unroll
        for (int k = 0; k < kWords; ++k) hw[k] = load_agent(hsrc + k * kThreads + tid);
    };
    announcement_seen();
    if (!missing) load_hidden();
    if (tid == 0) *s_missing = 0;
    lds_barrier();
    if (missing && lane == 0) *s_missing = 1;
    lds_barrier();
    if (*s_missing != 0) {  // (uniform) compute them here
        __syncthreads();
        for (int h = 0; h < NH; ++h) {
            const bf16x4 hv = small_hidden_tile<KQ, 1>(M, x, h, tt, T, d, red);
            if (w == 0)
                store_agent(reinterpret_cast<uint64_t*>(M.hid + (size_t)(16 * tt + c) * dh + 16 * h + 4 * q),
                            __builtin_bit_cast(uint64_t, hv));
            __syncthreads();
        }
        stores_are_out();
        __syncthreads();
        announcement_seen();
        load_hidden();
    }
#pragma unroll
    for (int k = 0; k < kWords; ++k) {
        const int i = k * kThreads + tid;  // word i % (dh / 4) of row i / (dh / 4)
        *reinterpret_cast<uint64_t*>(hid + (i / (dh / 4)) * kHRow + (i % (dh / 4)) * 8) = hw[k];
    }
    lds_barrier();
    // s = |R2 hid + c2|, 0 for the experts from E on
    const int tok = 16 * tt + c;
    bf16x8 hb[KS2];
#pragma unroll
    for (int ks = 0; ks < KS2; ++ks) hb[ks] = *reinterpret_cast<const bf16x8*>(hid + c * kHRow + ks * 64 + q * 16);
    float sc[kMost][4];
    float mx = 0.0f;  // (the scores are not negative)
    auto score_tile = [&](const bf16x8 (&a)[KS2], int j) {
        f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS2; ++ks) acc = mfma16(a[ks], hb[ks], acc);
        return router_scores4(acc, M.r_b2, min(16 * (w + KQ * j) + 4 * q, E - 1), E);
    };
#pragma unroll
    for (int j = 0; j < kMost; ++j) {
        const int e0 = 16 * (w + KQ * j) + 4 * q;
        if (w + KQ * j >= NE) break;  // uniform
        if (j >= kTiles) load_r2(j, r2[j % kTiles]);
        const float4 o = score_tile(r2[j % kTiles], j);
        sc[j][0] = e0 < E ? o.x : 0.0f; sc[j][1] = e0 < E ? o.y : 0.0f;
        sc[j][2] = e0 < E ? o.z : 0.0f; sc[j][3] = e0 < E ? o.w : 0.0f;
#pragma unroll
        for (int r = 0; r < 4; ++r) mx = fmaxf(mx, sc[j][r]);
        if (M.scores && tok < T && e0 < E) store_scores4(M.scores + (size_t)tok * E, e0, E, o);
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    if (q == 0) pmax[w * 16 + c] = mx;
    lds_barrier();
#pragma unroll
    for (int k = 0; k < KQ; ++k) mx = fmaxf(mx, pmax[k * 16 + c]);
    // the exact comparison: the fp64 product of two fp32 numbers is exact
    const double thr = (double)M.tau * (double)mx;
    const uint32_t keep_all = M.tau == 0.0f ? 1u : 0u, live = tok < T ? 1u : 0u;
    uint16_t* cm16 = reinterpret_cast<uint16_t*>(M.colmask);
    uint64_t* sets = set_words(M) + (size_t)tt * E;
    uint32_t bits[kMost];  // lane (q, c): its four experts of token c
#pragma unroll
    for (int j = 0; j < kMost; ++j) {
        const int et = w + KQ * j, e0 = 16 * et + 4 * q;
        if (et >= NE) break;  // uniform
        bits[j] = 0;
        uint64_t bal[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t ge = (double)sc[j][r] >= thr ? 1u : 0u;
            const uint32_t k = (keep_all | ge) & live & (e0 + r < E ? 1u : 0u);
            bits[j] |= k << r;
            bal[r] = __ballot(k);
        }
        // lane (q, c < 4): the set of expert 16 et + 4 q + c, announced and for small_down
        const uint64_t mine = c == 0 ? bal[0] : (c == 1 ? bal[1] : (c == 2 ? bal[2] : bal[3]));
        if (c < 4 && e0 + c < E) {
            const uint32_t set = (uint32_t)(mine >> (16 * q)) & 0xffffu;
            store_agent(sets + e0 + c, tag | set);
            cm16[4 * (e0 + c) + tt] = (uint16_t)set;
        }
    }
    // mask words, a quarter (the 16 experts of a tile) at a time; the quarters from E on are zero
    uint16_t* mask16 = reinterpret_cast<uint16_t*>(M.mask) + (size_t)tok * (4 * W);
#pragma unroll
    for (int j = 0; j < kMost; ++j) {
        const int et = w + KQ * j;
        if (et >= 4 * W) break;  // uniform
        uint32_t b = et < NE ? bits[j] << (4 * q) : 0u;
        b |= __shfl_xor(b, 16, 64);
        b |= __shfl_xor(b, 32, 64);
        if (q == 0 && tok < T) mask16[et] = (uint16_t)b;
    }
}

// ---- up-projection --------------------------------------------------------------------------------
// W8: the weight fragments hold one E4M3 byte per weight (half the stream); they are converted to
// bf16 in registers, and the per-expert power-of-two scales are applied to the fp32 sums.
// MTW: 16-row neuron tiles per work item (an expert's MT / MTW items follow each other); TT: token tiles; KQ
// wavefronts split K.  A workgroup takes the items b, b + n_wg, ... of all the experts or, once the token
// sets are known, of the touched ones; their weights are one stream: a fragment's registers are filled
// with the next batch as soon as it has been multiplied.
template <bool GATED, int MTW, int TT, bool W8, int KQ>
__global__ __launch_bounds__(64 * KQ, 2) void small_up_kernel(
    const SmallGroup G, const __bf16* __restrict__ x_router, const __bf16* __restrict__ x, int T, int d,
    int m, int MT, int act, int E, int dh, uint64_t tag, int wait, int n_wg, int give_up) {
    constexpr int BR = GATED ? 2 : 1;
    // k-steps whose weights are in flight (half of it where the accumulators leave no more registers)
    constexpr int kFrags = (TT + BR >= 5 && !W8 ? 16 : 32) / (BR * MTW);
    constexpr int kB = kFrags < 16 ? kFrags : 16;
    // ... and whose x rows are, as many as the registers allow: loads come back in order, so a wait for x rows that were
    // requested kX steps ago leaves only kX steps of weights on their way.  (Up-projection at 256 gated experts of
    // 64, d = 2048, with 2, or kB / 2 at one token tile, ahead -> kX: bf16 32 tokens 27.5 -> 25.3 us, 48: 27.8 -> 26.5;
    // e4m3 16: 21.3 -> 19.7, 32: 22.3 -> 19.9, 48: 24.9 -> 22.0, 64: 27.1 -> 26.5.)
    constexpr int kMostX = (W8 ? 24 : 16) / TT;
    constexpr int kX = kMostX >= 16 && kB >= 16 ? 16 : (kMostX >= 8 && kB >= 8 ? 8 : 4);
    static_assert(kB % kX == 0, "ring");
    // The first requests: step by step, but the weights before x where a wavefront's share of K is all on its way at
    // once and x is a small part of it (bf16, 16 tokens: 25.6 us step by step, 24.5 this way).
    constexpr bool kMixed = W8 || TT > 1;
    constexpr int kRefill = kMixed ? 1 : kX / 2;  // x rows requested again at once
    const SmallMod& M = G.m[blockIdx.z];
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int tid = threadIdx.x, lane = tid & 63, q = lane >> 4, c = lane & 15;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    int b = blockIdx.x;
    if (b == 0) {  // tickets of small_down
        for (int i = tid; i < d / 16; i += 64 * KQ) tickets_of(M)[i] = 0u;
    }
    if (dh > 0) {
        const int n_hidden = (dh / 16) * TT;
        if (b < n_hidden) {
            small_hidden_wg<KQ>(M, x_router, b % (dh / 16), b / (dh / 16), T, d, dh, tag, smem);
            return;
        }
        b -= n_hidden;
        if (b < TT) {
            const int budget = wait_budget(kHiddenPolls, give_up);
            switch (dh) {
            case 64: small_gate_wg<KQ, 2>(M, x_router, b, T, d, E, tag, budget, smem); return;
            case 128: small_gate_wg<KQ, 4>(M, x_router, b, T, d, E, tag, budget, smem); return;
            case 256: small_gate_wg<KQ, 8>(M, x_router, b, T, d, E, tag, budget, smem); return;
            default: small_gate_wg<KQ, 16>(M, x_router, b, T, d, E, tag, budget, smem); return;
            }
        }
        b -= TT;
    }
    const int per_e = MT / MTW;
    const int NK32 = d / 32, per = NK32 / KQ, k0 = w * per;  // KQ divides NK32
    f32x4* red = reinterpret_cast<f32x4*>(smem);             // [KQ][MTW][TT][BR][64]

    // compact list of the touched experts and their token sets: each wavefront scans kScan words a lane at a time
    constexpr int kScan = 4;
    constexpr uint64_t kAll = TT == 4 ? ~0ull : (1ull << (16 * TT)) - 1ull;
    uint64_t* s_cm = reinterpret_cast<uint64_t*>(red + KQ * MTW * TT * BR * 64);  // [E]
    uint16_t* s_list = reinterpret_cast<uint16_t*>(s_cm + E);                     // [E]
    bool compact = dh == 0 || ((wait >> blockIdx.z) & 1) != 0;
    int n_items = E * per_e, stride = n_wg;
    if (compact) {
        int* s_n = reinterpret_cast<int*>(red);  // [KQ] experts found; -1: not all announced in time
        const uint64_t* sets = set_words(M);
        const int budget = wait_budget(kSetPolls, give_up);
        int n_touched = 0, polls = 0;
        for (int round = 0; round < E; round += 64 * kScan * KQ) {
            const int base = round + 64 * kScan * w;
            uint64_t cm[kScan];
            int n = 0;
            if (base < E) {
                bool all_in = dh == 0;
                for (; polls < budget && !all_in; ++polls) {  // one word first: of some expert, another one per workgroup
                    all_in = __ballot(!has_tag(load_agent(sets + base + b % min(E - base, 64 * kScan)), tag)) == 0ull;
                    if (!all_in) __builtin_amdgcn_s_sleep(4);
                }
                all_in = false;
                for (; !all_in; ++polls) {
                    bool mine = true;
#pragma unroll
                    for (int k = 0; k < kScan; ++k) {
                        const int e = min(base + 64 * k + lane, E - 1);
                        cm[k] = 0ull;
                        if (dh == 0) {
                            cm[k] = M.colmask[e] & kAll;
                        } else {
#pragma unroll
                            for (int tt = 0; tt < TT; ++tt) {
                                const uint64_t v = load_agent(sets + (size_t)tt * E + e);
                                mine = mine && has_tag(v, tag);
                                cm[k] |= (v & 0xffffull) << (16 * tt);
                            }
                        }
                        if (base + 64 * k + lane >= E) cm[k] = 0ull;
                    }
                    all_in = __ballot(!mine) == 0ull;
                    if (!all_in && polls >= budget) break;
                }
#pragma unroll
                for (int k = 0; k < kScan; ++k) n += __popcll(__ballot(cm[k] != 0ull));
                if (!all_in) n = -1;
            }
            if (lane == 0) s_n[w] = n;
            lds_barrier();
            int at = n_touched;
            bool all_in = true;
#pragma unroll
            for (int k = 0; k < KQ; ++k) {
                const int nk = __builtin_amdgcn_readfirstlane(s_n[k]);
                all_in = all_in && nk >= 0;
                at += k < w ? nk : 0;
                n_touched += nk;
            }
            if (!all_in) {
                n_touched = -1;
                break;
            }
            if (n > 0) {
#pragma unroll
                for (int k = 0; k < kScan; ++k) {
                    const uint64_t bal = __ballot(cm[k] != 0ull);
                    if (cm[k] != 0ull) {
                        const int i = at + __popcll(bal & ((1ull << lane) - 1ull));
                        s_list[i] = (uint16_t)(base + 64 * k + lane);
                        s_cm[i] = cm[k];
                    }
                    at += __popcll(bal);
                }
            }
            lds_barrier();
        }
        if (n_touched >= 0) {
            n_items = n_touched * per_e;
        } else {  // all items, whatever the others do
            lds_barrier();
            compact = false;
            b = 0;
            stride = 1;
        }
    } else if (dh > 0) {
        // let the router's loads go first: behind the stream they would take three times as long (64 clocks a
        // unit; with 32 units instead of 8, 24 to 64 tokens of 256 x 64 were 0.2 to 1 us slower)
        __builtin_amdgcn_s_sleep(kMixed ? 8 : 32);
    }
    auto expert_of = [&](int item) {
        return compact ? __builtin_amdgcn_readfirstlane((int)s_list[item / per_e]) : item / per_e;
    };

    typedef typename std::conditional<W8, uint2, bf16x8>::type Frag;
    Frag a[kB][MTW][BR];
    // fragments of k-step kb + i of an item (at: the item's first fragment)
    auto first_of = [&](int item) {
        return (((size_t)expert_of(item) * MT + (item % per_e) * MTW) * NK32 + k0) * 512 + lane * 8;
    };
    auto load_step = [&](bool some, size_t first, int kb, int i) {
        if (some && kb + i < per) {  // uniform
#pragma unroll
            for (int t = 0; t < MTW; ++t)
#pragma unroll
                for (int br = 0; br < BR; ++br) {
                    const size_t at = first + ((size_t)t * NK32 + kb + i) * 512;
                    if constexpr (W8) a[i][t][br] = *reinterpret_cast<const uint2*>((br ? M.wgatef8 : M.wupf8) + at);
                    else a[i][t][br] = load8((br ? M.wgatef : M.wupf) + at);
                }
        }
    };
    int item = b;
    if (item >= n_items) return;
    size_t first = first_of(item);
    // Nothing is on its way any more, but the compiler, which sees the loads of the scan above in one of the
    // paths to here, would wait for them (vmcnt(0)) before each of the following requests: one after the
    // other instead of all at once, 2 us of the kernel's 26 at 32 tokens of 256 x 64.
    wait_vmem();
    const __bf16* xr[TT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) xr[tt] = x + (size_t)min(16 * tt + c, T - 1) * d + 8 * q + 32 * k0;
    bf16x8 xb[kX][TT];
    auto load_x = [&](int k, int i) {
        if (k < per) {  // uniform
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) xb[i][tt] = load8(xr[tt] + 32 * k);
        }
    };
#pragma unroll
    for (int i = 0; i < kB; ++i) {
        load_step(true, first, 0, i);
        if (kMixed && i < kX) load_x(i, i);
    }
#pragma unroll
    for (int i = 0; i < kX; ++i)
        if (!kMixed) load_x(i, i);
    const bool x_stays = kB == kX && per <= kB;  // one batch: its x rows serve every item
    for (;;) {
        const int next = item + stride;
        const bool more = next < n_items;
        const size_t first_next = more ? first_of(next) : 0;
        f32x4 acc[MTW][BR][TT];
#pragma unroll
        for (int t = 0; t < MTW; ++t)
#pragma unroll
            for (int br = 0; br < BR; ++br)
#pragma unroll
                for (int tt = 0; tt < TT; ++tt) acc[t][br][tt] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int kb = 0; kb < per; kb += kB) {
            const bool end = kb + kB >= per;
            const bool some = !end || more;
            const size_t first_load = end ? first_next : first;
            const int kb_load = end ? 0 : kb + kB;
#pragma unroll
            for (int i = 0; i < kB; ++i) {
                if (kb + i < per) {
#pragma unroll
                    for (int t = 0; t < MTW; ++t)
#pragma unroll
                        for (int br = 0; br < BR; ++br) {
                            bf16x8 av;
                            if constexpr (W8) av = e4m3x8_to_bf16(a[i][t][br]);
                            else av = a[i][t][br];
#pragma unroll
                            for (int tt = 0; tt < TT; ++tt)
                                acc[t][br][tt] = mfma16(av, xb[i % kX][tt], acc[t][br][tt]);
                        }
                }
                load_step(some, first_load, kb_load, i);
                if ((i + 1) % kRefill == 0) {
                    if (i + kX < kB) {
#pragma unroll
                        for (int j = i + 1 - kRefill; j <= i; ++j) load_x(kb + j + kX, j % kX);
                    } else if (some && !x_stays) {
#pragma unroll
                        for (int j = i + 1 - kRefill; j <= i; ++j) load_x(kb_load + j + kX - kB, j % kX);
                    }
                }
            }
        }
        // add the K slices up
#pragma unroll
        for (int t = 0; t < MTW; ++t)
#pragma unroll
            for (int tt = 0; tt < TT; ++tt)
#pragma unroll
                for (int br = 0; br < BR; ++br)
                    red[(((w * MTW + t) * TT + tt) * BR + br) * 64 + lane] = acc[t][br][tt];
        lds_barrier();
        const int e = expert_of(item), mt0 = (item % per_e) * MTW;
        const uint64_t set = compact ? s_cm[item / per_e] : kAll;
        float s_up = 1.0f, s_gate = 1.0f, s_down = 1.0f;
        if (W8) {
            s_up = M.w_scales[3 * e + 0];
            s_gate = M.w_scales[3 * e + 1];
            s_down = M.w_scales[3 * e + 2];  // folded into H: the down kernel sums over experts
        }
        for (int i = w; i < MTW * TT; i += KQ) {
            const int t = i / TT, tt = i % TT, mt = mt0 + t;
            f32x4 s[BR];
#pragma unroll
            for (int br = 0; br < BR; ++br) {
                s[br] = red[(i * BR + br) * 64 + lane];
#pragma unroll
                for (int k = 1; k < KQ; ++k) s[br] += red[((k * MTW * TT + i) * BR + br) * 64 + lane];
            }
            // lane (q, c): neurons neuron_of_slot(mt, 4q + r) of token c of tile tt
            const bool keep = 16 * tt + c < T && ((set >> (16 * tt + c)) & 1ull);
            bf16x4 hv;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int n = neuron_of_slot(mt, 4 * q + r);
                float v;
                if (GATED) {
                    v = activate_fast(act, s[BR - 1][r] * s_gate) * (s[0][r] * s_up);
                } else {
                    const float bias = M.b_up ? (float)M.b_up[(size_t)e * m + min(n, m - 1)] : 0.0f;
                    v = activate_fast(act, s[0][r] * s_up + bias);
                }
                v *= s_down;
                if (n >= m || !keep) v = 0.0f;
                hv[r] = (__bf16)v;
            }
            *reinterpret_cast<bf16x4*>(M.Hs + ((((size_t)e * (MT / 2) + (mt >> 1)) * TT + tt) * 64 + lane) * 8 + (mt & 1) * 4) = hv;
        }
        if (!more) break;
        lds_barrier();  // the slices of the next item take the same place
        item = next;
        first = first_next;
    }
}

// ---- down-projection ------------------------------------------------------------------------------
// grid = (16 CTW-column groups, expert groups, layers); KS = m_pad / 32; NW wavefronts split the experts
// (wavefront w: e0 + w, + NW, ...; at most 64 each), U of the touched ones in flight.  (Requesting the weights
// ahead of the token sets, of all experts, never gained more than 0.3 us, and lost from 2 MB on that
// nobody wanted: 0.6 to 2 us at 5 MB, 6 to 14 at 30.)
template <int KS, int TT, int CTW, int NW, int U, bool W8>
__global__ __launch_bounds__(64 * NW) void small_down_kernel(const SmallGroup G, int T, int d, int E, int per,
                                                             int dh) {
    const SmallMod& M = G.m[blockIdx.z];
    extern __shared__ __attribute__((aligned(16))) char smem[];
    f32x4* red = reinterpret_cast<f32x4*>(smem);  // [NW][CTW][TT][64]
    __shared__ int s_last;
    const int tid = threadIdx.x, lane = tid & 63, q = lane >> 4, c = lane & 15;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int cg = blockIdx.x, eg = blockIdx.y, EG = gridDim.y;
    const int e_first = eg * per + w, e_end = min(E, eg * per + per);
    constexpr uint64_t kAll = TT == 4 ? ~0ull : (1ull << (16 * TT)) - 1ull;
    // lane i: the token set of this wavefront's i-th expert
    const int e_lane = e_first + NW * lane;
    const uint64_t cm = e_lane < e_end ? M.colmask[e_lane] & kAll : 0ull;
    uint64_t todo = __ballot(cm != 0ull);

    const size_t w_tile = (size_t)KS * 512, w_expert = (size_t)(d / 16) * w_tile;  // elements
    const size_t wl = (size_t)(CTW * cg) * w_tile + lane * 8;
    typedef typename std::conditional<W8, uint2, bf16x8>::type Frag;
    f32x4 acc[CTW][TT];
#pragma unroll
    for (int ct = 0; ct < CTW; ++ct)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) acc[ct][tt] = f32x4{0.f, 0.f, 0.f, 0.f};
    // a ring of U experts in flight: a slot is filled again as soon as it has been multiplied
    Frag wa[U][CTW][KS];
    bf16x8 hb[U][KS][TT];
    int at[U];
    auto request = [&](int u) {
        at[u] = -1;
        if (todo != 0ull) {  // uniform
            at[u] = __builtin_ctzll(todo);
            todo &= todo - 1ull;
            const int e = e_first + NW * at[u];
#pragma unroll
            for (int ct = 0; ct < CTW; ++ct)
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    const size_t p = (size_t)e * w_expert + wl + ct * w_tile + ks * 512;
                    if constexpr (W8) wa[u][ct][ks] = *reinterpret_cast<const uint2*>(M.w2f8 + p);
                    else wa[u][ct][ks] = load8(M.w2f + p);
                }
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                for (int tt = 0; tt < TT; ++tt)
                    hb[u][ks][tt] = load8(M.Hs + (((size_t)e * KS + ks) * TT + tt) * 512 + lane * 8);
        }
    };
#pragma unroll
    for (int u = 0; u < U; ++u) request(u);
    bool more = at[0] >= 0;
    while (more) {  // uniform
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (at[u] >= 0) {
                const uint32_t lo = __builtin_amdgcn_readlane((int)(uint32_t)cm, at[u]);
                const uint32_t hi = TT > 2 ? __builtin_amdgcn_readlane((int)(uint32_t)(cm >> 32), at[u]) : 0;
#pragma unroll
                for (int tt = 0; tt < TT; ++tt) {
                    const bool keep = ((tt < 2 ? lo : hi) >> (16 * (tt & 1) + c)) & 1u;
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) {
                        const bf16x8 hv = keep ? hb[u][ks][tt] : zero8();
#pragma unroll
                        for (int ct = 0; ct < CTW; ++ct) {
                            bf16x8 av;
                            if constexpr (W8) av = e4m3x8_to_bf16(wa[u][ct][ks]);
                            else av = wa[u][ct][ks];
                            acc[ct][tt] = mfma16(av, hv, acc[ct][tt]);
                        }
                    }
                }
                request(u);
            }
        }
        more = at[0] >= 0;
    }
#pragma unroll
    for (int ct = 0; ct < CTW; ++ct)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) red[((w * CTW + ct) * TT + tt) * 64 + lane] = acc[ct][tt];
    if (dh > 0) {  // the flags of small_up, for the next replay
        const int stride = 64 * NW * gridDim.x * EG, first = (eg * gridDim.x + cg) * 64 * NW + tid;
        for (int i = first; i < kSmallMaxTiles * kMaxHidTiles + TT * E; i += stride) flag_words(M)[i] = 0ull;
    }
    lds_barrier();
    // wavefront i < CTW TT: column tile i / TT, token tile i % TT; lane (q, c): four columns of token c
    typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
    // (shares lie in accumulator order, so that a wavefront writes and reads whole lines)
    auto share = [&](int g, int i) {
        return reinterpret_cast<uint64_t*>(M.partial) + (((size_t)g * gridDim.x + cg) * (CTW * TT) + i) * 128 + lane;
    };
    auto out = [&](int t, int col, f32x4 v) {
        bf16x4 o;
#pragma unroll
        for (int r = 0; r < 4; ++r) o[r] = (__bf16)(v[r] + (M.b_down ? (float)M.b_down[col + r] : 0.0f));
        *reinterpret_cast<bf16x4*>(M.y + (size_t)t * d + col) = o;
    };
    for (int i = w; i < CTW * TT; i += NW) {
        f32x4 v = red[i * 64 + lane];
#pragma unroll
        for (int k = 1; k < NW; ++k) v += red[(k * CTW * TT + i) * 64 + lane];
        const int t = 16 * (i % TT) + c, col = 16 * (CTW * cg + i / TT) + 4 * q;
        if (t < T) {
            if (EG == 1) out(t, col, v);
        }
        if (EG > 1) {
            const u64x2 u = __builtin_bit_cast(u64x2, v);
            store_agent(share(eg, i), (uint64_t)u[0]);
            store_agent(share(eg, i) + 64, (uint64_t)u[1]);
        }
    }
    if (EG == 1) return;
    stores_are_out();
    __syncthreads();
    if (tid == 0)
        s_last = __hip_atomic_fetch_add(tickets_of(M) + cg, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)(EG - 1);
    __syncthreads();
    if (!s_last) return;
    announcement_seen();
    for (int i = w; i < CTW * TT; i += NW) {
        const int t = 16 * (i % TT) + c, col = 16 * (CTW * cg + i / TT) + 4 * q;
        f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int g0 = 0; g0 < EG; g0 += 8) {
            u64x2 u[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const uint64_t* p = share(min(g0 + k, EG - 1), i);
                u[k] = u64x2{load_agent(p), load_agent(p + 64)};
            }
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (g0 + k < EG) v += __builtin_bit_cast(f32x4, u[k]);
        }
        if (t < T) out(t, col, v);
    }
}

// Number of this call for the flags: never the same twice in a process, and unlikely to be what an
// unused workspace holds.
uint64_t next_tag() {
    static std::atomic<uint64_t> counter{(uint64_t)std::chrono::steady_clock::now().time_since_epoch().count() * 0x9e3779b97f4a7c15ull};
    return (counter.fetch_add(1, std::memory_order_relaxed) << 16) | 0x8000000000000000ull;  // (never the zero of a cleared word)
}

thread_local int g_give_up = 0;

// Share of the experts that a token keeps at threshold tau, for the scores of a random router: the share
// of a half-normal distribution above tau times the median of the largest of E.
double expected_density(int E, double tau) {
    double top = sqrt(2.0 * log(E + 1.0));
    for (int i = 0; i < 2; ++i) top = sqrt(std::max(0.45, 2.0 * log(1.15 * E / top)));  // E erfc(top / sqrt 2) = ln 2
    return std::max(erfc(tau * top * M_SQRT1_2), 1.0 / E);
}

// Whether an up-projection with the gate inside reads the weights of all experts without waiting for the
// token sets: the sets are there about 7 us after the launch, and against that stands the time to read,
// at 5 TB/s, what nobody of the T tokens turns out to want.  Measured with either course at 1 to 64
// tokens and thresholds 0.3 to 0.9 (256 x 64, 1024 x 24, 128 x 24, 24 x 128; weights from HBM and from the
// last-level cache): reading all is ahead by 2 to 16 us below 5 MB unwanted, between 7 ahead and 4 behind from 24
// to 36 MB, behind by 2 to 9 us from 55 to 66 MB and by 10 to 16 above 110.
bool small_reads_all(const dmoe_layer& L, int T, float tau) {
    const double bytes = (double)L.n_experts * (L.gated ? 2 : 1) * m_pad_of(L.expert_size) * L.d_model *
                         (weights_fp8(L) ? 1 : 2);
    constexpr double kUnwanted = 5e6 * 7.0;
    return bytes < kUnwanted || bytes * pow(1.0 - expected_density(L.n_experts, tau), T) < kUnwanted;
}

template <bool GATED, int MTW, int TT, bool W8, int KQ>
void launch_up_t(const dmoe_layer& L, const SmallGroup& G, int n_layers, const void* x_router, const void* x,
                 int T, bool gate, hipStream_t s) {
    const int E = L.n_experts, MT = m_pad_of(L.expert_size) / 16, dh = gate ? L.router_hidden : 0;
    size_t lds = (size_t)KQ * MTW * TT * (GATED ? 2 : 1) * 1024;
    int wait = 0;  // bit i: layer i waits for its token sets
    for (int i = 0; i < n_layers && gate; ++i) wait |= small_reads_all(L, T, G.m[i].tau) ? 0 : 1 << i;
    if (!gate || wait) lds += (sizeof(uint64_t) + sizeof(uint16_t)) * (size_t)E;
    if (gate)
        lds = std::max(lds, 16 * (2 * (size_t)dh + 16) + 16 * KQ * sizeof(float) + 16);
    static std::once_flag attr_once;  // kernel attributes: once per process, thread-safe
    std::call_once(attr_once, [&] {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&small_up_kernel<GATED, MTW, TT, W8, KQ>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    });
    // Two workgroups per CU are resident; with more items than that each takes several.
    const int n_wg = std::min(E * (MT / MTW), 512);
    launch_kernel(small_up_kernel<GATED, MTW, TT, W8, KQ>, dim3((dh > 0 ? (dh / 16 + 1) * TT : 0) + n_wg, 1, n_layers),
                  64 * KQ, lds, s, G, (const __bf16*)x_router, (const __bf16*)x, T, L.d_model, L.expert_size,
                  MT, L.act, E, dh, gate ? next_tag() : 0, wait, n_wg, g_give_up);
}

template <bool GATED, bool W8>
void launch_up_tt(const dmoe_layer& L, const SmallGroup& G, int n_layers, const void* x_router, const void* x,
                  int T, bool gate, hipStream_t s) {
    // One token tile: one neuron tile per workgroup, so that a few touched experts still spread over
    // the chip.  More: two, which halves the reads of x.
    switch (div_up(T, 16)) {
    case 1: launch_up_t<GATED, 1, 1, W8, 4>(L, G, n_layers, x_router, x, T, gate, s); break;
    case 2: launch_up_t<GATED, 2, 2, W8, 4>(L, G, n_layers, x_router, x, T, gate, s); break;
    case 3: launch_up_t<GATED, 2, 3, W8, 4>(L, G, n_layers, x_router, x, T, gate, s); break;
    default: launch_up_t<GATED, 2, 4, W8, 4>(L, G, n_layers, x_router, x, T, gate, s); break;
    }
}

template <int KS, bool W8>
void launch_down_tt(const dmoe_layer& L, const SmallGroup& G, int n_layers, int T, bool gate, hipStream_t s) {
    const int E = L.n_experts, d = L.d_model, TT = div_up(T, 16);
    const int dh = gate ? L.router_hidden : 0;
    // One token tile: 16 columns and 16 wavefronts per workgroup, which needs no shares in memory up to
    // a few experts per wavefront.  More: 32 columns, so that the hidden rows are read less often, and still 16
    // wavefronts, so that each has few experts to go through (8 where four token tiles of 128-neuron
    // experts leave no registers for 16).  64 columns and 8 wavefronts read the hidden rows half as often, but
    // write twice the shares: 128 x 24, d = 768, 32 / 64 tokens 8.8 / 10.3 us against 6.5 / 7.7; 256 x 64, d = 2048,
    // 15.7 / 19.2 against 14.6 / 17.2, from HBM 18.9 / 22.8 against 18.0 / 21.8.  16 columns: 16.5 at 32 tokens.
    // They stay for weights that come from HBM (below); E4M3, of which 32 columns are runs of 2 KB instead of 4: down weights of
    // 67 MB, 32 / 64 tokens, 20.2 / 26.7 us against 21.4 / 28.7, of 33 MB 12.4 / 16.1 against 12.8 / 16.5, and from the
    // last-level cache 17 MB 8.5 / 11.1 against 7.9 / 9.8.
    // Expert groups: one, or enough workgroups to fill the chip, and no more shares than the workspace
    // holds (kSmallMaxGroups x 16 rows).  The same for a layer of a group as for a layer alone: the
    // sums must not depend on that.
    auto go = [&](auto kernel, int ctw, int nw, int EG) {
        EG = std::max(std::min({EG, kSmallMaxGroups, kSmallMaxGroups / TT}), div_up(E, 64 * nw));
        const int per = div_up(E, std::max(1, EG));
        const size_t lds = (size_t)nw * ctw * TT * 1024;
        launch_kernel(kernel, dim3(d / (16 * ctw), div_up(E, per), n_layers), 64 * nw, lds, s, G, T, d, E, per, dh);
    };
    constexpr int U1 = KS <= 2 ? 4 : 2;  // (more would not fit the registers)
    constexpr int U2 = KS <= 2 ? 2 : 1, U4 = KS == 1 ? 2 : 1, NW4 = KS <= 2 ? 16 : 8;
    const int eg1 = div_up(E, 128);
    // As many groups as leave at most one workgroup per CU (of 16 wavefronts there is room for one, and a few in a second round cost as
    // much as the first).  Rounded up / down, us: d = 1280 (280 / 240 workgroups), 1000 x 24, 20 / 40 / 60 tokens 22.3 / 26.2 / 28.8 and 17.4
    // / 19.1 / 20.6; d = 768 (264 / 240), 1000 x 48, 20 tokens 29.2 and 22.1; d = 3072 (288 / 192), 500 x 24 23.9 / 28.0 / 30.4
    // and 19.2 / 20.8 / 22.7.
    const auto groups = [&](int ctw, int nw) { return std::min(std::max(1, 256 / (d / (16 * ctw))), E / nw); };
    // Weights from HBM: runs of 64 columns.  bf16 beyond the last-level cache or near it, 32 / 64 columns, 60 tokens: 1000 x 24, d = 3072
    // (196 MB) 59.4 / 41.3; 1600 x 24, d = 2048 (209 MB) 53.1 / 44.9, 1000 (131 MB) 27.4 / 28.6; d = 1536 1000 x 48 (196 MB) 50.4 / 48.0;
    // narrower layers not: d = 768, 1000 x 128 (196 MB) 59.2 / 75.2.
    if (TT > 1 && (W8 ? (size_t)E * 32 * KS * d > ((size_t)24 << 20) : d >= 1536 && (size_t)E * 64 * KS * d > ((size_t)150 << 20))) {
        switch (TT) {
        case 2: go(small_down_kernel<KS, 2, 4, 8, U2, W8>, 4, 8, groups(4, 8)); return;
        case 3: go(small_down_kernel<KS, 3, 4, 8, U2, W8>, 4, 8, groups(4, 8)); return;
        default: go(small_down_kernel<KS, 4, 4, 8, U2, W8>, 4, 8, groups(4, 8)); return;
        }
    }
    switch (TT) {
    case 1: go(small_down_kernel<KS, 1, 1, 16, U1, W8>, 1, 16, eg1); break;
    case 2: go(small_down_kernel<KS, 2, 2, 16, U2, W8>, 2, 16, groups(2, 16)); break;
    case 3: go(small_down_kernel<KS, 3, 2, 16, U2, W8>, 2, 16, groups(2, 16)); break;
    default: go(small_down_kernel<KS, 4, 2, NW4, U4, W8>, 2, NW4, groups(2, NW4)); break;
    }
}

}  // namespace

void small_give_up(int every) { g_give_up = every; }

size_t small_sync_bytes(const dmoe_layer& L) {
    return 8 * (size_t)kSmallMaxTiles * (kMaxHidTiles + std::min(L.n_experts, kSmallGateMaxE));
}
size_t small_ticket_bytes(const dmoe_layer& L) { return sizeof(uint32_t) * (size_t)(L.d_model / 16); }

bool small_bf16_supported(const dmoe_layer& L) {
    const int mp = m_pad_of(L.expert_size);
    return (mp == 32 || mp == 64 || mp == 128) && L.d_model % 256 == 0;
}

void launch_small_bf16(const dmoe_layer& L, const SmallGroup& G, int n_layers, const void* x_router,
                       const void* x, int T, bool gate, hipStream_t s) {
    const bool w8 = weights_fp8(L);
    {
        LaunchTimer tm(kSlotSmallUp, s);
        if (L.gated && w8) launch_up_tt<true, true>(L, G, n_layers, x_router, x, T, gate, s);
        else if (L.gated) launch_up_tt<true, false>(L, G, n_layers, x_router, x, T, gate, s);
        else if (w8) launch_up_tt<false, true>(L, G, n_layers, x_router, x, T, gate, s);
        else launch_up_tt<false, false>(L, G, n_layers, x_router, x, T, gate, s);
    }
    LaunchTimer tm(kSlotSmallDown, s);
    switch (m_pad_of(L.expert_size) / 32 * 2 + (w8 ? 1 : 0)) {
    case 2: launch_down_tt<1, false>(L, G, n_layers, T, gate, s); break;
    case 3: launch_down_tt<1, true>(L, G, n_layers, T, gate, s); break;
    case 4: launch_down_tt<2, false>(L, G, n_layers, T, gate, s); break;
    case 5: launch_down_tt<2, true>(L, G, n_layers, T, gate, s); break;
    case 8: launch_down_tt<4, false>(L, G, n_layers, T, gate, s); break;
    default: launch_down_tt<4, true>(L, G, n_layers, T, gate, s); break;
    }
}

}  // namespace dmoe
