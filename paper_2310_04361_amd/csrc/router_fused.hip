// Router (Sec. 3.3) fused with the dynamic-k gate (Sec. 3.4 Eq. 4) and the per-group expert counts
// that start the bucketing: one workgroup per group of 64 tokens.
//
//   stage 1  hid^T[d_h][64] = R1 * x^T.  The 64 x rows are staged in LDS (eight lanes per 128-byte
//            row piece), up to 768 columns at a time with all loads of the chunk in flight
//            together; each of the four wavefronts owns a quarter of the hidden units and reads
//            R1 as packed MFMA fragments.  bias + relu, round to bf16, park the hidden tile in LDS.
//   stage 2  s^T[E][64] = R2 * hid^T.  Each wavefront owns every fourth tile of 16 experts, reads
//            R2 as packed fragments and the hidden tile from LDS; |. + c2| goes to `scores`
//            (fp32, 16 bytes per lane) and stays in registers for
//   select   per-token maximum across the four wavefronts (LDS), the exact comparison
//            (double)s >= (double)tau * (double)max on those very fp32 scores, mask words
//            assembled per token, then the 64x64 ballot transpose that counts, per expert, the
//            tokens of the group that keep it.
// The scores that are written and the mask come from the same registers, so a caller that gates
// the returned scores again gets the same mask bit for bit.
#include <algorithm>
#include <type_traits>

#include "dmoe_internal.h"
#include "mfma.h"
#include "quantize.h"

namespace dmoe {

namespace {

constexpr int kMaxTilesPerWave = 8;   // expert tiles per wavefront: E <= 4 * 8 * 16 = 512

// Eight rows x 128 bytes, 16 bytes a lane, straight to 1 KB of LDS
__device__ __forceinline__ void row_set_to_lds(const __bf16* p, char* lds) {
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)p, (__attribute__((address_space(3))) void*)lds, 16, 0, 0);
}

// NH = d_h / 16; ETW = expert tiles per wavefront (E <= 64 * ETW); KBC = K blocks (64 wide) of x
// that sit in LDS at a time: 12 (all of d = 768) when there is at most about one workgroup per
// CU and its own latency is what counts, 4 when several workgroups share a CU and hide it.
// TT = tiles of 16 tokens per workgroup: 4 (a whole select group of 64 tokens), or 2 / 1 when
// there are too few groups to fill the chip -- a workgroup then handles a half or a quarter of a
// group and writes its expert counts to its own row of a table with 4 / TT rows per group, which
// the scan over the groups adds up.
// MODE: kWhole: both products (and the gate) in one workgroup.  A router whose two matrices take
// megabytes (d_h = 512, thousands of experts) would stream all of them through every CU; it runs
// as two launches instead, with the matrices split over blockIdx.y: kHiddenSlice computes the NH * 16
// hidden units from blockIdx.y * NH * 16 on and stores them to hid_g[T][dh_g]; kScoresSlice (NH * 16 =
// d_h) reads the stored hidden rows and computes the expert tiles blockIdx.y * tiles_y .. + tiles_y - 1.
enum { kWhole = 0, kHiddenSlice = 1, kScoresSlice = 2 };
// Registers for four workgroups per CU, whose LDS they leave room for.
constexpr bool four_per_cu(int nh, int etw, int kbc, int mode) { return mode == kWhole && kbc == 4 && nh <= 8 && etw <= 2; }
// DIRECT: the rows of x straight to LDS, which want x at a 16-byte address; otherwise through registers, all loads of a chunk
// in flight as well.  (Written block by block as they came, the router alone on an x at 8 bytes from such an address took, 128 experts,
// d = 768, 16384 tokens 10.6 us, so 9.1; 50000 tokens 35.0 / 29.7; d = 2048, d_h = 256, 256 experts, 8000 tokens 25.2 / 20.8.)
template <int NH, int ETW, int KBC, int TT, int MODE = kWhole, bool DIRECT = true>
__global__ __launch_bounds__(256, (DIRECT && four_per_cu(NH, ETW, KBC, MODE) ? 4 : 1)) void router_fused_kernel(
    const __bf16* __restrict__ x, const __bf16* __restrict__ r1f, const __bf16* __restrict__ r_b1,
    const __bf16* __restrict__ r2f, const __bf16* __restrict__ r_b2, float* __restrict__ scores,
    int T, int d, int E, float tau, int do_select /* 2: token sets */, uint64_t* __restrict__ mask,
    int32_t* __restrict__ group_cnt, __bf16* __restrict__ hid_g, int dh_g, int tiles_y) {
    constexpr int dh = NH * 16, HT = NH / 4, TOK = 16 * TT;
    constexpr int kBlock = TOK * 128;    // bytes of a staged K block: rows of 128
    constexpr int kHRow = dh * 2 + 16;  // bytes per hidden row in LDS
    extern __shared__ __attribute__((aligned(128))) char smem[];
    char* xs = smem;                                            // [KBC][TOK][128]
    // [TOK][kHRow]: afterwards, in the place of x, where several workgroups shall fit a CU
    constexpr bool kInPlace = KBC == 4;
    char* hid = MODE == kScoresSlice || kInPlace ? smem : smem + KBC * kBlock;
    float* pmax = reinterpret_cast<float*>(hid + TOK * kHRow);  // [4][64]
    uint64_t* pw = reinterpret_cast<uint64_t*>(pmax + 256);     // [4][64][W]
    const int W = (E + 63) >> 6;
    uint64_t* fin = pw + 4 * 64 * W;                            // [64][W]

    const int g = blockIdx.x, t0 = g * TOK;  // g: row of the count table
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, q = lane >> 4, c = lane & 15;
    const int NK32 = d / 32, NKB = d / 64;

    // ---------------------------------------------------------------- stage 1
    // x comes from HBM: all loads of a chunk are issued together so that their latency is paid
    // once per chunk, not once per K block (loads complete in issue order, so a prefetch of x
    // inside the K loop would hold up the R1 fragments behind it).  The K loop itself has no
    // barrier and only L2-resident loads.
    // Straight to LDS, eight rows a load (staged through registers, a ds_write_b128 took 35 clocks of the CU per KB): 16-byte
    // piece p of row r of a block lies at p ^ (r / 2), so that the 16 lanes that read a piece of 16 rows use all the banks.
    // Forward, through registers / so: 128 experts of 24, d = 768, 300 tokens 35.6 / 35.4 us, 3000 62.9 / 62.5, 16384 126.3 / 126.3, 50432 (with
    // the hidden rows in the place of x, two -> four workgroups per CU) 358.7 / 354.5; 512 experts of 6, 1300 tokens 57.2 / 57.0, 5000 105.7 / 106.6;
    // 256 experts of 8, d = 1024, d_h = 512, 20000 tokens 259 / 248.
    constexpr int kRowSets = TOK / 8;                        // loads per K block, dealt to the wavefronts in turn
    constexpr int kOwn = kRowSets >= 4 ? kRowSets / 4 : 1;   // row sets of a wavefront
    const __bf16* xp[kOwn];
#pragma unroll
    for (int i = 0; i < kOwn; ++i) {
        const int rs = kRowSets >= 4 ? w + 4 * i : w % kRowSets, r = lane >> 3;
        xp[i] = x + (size_t)min(t0 + 8 * rs + r, T - 1) * d + 8 * ((lane & 7) ^ (4 * (rs & 1) + (r >> 1)));
    }
    // (a hidden slice starts at hidden tile blockIdx.y * NH)
    const __bf16* af = r1f + (((size_t)(MODE == kHiddenSlice ? blockIdx.y * NH : 0) + w * HT) * NK32 * 64 + lane) * 8;

    f32x4 acc[HT][TT];
#pragma unroll
    for (int h = 0; h < HT; ++h)
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) acc[h][tt] = f32x4{0.f, 0.f, 0.f, 0.f};

    // R1 fragments: a ring of four K blocks, requested three blocks before their use (an L2
    // round trip takes longer than the 16 to 32 MFMAs of one block)
    bf16x8 ar[4][2][HT];
    auto load_a = [&](int kb, bf16x8 (&a)[2][HT]) {
        kb = min(kb, NKB - 1);  // the last trips re-read a block they will not use
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int h = 0; h < HT; ++h) a[ks][h] = load8(af + ((size_t)h * NK32 + 2 * kb + ks) * 512);
    };
    auto compute = [&](int kbl, const bf16x8 (&a)[2][HT]) {
        const char* src = xs + kbl * kBlock + c * 128;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            bf16x8 b[TT];
#pragma unroll
            for (int tt = 0; tt < TT; ++tt)
                b[tt] = *reinterpret_cast<const bf16x8*>(src + tt * 16 * 128 + (((4 * ks + q) ^ (c >> 1)) << 4));
#pragma unroll
            for (int h = 0; h < HT; ++h)
#pragma unroll
                for (int tt = 0; tt < TT; ++tt) acc[h][tt] = mfma16(a[ks][h], b[tt], acc[h][tt]);
        }
    };

    if constexpr (MODE != kScoresSlice) {
    for (int kb0 = 0; kb0 < NKB; kb0 += KBC) {
        const int nkb = min(KBC, NKB - kb0);  // a multiple of 4: d is a multiple of 256
        constexpr int kAtOnce = kRowSets >= 4 ? 1 : 4 / kRowSets;  // K blocks that the wavefronts share at a time
        auto place = [&](int k0, int i, int& k) {
            k = kRowSets >= 4 ? k0 : k0 + w / kRowSets;
            return xs + k * kBlock + ((kRowSets >= 4 ? w : w % kRowSets) + 4 * i) * 1024;
        };
        bf16x8 xr[DIRECT ? 1 : KBC / kAtOnce][kOwn];
        if constexpr (!DIRECT) {
#pragma unroll
            for (int j = 0; j < KBC / kAtOnce; ++j)
                if (j * kAtOnce < nkb) {
#pragma unroll
                    for (int i = 0; i < kOwn; ++i) {
                        int k;
                        place(j * kAtOnce, i, k);
                        xr[j][i] = load8(xp[i] + 64 * (kb0 + k));
                    }
                }
        }
        if (DIRECT && kb0 == 0) {
#pragma unroll
            for (int i = 0; i < 3; ++i) load_a(i, ar[i]);
        }
        if (kb0 > 0) lds_barrier();  // the previous chunk has been consumed
#pragma unroll
        for (int j = 0; j < KBC / kAtOnce; ++j)
            if (j * kAtOnce < nkb) {
#pragma unroll
                for (int i = 0; i < kOwn; ++i) {
                    int k;
                    char* const to = place(j * kAtOnce, i, k);
                    if constexpr (DIRECT) row_set_to_lds(xp[i] + 64 * (kb0 + k), to);
                    else *reinterpret_cast<bf16x8*>(to + lane * 16) = xr[j][i];
                }
            }
        if constexpr (DIRECT) wait_vmem();
        if (!DIRECT && kb0 == 0) {  // behind x, which is waited for alone
#pragma unroll
            for (int i = 0; i < 3; ++i) load_a(i, ar[i]);
        }
        lds_barrier();
        for (int kbl = 0; kbl < nkb; kbl += 4) {  // nkb is a multiple of 4
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                load_a(kb0 + kbl + i + 3, ar[(i + 3) & 3]);
                compute(kbl + i, ar[i]);
            }
        }
    }

    }  // stage 1

    // R2 fragments of this wavefront's first expert tile: requested now, so that their latency
    // passes while the hidden tile is finished and stored
    constexpr int KS2 = dh / 32;
    const int NE = (E + 15) >> 4;
    // two sets of R2 fragments alternate (a third in flight measured the same on a router of
    // 2048 experts and d_h = 512)
    constexpr int kR2Ring = 2;
    bf16x8 r2a[kR2Ring][KS2];
    auto load_r2 = [&](int et, bf16x8 (&a)[KS2]) {
        et = min(et, NE - 1);
#pragma unroll
        for (int ks = 0; ks < KS2; ++ks) a[ks] = load8(r2f + (((size_t)et * KS2 + ks) * 64 + lane) * 8);
    };
    if constexpr (MODE == kScoresSlice) load_r2(blockIdx.y * tiles_y + w, r2a[0]);
    else if constexpr (MODE == kWhole) load_r2(w, r2a[0]);

    if constexpr (MODE == kWhole && kInPlace) lds_barrier();  // every wavefront is done with x
    // lane (q, c) of tile (h, tt): hidden units 16*(w*HT + h) + 4q + r of token 16tt + c
#pragma unroll
    for (int h = 0; h < HT && MODE != kScoresSlice; ++h) {
        const int hu0 = 16 * (w * HT + h) + 4 * q;                      // within this workgroup's units
        const int hu_g = (MODE == kHiddenSlice ? blockIdx.y * dh : 0) + hu0;  // within the layer's
        float b1[4] = {0.f, 0.f, 0.f, 0.f};
        if (r_b1) {
#pragma unroll
            for (int r = 0; r < 4; ++r) b1[r] = (float)r_b1[hu_g + r];
        }
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
            bf16x4 hv;
#pragma unroll
            for (int r = 0; r < 4; ++r) hv[r] = (__bf16)fmaxf(acc[h][tt][r] + b1[r], 0.0f);
            if constexpr (MODE == kHiddenSlice) {
                const int t = t0 + 16 * tt + c;
                if (t < T) *reinterpret_cast<bf16x4*>(hid_g + (size_t)t * dh_g + hu_g) = hv;
            } else {
                *reinterpret_cast<bf16x4*>(hid + (16 * tt + c) * kHRow + hu0 * 2) = hv;
            }
        }
    }
    if constexpr (MODE == kHiddenSlice) return;
    if constexpr (MODE == kScoresSlice) {
        // the stored hidden rows of the group's tokens: 16-byte pieces, rows past T read row T - 1
        // (all loads of a thread in flight before the first store)
        constexpr int kPieces = dh / 8, kTrips = TOK * kPieces / 256;
        bf16x8 hr[kTrips];
#pragma unroll
        for (int j = 0; j < kTrips; ++j) {
            const int i = tid + 256 * j, row = i / kPieces, piece = i % kPieces;
            hr[j] = load8(hid_g + (size_t)min(t0 + row, T - 1) * dh_g + piece * 8);
        }
#pragma unroll
        for (int j = 0; j < kTrips; ++j) {
            const int i = tid + 256 * j, row = i / kPieces, piece = i % kPieces;
            *reinterpret_cast<bf16x8*>(hid + row * kHRow + piece * 16) = hr[j];
        }
    }
    lds_barrier();  // the hidden tile is in LDS (a full barrier would also wait for global stores)

    // ---------------------------------------------------------------- stage 2
    // scores of expert tile et for the group's 64 tokens: |R2 hid + c2| to `scores` and to o
    auto score_tile = [&](int et, const bf16x8 (&a)[KS2], float (&o)[TT][4]) {
        f32x4 a2[TT];
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) a2[tt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS2; ++ks) {
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) {
                const bf16x8 b = *reinterpret_cast<const bf16x8*>(
                    hid + (16 * tt + c) * kHRow + ks * 64 + q * 16);
                a2[tt] = mfma16(a[ks], b, a2[tt]);
            }
        }
        const int e0 = 16 * et + 4 * q;  // this lane: experts e0 .. e0+3
        // the second-layer biases as an accumulator-shaped vector (0 for experts from E on)
        // (every load unconditional, from a clamped index: under `if (e0 + r < E)` each of them
        // became a block of its own that waited for its value before the next one was requested)
        f32x4 b2 = f32x4{0.f, 0.f, 0.f, 0.f};
        if (r_b2) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float bv = (float)r_b2[min(e0 + r, E - 1)];
                b2[r] = e0 + r < E ? bv : 0.0f;
            }
        }
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
            const int t = t0 + 16 * tt + c;
            // padding experts (from E on) score 0
            const float4 out = e0 < E ? router_scores4(a2[tt] + b2, nullptr, e0, E)
                                      : make_float4(0.f, 0.f, 0.f, 0.f);
            if (scores && t < T && e0 < E) store_scores4(scores + (size_t)t * E, e0, E, out);
            o[tt][0] = out.x; o[tt][1] = out.y; o[tt][2] = out.z; o[tt][3] = out.w;
        }
    };
    if (!do_select) {
        // router alone: any number of expert tiles, the fragments of the next tile on their way
        // while the current one is multiplied
        float o[TT][4];
        const int et0 = MODE == kScoresSlice ? blockIdx.y * tiles_y : 0;
        const int et1 = MODE == kScoresSlice ? min(NE, et0 + tiles_y) : NE;
        load_r2(et0 + w + 4, r2a[1]);
        for (int et = et0 + w; et < et1; et += 4 * kR2Ring) {
#pragma unroll
            for (int i = 0; i < kR2Ring; ++i) {
                if (et + 4 * i < et1) score_tile(et + 4 * i, r2a[i], o);  // uniform per wavefront
                load_r2(et + 4 * (i + kR2Ring), r2a[i]);  // past the end: the last tile again
            }
        }
        return;
    }
    float sc[ETW][TT][4];  // [my tile][token tile][r]
    float vmax[TT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) vmax[tt] = 0.f;
#pragma unroll
    for (int j = 0; j < ETW; ++j) {
        const int et = w + 4 * j;
        if (j + 1 < ETW) load_r2(et + 4, r2a[(j + 1) & 1]);
        if (et < NE) {  // uniform per wavefront
            score_tile(et, r2a[j & 1], sc[j]);
#pragma unroll
            for (int tt = 0; tt < TT; ++tt)
                vmax[tt] = fmaxf(vmax[tt], fmaxf(fmaxf(sc[j][tt][0], sc[j][tt][1]),
                                                 fmaxf(sc[j][tt][2], sc[j][tt][3])));
        }
    }

    // ---------------------------------------------------------------- select
    // maximum of each token over this wavefront's experts, then over the four wavefronts
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
        float m = vmax[tt];
        m = fmaxf(m, __shfl_xor(m, 16, 64));
        m = fmaxf(m, __shfl_xor(m, 32, 64));
        if (q == 0) pmax[w * 64 + 16 * tt + c] = m;
    }
    lds_barrier();  // LDS only: the scores' stores to global memory need not have landed
    const uint32_t keep_all = tau == 0.0f ? 1u : 0u;
    double thr[TT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) {
        const int tk = 16 * tt + c;
        const float m = fmaxf(fmaxf(pmax[tk], pmax[64 + tk]), fmaxf(pmax[128 + tk], pmax[192 + tk]));
        thr[tt] = (double)tau * (double)m;  // exact: at most 48 significant bits
    }
    // this wavefront's bits of each token: its tile et = w + 4j is the only one it has in word j
    // (bits 16w .. 16w+15), so the word is stored whole, zero where the tile lies beyond E
#pragma unroll
    for (int j = 0; j < ETW; ++j) {
        const int et = w + 4 * j;
        const int e0 = 16 * et + 4 * q;
        if (j < W) {  // uniform
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) {
                uint32_t bits = 0;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    // integer logic, no short circuit: as `a || b`, `c && d` this became a
                    // branch around every one of the 64-bit comparisons
                    const uint32_t ge = (double)sc[j][tt][r] >= thr[tt] ? 1u : 0u;
                    const uint32_t in = (et < NE ? 1u : 0u) & (e0 + r < E ? 1u : 0u);
                    bits |= ((keep_all | ge) & in) << (4 * q + r);
                }
                bits |= __shfl_xor(bits, 16, 64);
                bits |= __shfl_xor(bits, 32, 64);  // 16 bits: experts 16et .. 16et+15 of token c
                if (q == 0) pw[(w * 64 + 16 * tt + c) * W + j] = (uint64_t)bits << (16 * w);
            }
        }
    }
    lds_barrier();
    if (tid < 64) {
        const int t = t0 + tid;
        const bool mine = tid < TOK && t < T;  // lanes from TOK up: no token, an all-zero row
        for (int wi = 0; wi < W; ++wi) {
            uint64_t word = 0ull;
            if (tid < TOK)
                word = pw[(0 * 64 + tid) * W + wi] | pw[(1 * 64 + tid) * W + wi] |
                       pw[(2 * 64 + tid) * W + wi] | pw[(3 * 64 + tid) * W + wi];
            fin[tid * W + wi] = mine ? word : 0ull;
            if (mine) mask[(size_t)t * W + wi] = word;
        }
    }
    lds_barrier();
    // ballot transpose: lane = token; wavefront w handles the experts 64wi + 16w .. +15 of every
    // word wi (sixteen ballots per word and wavefront)
    for (int wi = 0; wi < W; ++wi) {
        const uint64_t word = fin[lane * W + wi];
        uint64_t col = 0;  // lane b: which tokens of the group keep expert 64wi + b
#pragma unroll
        for (int bi = 0; bi < 16; ++bi) {
            const int b = 16 * w + bi;
            const uint64_t bal = __ballot((word >> b) & 1ull);
            if (lane == b) col = bal;
        }
        const int e = 64 * wi + lane;
        // (two: token sets instead of their sizes, of 16 tokens a workgroup)
        if ((lane >> 4) == w && e < E) group_cnt[(size_t)g * E + e] = TT == 1 && do_select == 2 ? (int32_t)col : __popcll(col);
    }
}

template <int NH, int ETW, int KBC, int TT>
void launch_t3(const dmoe_layer& L, const void* x, int T, float* scores, float tau, uint64_t* mask,
               int32_t* group_cnt, bool sets, hipStream_t s) {
    const PackedLayout P = packed_layout(L);
    const int E = L.n_experts, W = div_up(E, 64);
    constexpr int TOK = 16 * TT;
    const size_t hid = TOK * (NH * 32 + 16) + 256 * 4 + (mask ? (size_t)5 * 64 * W * 8 : 0);  // the gate's words only when it runs
    const size_t lds = KBC == 4 ? std::max<size_t>(TOK * KBC * 128, hid) : TOK * KBC * 128 + hid;
    const char* pk = static_cast<const char*>(L.packed);
    auto go = [&](auto kernel, std::once_flag& attr_once) {
        std::call_once(attr_once, [&] {  // kernel attributes: once per process, thread-safe
            (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
        });
        launch_kernel(kernel, div_up(T, TOK), 256, lds, s,
            (const __bf16*)x, (const __bf16*)(pk + P.r1f), (const __bf16*)L.r_b1,
            (const __bf16*)(pk + P.r2f), (const __bf16*)L.r_b2, scores, T, L.d_model, E, tau,
            mask ? (sets ? 2 : 1) : 0, mask, group_cnt, nullptr, 0, 0);
    };
    static std::once_flag once[2];
    // Through registers also where two workgroups of 32 tokens share a CU and there are more of them than CUs: on an x
    // that comes from memory a workgroup whose loads go to LDS, which can only wait for all of them, then takes longer.  d = 768, 128 experts of
    // 24, forward, straight to LDS / so: 9000 tokens 85.2 / 83.8 us, 10000 91.5 / 90.4, 12000 104.2 / 102.7.
    // With at most one per CU 7000 tokens 75.2 / 75.5; with LDS for one only (512 experts with the gate, 12000 tokens) 177.1 / 177.2.
    const bool share = TT == 2 && div_up(T, TOK) > 256 && lds <= 80 * 1024;
    // And where the router runs alone, which writes all the scores: d = 768, d_h = 128, straight to LDS / so: 512 experts, 5000 tokens 13.2 / 12.4 us,
    // 20000 31.0 / 28.3, 50432 68.3 / 51.1; 128 experts, 50432 39.6 / 33.0; d = 2048, d_h = 256, 20000 tokens 53.1 / 50.3.  Not at d_h = 512
    // (d = 2048, 12500 tokens 44.8 / 55.7, 20000 87 / 109), nor for the chunks of four blocks at d_h = 64 (64 experts, 65536 tokens 25.3 / 27.9;
    // 256 experts, 40000 25.4 / 28.3).
    const bool alone = !mask && NH <= 16 && !(NH == 4 && KBC == 4);
    if (share || alone || (reinterpret_cast<uintptr_t>(x) & 15)) go(router_fused_kernel<NH, ETW, KBC, TT, kWhole, false>, once[1]);
    else go(router_fused_kernel<NH, ETW, KBC, TT>, once[0]);
}

template <int NH, int ETW>
void launch_t2(const dmoe_layer& L, const void* x, int T, int split, float* scores, float tau,
               uint64_t* mask, int32_t* group_cnt, bool sets, hipStream_t s) {
    constexpr int kBig = NH <= 8 ? 12 : (NH == 16 ? 8 : 4);
    // parts of a group per workgroup: only where workgroups are few (one per CU, nothing hides
    // the latency of an x chunk), and the fewer rows leave LDS for chunks of 1024 columns
    if (split == 4)
        launch_t3<NH, ETW, 16, 1>(L, x, T, scores, tau, mask, group_cnt, sets, s);
    else if (split == 2)
        launch_t3<NH, ETW, 16, 2>(L, x, T, scores, tau, mask, group_cnt, sets, s);
    // (chunks of four blocks and the hidden rows in their place: four workgroups of d_h <= 128 and up to 128 experts share a CU
    // and hide each other's latency, which pays as soon as a CU has more than one.  Forward, 128 experts of 24, d = 768, large chunks up to
    // 512 groups / up to 256: 17000 tokens 145.5 / 141.0 us, 20000 157.4 / 152.2, 32768 234.6 / 229.1.  The router alone: up to 512)
    else if (kBig > 4 && div_up(T, 64) <= (mask && four_per_cu(NH, ETW, 4, kWhole) ? 256 : 512))
        launch_t3<NH, ETW, kBig, 4>(L, x, T, scores, tau, mask, group_cnt, sets, s);
    else
        launch_t3<NH, ETW, 4, 4>(L, x, T, scores, tau, mask, group_cnt, sets, s);
}

// ---- hidden rows of a large router, tile by tile ------------------------------------------------------
// hid[T][d_h] = relu(x R1^T + c1) rounded to bf16.  What bounds it is how many bytes a CU gets: with one workgroup per 16
// tokens for the whole router every CU read all of R1.  Every sum is ONE chain of MFMAs over the k-steps in
// ascending order, as in router_fused_kernel: a hidden value has the same bits whichever of the forms runs, so
// that dmoe_forward decides by the very scores that dmoe_router returns at every batch size.  (K split over four wavefronts, as it
// once was, is up to 1.2 us faster at 65 to 250 tokens, d = 2048: the chain is 64 MFMAs long.  In tiles of 16 x 16, a quarter of K's operands
// held by each wavefront and the sum handed on, those batches take the same time as in 32 x 32.)
// Workgroup b runs on XCD b % 8: by_tokens, one XCD takes all the hidden units of a tile of tokens, so that x leaves
// memory once, and R1, which is then the smaller, once per XCD; otherwise an XCD takes a few hidden units of all the
// tokens.
constexpr int kHidRow = 144;  // bytes per staged x row: 64 columns and 16 bytes of bank skew

// Second product, gate and counts of a router of more than 512 experts: a workgroup has 16 tokens and all the experts, its
// eight wavefronts NTW tiles of 16 experts each, whose scores stay in registers until the token's maximum is known.  Sums,
// decisions and rows of counts are those of router_fused_kernel and gate_counts_kernel.  What bounds it: every workgroup
// reads all of R2 out of its XCD's L2 (2 MB for 2048 experts and d_h = 512: 15 us at 60 B per clock and CU); as two launches the
// scores went to memory and back (4096 tokens: 33 MB each way).
template <int KS2, int NTW>
__global__ __launch_bounds__(512, 2) void scores_gate_kernel(
    const __bf16* __restrict__ hid, const __bf16* __restrict__ r2f, const __bf16* __restrict__ r_b2,
    float* __restrict__ scores, int T, int E, float tau, uint64_t* __restrict__ mask, int32_t* __restrict__ cnt, int sets) {
    __shared__ float pmax[8][16];
    const int lane = threadIdx.x & 63, q = lane >> 4, c = lane & 15;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t = (int)blockIdx.x * 16 + c, W = (E + 63) >> 6, NE = (E + 15) >> 4, et0 = w * NTW;
    const bool real = t < T;
    // R2 fragments one after the other through a ring, two tiles' worth in flight
    constexpr int kFrags = NTW * KS2, kAhead = 16;
    bf16x8 ring[kAhead];
    const __bf16* const rp = r2f + lane * 8;
    auto request = [&](int f) {  // (past the last tile of the router that tile again)
        const int et = min(et0 + f / KS2, NE - 1);
        ring[f % kAhead] = load8(rp + ((size_t)et * KS2 + f % KS2) * 512);
    };
    bf16x8 b[KS2];
    const __bf16* const hrow = hid + (size_t)min(t, T - 1) * (KS2 * 32) + 8 * q;
#pragma unroll
    for (int ks = 0; ks < KS2; ++ks) b[ks] = load8(hrow + 32 * ks);
#pragma unroll
    for (int f = 0; f < kAhead; ++f) request(f);
    float sc[NTW][4], m = 0.f;
#pragma unroll
    for (int j = 0; j < NTW; ++j) {
        f32x4 a2 = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS2; ++ks) {
            const int f = j * KS2 + ks;
            a2 = mfma16(ring[f % kAhead], b[ks], a2);
            if (f + kAhead < kFrags) request(f + kAhead);
        }
        const int e0 = 16 * (et0 + j) + 4 * q;  // this lane: experts e0 .. e0+3 of token c
        f32x4 b2 = f32x4{0.f, 0.f, 0.f, 0.f};
        if (r_b2) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float bv = (float)r_b2[min(e0 + r, E - 1)];
                b2[r] = e0 + r < E ? bv : 0.0f;
            }
        }
        // padding experts (from E on) score 0
        const float4 out = e0 < E ? router_scores4(a2 + b2, nullptr, e0, E) : make_float4(0.f, 0.f, 0.f, 0.f);
        if (scores && real && e0 < E) store_scores4(scores + (size_t)t * E, e0, E, out);
        sc[j][0] = out.x; sc[j][1] = out.y; sc[j][2] = out.z; sc[j][3] = out.w;
        m = fmaxf(m, fmaxf(fmaxf(out.x, out.y), fmaxf(out.z, out.w)));
        __builtin_amdgcn_sched_barrier(0);
    }
    m = fmaxf(m, __shfl_xor(m, 16, 64));
    m = fmaxf(m, __shfl_xor(m, 32, 64));
    if (q == 0) pmax[w][c] = m;
    lds_barrier();
    m = pmax[0][c];
#pragma unroll
    for (int i = 1; i < 8; ++i) m = fmaxf(m, pmax[i][c]);
    const double thr = (double)tau * (double)m;  // exact: at most 48 significant bits
    const uint32_t keep_all = tau == 0.0f ? 1u : 0u, row = real ? 1u : 0u;
#pragma unroll
    for (int i = 0; i < NTW / 4; ++i) {
        const int wi = et0 / 4 + i;
        if (wi >= W) break;  // uniform
        uint64_t word = 0ull;  // of token c
        int set = 0;           // of expert 64 wi + lane: which of the tokens keep it
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int e0 = 64 * wi + 16 * k + 4 * q;
            uint32_t bits = 0;
            uint64_t kept[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const uint32_t ge = (double)sc[4 * i + k][r] >= thr ? 1u : 0u;
                const uint32_t keep = (keep_all | ge) & row & (e0 + r < E ? 1u : 0u);
                bits |= keep << (4 * q + r);
                kept[r] = __ballot(keep != 0u);  // bit 16 q + c
            }
            bits |= __shfl_xor(bits, 16, 64);
            bits |= __shfl_xor(bits, 32, 64);
            word |= (uint64_t)bits << (16 * k);
            // lane 16 k + 4 q' + r' takes expert 16 k + 4 q' + r' of the word
            const uint64_t mine = (c & 2) ? ((c & 1) ? kept[3] : kept[2]) : ((c & 1) ? kept[1] : kept[0]);
            const int field = (int)(mine >> (16 * (c >> 2))) & 0xffff;
            set = q == k ? field : set;
        }
        if (q == 0 && real) mask[(size_t)t * W + wi] = word;
        const int e = 64 * wi + lane;
        if (e < E) cnt[(size_t)blockIdx.x * E + e] = sets ? set : __popc(set);
    }
}

// 32 tokens x 16 UT hidden units; a wavefront owns NU tiles of units and 16 TTW tokens.  x goes through LDS, which all
// wavefronts read, in chunks of 256 columns: while chunk k is multiplied, k + 1 is in LDS, k + 2 goes there and k + 3
// and k + 4 are on their way; R1 fragments are requested four chunks ahead.  The last trip of four chunks requests nothing.
// QUANT: the workgroups from n_hidden on quantise the rows of x.
template <int UT, bool QUANT>
__global__ __launch_bounds__(256, UT > 4 ? 1 : 2) void router_hidden_kernel(
    const __bf16* __restrict__ x, const __bf16* __restrict__ r1f, const __bf16* __restrict__ r_b1,
    __bf16* __restrict__ hid_g, int T, int d, int dh, int by_tokens, int n_hidden, const QuantX q) {
    if (QUANT && (int)blockIdx.x >= n_hidden) {
        const int step = 4 * ((int)gridDim.x - n_hidden);
        for (int t = 4 * ((int)blockIdx.x - n_hidden) + (int)(threadIdx.x >> 6); t < T; t += step)
            quantize_row(x, t, d, q.x8, q.xscale, q.xhat);
        return;
    }
    constexpr int NU = UT > 4 ? UT / 4 : 1, WU = UT / NU;  // WU: wavefronts side by side over the units
    constexpr int TTW = WU / 2;
    extern __shared__ __attribute__((aligned(16))) char smem[];  // [4 chunks][4 blocks][32][kHidRow]
    const int lane = threadIdx.x & 63, lq = lane >> 4, c = lane & 15;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n_u = dh / (16 * UT), i = by_tokens ? blockIdx.x >> 3 : blockIdx.x;
    const int t0 = 32 * (by_tokens ? i / n_u * 8 + (blockIdx.x & 7) : i / n_u);
    const int u = i % n_u * UT + w % WU * NU, tt0 = w / WU * TTW;  // this wavefront's first tiles
    if (t0 >= T) return;  // (by_tokens: the last eight)
    const int NK32 = d / 32, NKB = d / 64;
    const int ld_row = threadIdx.x >> 3, ld_piece = threadIdx.x & 7;
    const __bf16* xp = x + (size_t)min(t0 + ld_row, T - 1) * d + 8 * ld_piece;
    const __bf16* af = r1f + (size_t)u * NK32 * 512 + lane * 8;
    char* const xdst = smem + ld_row * kHidRow + ld_piece * 16;
    const char* const xsrc = smem + (16 * tt0 + c) * kHidRow + lq * 16;
    bf16x8 xr[2][4], a[16][NU][2], b[2][2][TTW];  // two chunks of x; R1 of four chunks; x operands of two blocks
    // (past the end: the last block again, never used)
    auto load_x = [&](int kb, bf16x8& r) { r = load8(xp + 64 * min(kb, NKB - 1)); };
    auto park_x = [&](int slot, const bf16x8& r) { *reinterpret_cast<bf16x8*>(xdst + slot * 32 * kHidRow) = r; };
    auto load_a = [&](int kb, bf16x8 (&r)[NU][2]) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int n = 0; n < NU; ++n) r[n][ks] = load8(af + ((size_t)n * NK32 + 2 * min(kb, NKB - 1) + ks) * 512);
    };
    auto read_b = [&](int slot, bf16x8 (&r)[2][TTW]) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int tt = 0; tt < TTW; ++tt)
                r[ks][tt] = *reinterpret_cast<const bf16x8*>(xsrc + (slot * 32 + 16 * tt) * kHidRow + ks * 64);
    };
    f32x4 acc[NU][TTW];
#pragma unroll
    for (int n = 0; n < NU; ++n)
#pragma unroll
        for (int tt = 0; tt < TTW; ++tt) acc[n][tt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 8; ++i) load_x(i, xr[i / 4][i % 4]);
#pragma unroll
    for (int i = 0; i < 8; ++i) load_a(i, a[i]);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        park_x(i, xr[i / 4][i % 4]);
        load_x(8 + i, xr[i / 4][i % 4]);
        load_a(8 + i, a[8 + i]);
    }
    lds_barrier();
    read_b(0, b[0]);
    // chunk C of the trip that starts at block kb0
    auto chunk = [&](auto c_c, auto more_c, int kb0) {
        constexpr int C = decltype(c_c)::value;
        constexpr bool kMore = decltype(more_c)::value;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int i = 4 * C + j;
            __builtin_amdgcn_sched_barrier(0);
            read_b((i + 1) & 15, b[(i + 1) & 1]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int n = 0; n < NU; ++n)
#pragma unroll
                    for (int tt = 0; tt < TTW; ++tt) acc[n][tt] = mfma16(a[i][n][ks], b[i & 1][ks][tt], acc[n][tt]);
            if (kMore || C < 2) park_x((i + 8) & 15, xr[C & 1][j]);
            if (kMore) {
                load_a(kb0 + i + 16, a[i]);
                load_x(kb0 + i + 16, xr[C & 1][j]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        lds_barrier();
    };
    const std::integral_constant<int, 0> c0;
    const std::integral_constant<int, 1> c1;
    const std::integral_constant<int, 2> c2;
    const std::integral_constant<int, 3> c3;
    int kb0 = 0;
    for (; kb0 + 16 < NKB; kb0 += 16) {
        chunk(c0, std::true_type{}, kb0);
        chunk(c1, std::true_type{}, kb0);
        chunk(c2, std::true_type{}, kb0);
        chunk(c3, std::true_type{}, kb0);
    }
    chunk(c0, std::false_type{}, kb0);
    if (kb0 + 4 < NKB) {  // (uniform)
        chunk(c1, std::false_type{}, kb0);
        if (kb0 + 8 < NKB) {
            chunk(c2, std::false_type{}, kb0);
            if (kb0 + 12 < NKB) chunk(c3, std::false_type{}, kb0);
        }
    }
    // lane (q, c) of tile (n, tt): units 16 (u + n) + 4 q .. + 3 of token 16 tt + c
#pragma unroll
    for (int n = 0; n < NU; ++n) {
        const int hu = 16 * (u + n) + 4 * lq;
#pragma unroll
        for (int tt = 0; tt < TTW; ++tt) {
            const int t = t0 + 16 * (tt0 + tt) + c;
            bf16x4 hv;
#pragma unroll
            for (int r = 0; r < 4; ++r) hv[r] = (__bf16)fmaxf(acc[n][tt][r] + (r_b1 ? (float)r_b1[hu + r] : 0.0f), 0.0f);
            if (t < T) *reinterpret_cast<bf16x4*>(hid_g + (size_t)t * dh + hu) = hv;
        }
    }
}

// ---- T <= 16: the same two products spread over many workgroups --------------------------------
// With so few tokens the router is a weight stream (R1 is 1 MiB at d = 2048, d_h = 256) and one
// workgroup per 64 tokens would leave it to a single CU.
//   hidden: workgroup = one tile of 16 hidden units, its (up to) sixteen wavefronts split K and
//           reduce through LDS; hid[16][d_h] (bf16) goes to a small global buffer.
//   scores: wavefront = one tile of 16 experts.
// The gate then runs as the stand-alone mask kernel on the stored scores.
__global__ __launch_bounds__(1024) void router_small_hidden_kernel(
    const SmallGroup G, const __bf16* __restrict__ x, int T, int d, int dh, int KQ) {
    const SmallMod& M = G.m[blockIdx.z];
    const __bf16* __restrict__ r1f = M.r1f;
    const __bf16* __restrict__ r_b1 = M.r_b1;
    __bf16* __restrict__ hid = M.hid;
    __shared__ float red[16][64][4];
    const int h = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, q = lane >> 4, c = lane & 15;
    const int NK32 = d / 32, per = NK32 / KQ;  // KQ <= 16 wavefronts split K; KQ divides NK32
    const __bf16* xr = x + (size_t)min(c, T - 1) * d + 8 * q;
    const __bf16* af = r1f + (((size_t)h * NK32) * 64 + lane) * 8;
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    if (w < KQ) {
#pragma unroll 8
        for (int ks = w * per; ks < (w + 1) * per; ++ks)
            acc = mfma16(load8(af + (size_t)ks * 512), load8(xr + 32 * ks), acc);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) red[w][lane][r] = acc[r];
    __syncthreads();
    if (w == 0) {  // lane (q, c): hidden units 16h + 4q + r of token c
        bf16x4 hv;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float v = 0.0f;
            for (int k = 0; k < KQ; ++k) v += red[k][lane][r];
            if (r_b1) v += (float)r_b1[16 * h + 4 * q + r];
            hv[r] = (__bf16)fmaxf(v, 0.0f);
        }
        *reinterpret_cast<bf16x4*>(hid + (size_t)c * dh + 16 * h + 4 * q) = hv;
    }
}

__global__ __launch_bounds__(256) void router_small_scores_kernel(const SmallGroup G, int T,
                                                                  int dh, int E) {
    const SmallMod& M = G.m[blockIdx.z];
    const __bf16* __restrict__ hid = M.hid;
    const __bf16* __restrict__ r2f = M.r2f;
    const __bf16* __restrict__ r_b2 = M.r_b2;
    float* __restrict__ scores = M.scores;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, q = lane >> 4, c = lane & 15;
    const int et = blockIdx.x * 4 + w;
    if (et >= (E + 15) / 16) return;
    const int KS2 = dh / 32;
    const __bf16* af = r2f + (((size_t)et * KS2) * 64 + lane) * 8;
    const __bf16* hb = hid + (size_t)c * dh + 8 * q;
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int ks = 0; ks < KS2; ++ks)
        acc = mfma16(load8(af + (size_t)ks * 512), load8(hb + 32 * ks), acc);
    const int e0 = 16 * et + 4 * q;
    if (c < T && e0 < E) {
        store_scores4(scores + (size_t)c * E, e0, E, router_scores4(acc, r_b2, e0, E));
    }
}

template <int NH>
void launch_t(const dmoe_layer& L, const void* x, int T, int split, float* scores, float tau,
              uint64_t* mask, int32_t* group_cnt, bool sets, hipStream_t s) {
    if (L.n_experts <= 128 || !mask)  // the router alone keeps no scores in registers
        launch_t2<NH, 2>(L, x, T, split, scores, tau, mask, group_cnt, sets, s);
    else if (L.n_experts <= 256)
        launch_t2<NH, 4>(L, x, T, split, scores, tau, mask, group_cnt, sets, s);
    else
        launch_t2<NH, 8>(L, x, T, split, scores, tau, mask, group_cnt, sets, s);
}

}  // namespace

void launch_router_small(const dmoe_layer& L, const SmallGroup& G, int n_layers, const void* x,
                         int T, hipStream_t s) {
    LaunchTimer tm(kSlotRouter, s);
    const int dh = L.router_hidden, E = L.n_experts;
    int KQ = 16;  // wavefronts that split K: as many as divide the k-steps
    while (KQ > 1 && (L.d_model / 32) % KQ != 0) KQ >>= 1;
    launch_kernel(router_small_hidden_kernel, dim3(dh / 16, 1, n_layers), 1024, 0, s, G, (const __bf16*)x, T,
                  L.d_model, dh, KQ);
    launch_kernel(router_small_scores_kernel, dim3(div_up(div_up(E, 16), 4), 1, n_layers), 256, 0, s, G, T, dh, E);
}

bool router_fused_scores_supported(const dmoe_layer& L) {
    const int dh = L.router_hidden;
    return L.packed != nullptr && (dh == 64 || dh == 128 || dh == 256 || dh == 512) &&
           L.d_model % 256 == 0;
}

bool router_fused_supported(const dmoe_layer& L) {
    return router_fused_scores_supported(L) && L.n_experts <= 64 * kMaxTilesPerWave;
}

// A router whose two matrices take 2 MB or more runs as two launches with the matrices split over
// the workgroups (see router_fused_kernel); needs a [T][d_h] bf16 buffer for the hidden rows.
bool router_sliced(const dmoe_layer& L) {
    const int dh = L.router_hidden;
    return router_fused_scores_supported(L) && (dh == 256 || dh == 512) &&
           2 * (size_t)dh * ((size_t)L.d_model + L.n_experts) >= (2u << 20);
}

template <int NH>
static void launch_scores_slices(const dmoe_layer& L, const PackedLayout& P, int T,
                                 const __bf16* hid, float* scores, hipStream_t s) {
    const int NG = div_up(T, kGroup), NE = div_up(L.n_experts, 16);
    // expert slices: enough workgroups for the chip, at least one tile per wavefront
    const int want = std::max(1, std::min(NE / 4, div_up(256, NG)));
    const int tiles_y = round_up(div_up(NE, want), 4);
    const size_t lds = 64 * (NH * 32 + 16) + 256 * 4;
    static std::once_flag attr_once;  // kernel attributes: once per process, thread-safe
    std::call_once(attr_once, [&] {
        (void)hipFuncSetAttribute(
            reinterpret_cast<const void*>(&router_fused_kernel<NH, 2, 4, 4, kScoresSlice>),
            hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    });
    const char* pk = static_cast<const char*>(L.packed);
    launch_kernel(router_fused_kernel<NH, 2, 4, 4, kScoresSlice>, dim3(NG, div_up(NE, tiles_y)), 256, lds, s, 
        nullptr, nullptr, nullptr, (const __bf16*)(pk + P.r2f), (const __bf16*)L.r_b2, scores, T,
        L.d_model, L.n_experts, 0.0f, 0, nullptr, nullptr,
        const_cast<__bf16*>(hid), L.router_hidden, tiles_y);
}

// Hidden rows of small and medium batches.  Router in all, us, against one workgroup per 16 or 64 tokens and all
// (or 128) hidden units: d = 2048, d_h = 256, 256 experts, 333 / 1000 / 2000 / 4096 / 6000 tokens 16.4 / 16.3 / 18.0 / 20.7 /
// 36.8 before, 11.4 / 12.2 / 14.0 / 19.4 / 27.6 now; d_h = 512, 500 / 1000 / 2000 / 4096 tokens 27.9 / 27.4 / 28.3 / 32.1 before,
// 13.4 / 15.2 / 17.8 / 22.4 now; d_h = 128, 4096 tokens 13.6 before, 11.4 now.
// From 6144 tokens on (6200: 25.0 in one launch, 32.3 in two; d_h = 512, 8192: 36.3 and 42.3) a workgroup of the one
// launch has more than 16 tokens to use its share of R1 for.
static bool router_tiles(const dmoe_layer&, int T) { return div_up(T, kGroup) < 96; }
static bool launch_router_hidden(const dmoe_layer& L, const void* x, int T, void* hid, const QuantX* q, hipStream_t s) {
    const PackedLayout P = packed_layout(L);
    const int dh = L.router_hidden;
    const __bf16* r1f = (const __bf16*)(static_cast<const char*>(L.packed) + P.r1f);
    const int NG = div_up(T, kGroup);
    if (NG * (dh / 128) >= 256) {  // tiles of 64 x 128 fill the chip: 4096 tokens, d_h = 512, 2048 experts 39.5 against 43.8 us
        constexpr int NH = 8, KBC = 12;
        const size_t lds = 64 * KBC * 128;
        auto go = [&](auto kernel, std::once_flag& attr_once) {
            std::call_once(attr_once, [&] {
                (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
            });
            launch_kernel(kernel, dim3(NG, dh / 128), 256, lds, s,
                (const __bf16*)x, r1f, (const __bf16*)L.r_b1, nullptr, nullptr,
                nullptr, T, L.d_model, L.n_experts, 0.0f, 0, nullptr, nullptr,
                (__bf16*)hid, dh, 0);
        };
        static std::once_flag once[2];
        if (reinterpret_cast<uintptr_t>(x) & 15) go(router_fused_kernel<NH, 2, KBC, 4, kHiddenSlice, false>, once[1]);
        else go(router_fused_kernel<NH, 2, KBC, 4, kHiddenSlice>, once[0]);
        return false;
    }
    // x is the larger of the two that the XCDs share (by_tokens 1 / 0, router in all: d_h = 256, 333 tokens 11.5 us either
    // way, 1000 tokens 12.2 / 13.3; d_h = 128, 4096 tokens 11.4 / 15.3; d_h = 512, 333 tokens 14.2 / 13.1, 2000 tokens 17.9 / 18.2)
    const int by_tokens = T >= 2 * dh ? 1 : 0;
    constexpr size_t kTileLds = 16 * 32 * kHidRow;
    const int n4 = div_up(T, 32) * (dh / 64);
    const bool quant = q && n4 <= 256;  // (see below)
    auto go = [&](auto kernel, int tok, int units) {
        const int n = div_up(T, tok), n_hidden = (by_tokens ? round_up(n, 8) : n) * (dh / units);
        launch_kernel(kernel, n_hidden + (quant ? std::min(div_up(T, 4), 256) : 0), 256, kTileLds, s, (const __bf16*)x, r1f,
                      (const __bf16*)L.r_b1, (__bf16*)hid, T, L.d_model, dh, by_tokens, n_hidden, quant ? *q : QuantX{});
    };
    static std::once_flag tile_once;  // kernel attributes: once per process, thread-safe
    std::call_once(tile_once, [] {
        for (const void* f : {reinterpret_cast<const void*>(&router_hidden_kernel<8, false>),
                              reinterpret_cast<const void*>(&router_hidden_kernel<4, false>),
                              reinterpret_cast<const void*>(&router_hidden_kernel<2, false>),
                              reinterpret_cast<const void*>(&router_hidden_kernel<4, true>),
                              reinterpret_cast<const void*>(&router_hidden_kernel<2, true>)})
            (void)hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    });
    // The larger tile reads less and needs workgroups enough to fill the chip.  Router in all, d_h = 256, in tiles of 32 x
    // 32 / 64 / 128: 1000 tokens (n4 = 128) 12.0 / 14.1 / 17.2 us, 1250 (160) 14.5 / 13.3 / 16.6, 2000 (252) 16.4 / 14.0 / 17.5,
    // 3000 (376) 20.0 / 18.8 / 18.0, 4096 (512: as many tiles of 128 as CUs) 24.9 / 19.8 / 18.4, 6000 (752) 36.3 / 27.6 /
    // 30.9; d_h = 512, 500 tokens (128) 13.3 / 14.6 / 16.6, 1000 (256) 16.5 / 15.3 / 16.8, 2000 (504) 23.3 / 19.4 / 17.7.
    // The rows of x are quantised here where the hidden rows leave room for it.  Forward, fully 8-bit layer of 256
    // gated experts of 64, d = 2048, in a launch of its own / here: 300 tokens (n4 = 40) 71 / 67 us, 1000 (128) 105 / 104, 2000 (252)
    // 159 / 156; 4096 tokens 255 / 261.
    if (n4 >= 320 && n4 <= 512) go(router_hidden_kernel<8, false>, 32, 128);
    else if (n4 >= 160 && quant) go(router_hidden_kernel<4, true>, 32, 64);
    else if (n4 >= 160) go(router_hidden_kernel<4, false>, 32, 64);
    else if (quant) go(router_hidden_kernel<2, true>, 32, 32);
    else go(router_hidden_kernel<2, false>, 32, 32);
    return quant;
}

bool router_two_launches(const dmoe_layer& L, int T) {
    return router_fused_supported(L) && L.router_hidden >= 128 && 2 * (size_t)L.router_hidden * L.d_model >= (512u << 10) &&
           router_tiles(L, T);
}

template <int NH, int ETW, int TT>
static void launch_gate_rows(const dmoe_layer& L, int T, const __bf16* hid, float* scores, float tau, uint64_t* mask,
                             int32_t* group_cnt, bool sets, hipStream_t s) {
    const PackedLayout P = packed_layout(L);
    const int E = L.n_experts, W = div_up(E, 64);
    constexpr int TOK = 16 * TT;
    const size_t lds = TOK * (NH * 32 + 16) + 256 * 4 + (size_t)5 * 64 * W * 8;
    static std::once_flag attr_once;  // kernel attributes: once per process, thread-safe
    std::call_once(attr_once, [&] {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&router_fused_kernel<NH, ETW, 4, TT, kScoresSlice>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    });
    launch_kernel(router_fused_kernel<NH, ETW, 4, TT, kScoresSlice>, div_up(T, TOK), 256, lds, s, nullptr, nullptr, nullptr,
                  (const __bf16*)(static_cast<const char*>(L.packed) + P.r2f), (const __bf16*)L.r_b2, scores, T, L.d_model, E,
                  tau, sets ? 2 : 1, mask, group_cnt, const_cast<__bf16*>(hid), L.router_hidden, div_up(E, 16));
}
template <int NH, int ETW>
static void launch_gate_split(const dmoe_layer& L, int T, int split, const __bf16* hid, float* scores, float tau,
                              uint64_t* mask, int32_t* group_cnt, bool sets, hipStream_t s) {
    if (split == 4) launch_gate_rows<NH, ETW, 1>(L, T, hid, scores, tau, mask, group_cnt, sets, s);
    else if (split == 2) launch_gate_rows<NH, ETW, 2>(L, T, hid, scores, tau, mask, group_cnt, sets, s);
    else launch_gate_rows<NH, ETW, 4>(L, T, hid, scores, tau, mask, group_cnt, sets, s);
}
template <int NH>
static void launch_gate(const dmoe_layer& L, int T, int split, const __bf16* hid, float* scores, float tau, uint64_t* mask,
                        int32_t* group_cnt, bool sets, hipStream_t s) {
    if (L.n_experts <= 128) launch_gate_split<NH, 2>(L, T, split, hid, scores, tau, mask, group_cnt, sets, s);
    else if (L.n_experts <= 256) launch_gate_split<NH, 4>(L, T, split, hid, scores, tau, mask, group_cnt, sets, s);
    else launch_gate_split<NH, 8>(L, T, split, hid, scores, tau, mask, group_cnt, sets, s);
}

bool launch_router_two(const dmoe_layer& L, const void* x, int T, int split, void* hid, float* scores, float tau,
                       uint64_t* mask, int32_t* group_cnt, bool sets, const QuantX* q, hipStream_t s) {
    LaunchTimer tm(kSlotRouter, s);
    const bool quantised = launch_router_hidden(L, x, T, hid, q, s);
    const __bf16* h = (const __bf16*)hid;
    if (L.router_hidden == 128) launch_gate<8>(L, T, split, h, scores, tau, mask, group_cnt, sets, s);
    else if (L.router_hidden == 256) launch_gate<16>(L, T, split, h, scores, tau, mask, group_cnt, sets, s);
    else launch_gate<32>(L, T, split, h, scores, tau, mask, group_cnt, sets, s);
    return quantised;
}

// E above 512: the gate of fewer experts is router_fused_kernel's; a wavefront has 16 tiles at most.  Rows of counts as
// gate_counts_kernel leaves them, so below its limit on the tokens (its other condition, more rows of counts than the list fill adds up
// itself, always holds here).  The launch reads all of R2 once per 16 tokens, and takes as long for few tokens as for 4096 and for few experts as for
// the 1024 or 2048 that its wavefronts hold.  Whole forward of gated experts of 8, us, as two launches / one, d_h = 512: 2048 experts, d = 2048,
// 1300 tokens 169.0 / 170.5, 1500 222 / 217, 2500 329 / 326, 4096 440 / 420, 9000 1043 / 1010; 1900 experts 1500 tokens 200 / 206, 1700 220 / 214,
// 2500 306 / 307; 1300 experts 1700 tokens 177 / 183, 2300 226 / 232, 2600 253 / 249; 1025 experts, d = 1280, 1500 tokens 115 / 122, 2500 165 / 167,
// 2700 173 / 170; 1024 experts 1500 tokens 108 / 109, 2000 133 / 134, 2300 158 / 152, 4096 202 / 195; 640 experts, d = 2048, 2000 tokens 132 / 134,
// 4096 188 / 186.  d_h = 256: 2048 experts, d = 2304, 1500 tokens 231 / 228, 4096 533 / 514.
bool scores_gate_supported(const dmoe_layer& L, int T) {
    const int E = L.n_experts;
    return router_sliced(L) && E > 512 && E <= 2048 && T >= (E <= 1024 ? 2300 : E <= 1792 ? 2600 : 1500) && gate_counts_supported(T, E);
}

template <int KS2>
static void launch_scores_gate_t(const dmoe_layer& L, int T, const __bf16* hid, float* scores, float tau, uint64_t* mask, int32_t* cnt,
                                 bool sets, hipStream_t s) {
    const __bf16* r2f = (const __bf16*)(static_cast<const char*>(L.packed) + packed_layout(L).r2f);
    auto go = [&](auto kernel) {
        launch_kernel(kernel, div_up(T, 16), 512, 0, s, hid, r2f, (const __bf16*)L.r_b2, scores, T, L.n_experts, tau, mask, cnt, sets ? 1 : 0);
    };
    if (L.n_experts <= 1024) go(scores_gate_kernel<KS2, 8>);
    else go(scores_gate_kernel<KS2, 16>);
}

void launch_router_gate_sliced(const dmoe_layer& L, const void* x, int T, void* hid, float* scores, float tau, uint64_t* mask,
                               int32_t* cnt, bool sets, hipStream_t s) {
    LaunchTimer tm(kSlotRouter, s);
    launch_router_hidden(L, x, T, hid, nullptr, s);
    if (L.router_hidden == 256) launch_scores_gate_t<8>(L, T, (const __bf16*)hid, scores, tau, mask, cnt, sets, s);
    else launch_scores_gate_t<16>(L, T, (const __bf16*)hid, scores, tau, mask, cnt, sets, s);
}

void launch_router_sliced(const dmoe_layer& L, const void* x, int T, void* hid, float* scores,
                          hipStream_t s) {
    LaunchTimer tm(kSlotRouter, s);
    const PackedLayout P = packed_layout(L);
    const int dh = L.router_hidden;
    launch_router_hidden(L, x, T, hid, nullptr, s);
    if (dh == 256) launch_scores_slices<16>(L, P, T, (const __bf16*)hid, scores, s);
    else launch_scores_slices<32>(L, P, T, (const __bf16*)hid, scores, s);
}

int router_fused_split(const dmoe_layer&, int T) {
    // measured (router alone, 1 / 2 / 4 workgroups per group): 4096 tokens, d = 2048, d_h = 256:
    // 39 / 31 / 28 us; the same with d_h = 512 and 2048 experts: 101 / 72 / 67 us; 16384 tokens,
    // d = 768: 21 / 21 / 26 us
    const int NG = div_up(T, kGroup);
    return NG >= 192 ? 1 : (NG >= 96 ? 2 : 4);
}

void launch_router_fused(const dmoe_layer& L, const void* x, int T, int split, float* scores,
                         float tau, uint64_t* mask, int32_t* group_cnt, bool sets, hipStream_t s) {
    LaunchTimer tm(kSlotRouter, s);
    switch (L.router_hidden) {
    case 64: launch_t<4>(L, x, T, split, scores, tau, mask, group_cnt, sets, s); break;
    case 128: launch_t<8>(L, x, T, split, scores, tau, mask, group_cnt, sets, s); break;
    case 256: launch_t<16>(L, x, T, split, scores, tau, mask, group_cnt, sets, s); break;
    case 512: launch_t<32>(L, x, T, split, scores, tau, mask, group_cnt, sets, s); break;
    default: break;  // refused by router_fused_supported
    }
}

}  // namespace dmoe
