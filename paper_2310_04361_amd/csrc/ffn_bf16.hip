// bf16 expert up-projection (+ gate) and activation (Sec. 3.2, Appendix G) on the gfx950 matrix
// cores, and the one-time packing of the expert and router weights.
//
//   up    expert-major grouped GEMM over the compact lists.  A wavefront owns UR = 16*TT list
//         rows of one expert, gathers those rows of x in 128-byte pieces (eight lanes per row, so
//         the vector memory path sees whole cache lines), stages them in its own LDS buffers and
//         multiplies them with the expert's up (and gate) rows; bias + activation in fp32; the
//         hidden activations go out rounded to bf16, one row of m_pad values per list row.
// Tokens ride on the MFMA column axis, so four consecutive neurons of one token land in one lane.
//
// Fragment order.  Every weight operand that a wavefront reads with one load instruction is
// stored as the 1 KiB block  [lane 0..63][8 bf16]  in exactly the register layout of the MFMA,
// because a 16-byte-per-lane access with a 64-byte or larger lane stride costs a cache-line
// lookup per lane and that, not bandwidth, bounded the first version of these kernels.
//   H row (m_pad bf16): natural neuron order -- the packed up weights place the neurons on the
//     MFMA rows (neuron_of_slot in mfma.h) so that the accumulators of lane (q, .) for the tile
//     pair (2ks, 2ks+1) are the eight consecutive neurons of the 16-byte piece 4ks + q.
//   An expert's H rows start at a multiple of UR rows (its first up-projection work item).
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "pack.h"
#include "token_sets.h"

namespace dmoe {

namespace {

constexpr int kUpRowBytes = 144;               // 64 bf16 of one x row + 16 bytes of bank skew

// ---- one-time weight packing ------------------------------------------------------------------------
// Scales of 8-bit weights -> the nearest power of two (in log2; the sign is kept, zero stays
// zero): with such a scale scale * e4m3(byte) is exactly a bf16 number, which is what makes the
// bf16 copies of the prefill kernels and the in-register conversion of the small-token kernels
// the same layer.
__global__ void snap_scales_kernel(const float* __restrict__ in, float* __restrict__ out, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float v = in[i], a = fabsf(v);
    float r = 0.0f;
    if (a > 0.0f && a < INFINITY) r = copysignf(exp2f(rintf(log2f(a))), v);
    out[i] = r;
}

// (small-token path) w_down[E][m][d] -> w2f[E][d/16][KS][64][8]: lane (q, c) of fragment (e, column tile ct, ks)
// holds W_down[e][8*(4ks + q) + s][16ct + c] (piece 4ks + q of an H row), zero for neurons >= m.
// OUT = __bf16: the weight as a bf16 number (8-bit weights are scaled out); OUT = uint8_t: the
// raw E4M3 byte (8-bit weights only), for the kernels that convert in registers.
struct SmallDownMap {
    static constexpr int kCols = 16;
    int KS, blocks;  // blocks: E * KS
    __device__ void row(int b, int q, int s, int& e, int& neuron) const {
        e = b / KS;
        neuron = 8 * (4 * (b % KS) + q) + s;
    }
    static __device__ int lane(int col) { return col; }
    __device__ size_t block(int b, int ct, int n_ct) const { return ((size_t)(b / KS) * n_ct + ct) * KS + b % KS; }
};

// w[E][m][d] -> wf[E][MT][d/32][64][8]: lane (q, c) of fragment (e, neuron tile mt, k-step) holds
// w[e][n(mt, c)][32 kstep + 8q + s], zero rows for neurons >= m; n(mt, c) = neuron_of_slot for the
// expert matrices (whose order makes H pieces consecutive), 16mt + c for the router matrices.
// `which`: 0 up, 1 gate (selects the scale of 8-bit weights).  A thread fills a lane's eight values; the 64 of a
// fragment read 64 bytes of each of its 16 rows.
template <typename OUT>
__global__ void pack_up_kernel(const void* __restrict__ w, const float* __restrict__ scales, int fp8,
                               int which, OUT* __restrict__ wf, int E, int m, int d, int MT,
                               int piece_order) {
    typedef typename Packed8<OUT>::type Vec;
    const size_t n = (size_t)E * MT * 2 * d;
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) {
        const int q = (int)(i & 3), c = (int)((i >> 2) & 15);
        const size_t block = i >> 6;
        size_t f = block;
        const int kstep = (int)(f % (d / 32));
        f /= (d / 32);
        const int mt = (int)(f % MT), e = (int)(f / MT);
        const int neuron = piece_order ? neuron_of_slot(mt, c) : 16 * mt + c;
        const Vec v = neuron < m ? Packed8<OUT>::load(w, scales, fp8, which, e, ((size_t)e * m + neuron) * d + 32 * kstep + 8 * q)
                                 : Vec{};
        *reinterpret_cast<Vec*>(wf + (block * 64 + 16 * q + c) * 8) = v;
    }
}

// Experts of one weight tile: w_up (, w_gate) [E][m][d] -> wt[E][d/32][64][8], one 16-row tile per
// expert and k-step.  Gated (m <= 8): rows 0..7 are the up rows and 8..15 the gate rows; plain
// (m <= 16): row c is neuron c.  Zero rows for neurons >= m; lane (q, c) holds row c, columns
// 32 kstep + 8q + s.
__global__ void pack_up_tiny_kernel(const void* __restrict__ w_up, const void* __restrict__ w_gate,
                                    const float* __restrict__ scales, int fp8,
                                    __bf16* __restrict__ wt, int E, int m, int d, int gated) {
    const size_t n = (size_t)E * 2 * d;
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) {
        const int q = (int)(i & 3), c = (int)((i >> 2) & 15);
        const size_t block = i >> 6;
        const int kstep = (int)(block % (d / 32)), e = (int)(block / (d / 32));
        const int neuron = gated ? (c & 7) : c, which = gated ? (c >> 3) : 0;  // 0 up, 1 gate
        const bf16x8 v = neuron < m ? Packed8<__bf16>::load(which ? w_gate : w_up, scales, fp8, which, e,
                                                            ((size_t)e * m + neuron) * d + 32 * kstep + 8 * q)
                                    : zero8();
        *reinterpret_cast<bf16x8*>(wt + (block * 64 + 16 * q + c) * 8) = v;
    }
}

// ---- up-projection ---------------------------------------------------------------------------------
// Which of an XCD's n_waves wavefronts this one is: neighbouring items (one expert's, as a rule) go to
// one workgroup, whose wavefronts then find its weights in their L1, unless there are too few items
// for that: then every CU gets one before any gets two.
__device__ __forceinline__ int wave_of(int n_items, int wave_in_block, int n_waves) {
    const int wg = (int)(blockIdx.x >> 3);
    return n_items > n_waves ? wg * 4 + wave_in_block : wave_in_block * (n_waves >> 2) + wg;
}

// The rows of x that a lane of the narrow kernels gathers.  NEAR: x is smaller than 2 GiB, a row is a 32-bit offset
// into a buffer and a padding row (-1) an offset beyond it, which moves no data.  Otherwise 16-byte units from
// x, and padding rows read token 0.  Either way they produce H rows that nobody merges.
constexpr int kRawBuffer = 0x00020000;  // offsets from num_records on read as zero and move no data
typedef __attribute__((address_space(3))) void* LdsPtr;
// 16 bytes a lane straight to 1 KB of LDS
__device__ __forceinline__ void buffer_to_lds(__amdgpu_buffer_rsrc_t buf, uint32_t lane_off, uint32_t off, char* lds) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(buf, (LdsPtr)lds, 16, lane_off, off, 0, 0);
}
template <bool NEAR>
struct XRows {
    __amdgpu_buffer_rsrc_t buf;
    const __bf16* x;
    int d;
    __device__ __forceinline__ XRows(const __bf16* x_, int d_) : x(x_), d(d_) {
        buf = __builtin_amdgcn_make_buffer_rsrc((void*)x_, 0, 0x7fffffff, kRawBuffer);
    }
    // piece: 16-byte piece of the first 128 bytes
    __device__ __forceinline__ uint32_t row(int tok, int piece) const {
        if (NEAR) return tok < 0 ? 0x80000000u : (uint32_t)tok * (uint32_t)(2 * d) + 16u * (uint32_t)piece;
        return (uint32_t)(((size_t)max(tok, 0) * d) >> 3) + (uint32_t)piece;
    }
    // K block kb of 64 columns, 16 bytes a lane, to 1 KB of LDS
    __device__ __forceinline__ void to_lds(uint32_t row, int kb, char* lds) const {
        if (NEAR) buffer_to_lds(buf, row, 128 * kb, lds);
        else __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(x + (((size_t)row + 8 * kb) << 3)), (LdsPtr)lds, 16, 0, 0);
    }
    __device__ __forceinline__ bf16x8 load(uint32_t row, int kb) const {  // K block kb of 64 columns
        if (NEAR) return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(buf, row, 128 * kb, 0));
        return load8(x + (((size_t)row + 8 * kb) << 3));
    }
};

// One wavefront per work item = (expert, UR = 16*TT consecutive list rows); no workgroup-level
// synchronisation after the work-item table has been staged.  MT = m_pad / 16 neuron tiles per
// branch.  K advances in blocks of 64: the wavefront loads the next block of its x rows
// (lane = (row % 8, 16-byte piece of the 128-byte row segment)) and of the weight fragments
// while the MFMAs run on the current block out of LDS / registers.
// PTR: the weights by address and all lanes, with as many registers as one wavefront per SIMD may have.
// SETS: a small batch, whose items come from the token sets (token_sets.h) instead of the lists.
template <int MT, bool GATED, int TT, int NBUF, bool NEAR, bool PTR = false, bool SETS = false>
__global__ __launch_bounds__(256, NBUF == 1 ? 3 : (SETS ? 2 : 1)) void up_bf16_kernel(
    const __bf16* __restrict__ x, const __bf16* __restrict__ wupf,
    const __bf16* __restrict__ wgatef, const __bf16* __restrict__ b_up,
    const int32_t* __restrict__ witem, const int32_t* __restrict__ wfirst, int NW,
    const int32_t* __restrict__ alist, __bf16* __restrict__ Hf, int d, int E, int m, int act, const SetsArg<SETS> S) {
    constexpr int BR = GATED ? 2 : 1;
    constexpr int KS = MT / 2;
    constexpr int UR = TT * 16;
    constexpr int NL = TT * 2;  // x load instructions per K block: 8 rows x 128 bytes each
    static_assert(!SETS || UR == 64, "a wavefront's list of rows");
    extern __shared__ char smem[];
    int32_t* s_wit = reinterpret_cast<int32_t*>(smem);  // witem[w][0..E], then wfirst[w][0..E-1]
    int32_t* s_wf = s_wit + (E + 1);
    const int items_bytes = SETS ? 4 * 64 * 4 : ((2 * E + 1) * 4 + 15) & ~15;
    const int lane = threadIdx.x & 63, q = lane >> 4, c = lane & 15;
    const int wave_in_block = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int32_t* s_list = s_wit + 64 * wave_in_block;  // SETS: the rows of this wavefront's item
    char* xs = smem + items_bytes + wave_in_block * (NBUF * UR * kUpRowBytes);
    const int NK32 = d / 32, NKB = d / 64;
    const int ld_row = lane >> 3, ld_piece = lane & 7;

    // Work items are walked window by window: the wavefronts of XCD k (workgroups are dealt
    // round-robin to the 8 XCDs; the grid is a multiple of 8) take the windows k, k+8, ... so that the
    // x rows they gather -- each row is used by every expert its token selected -- stay in that XCD's
    // L2; gathered out of the last-level cache the same rows come in at about a third of the rate.
    // Of fewer than eight windows each belongs to several XCDs, which share its items: neighbouring
    // experts on one XCD.
    const int xcd = blockIdx.x & 7, shares = NW < 8 ? 8 / NW : 1, share = xcd % shares;
    for (int wdx = SETS ? 0 : xcd / shares; wdx < (SETS ? 1 : NW); wdx += 8) {
    if (!SETS) {
        __syncthreads();  // the previous window's table is no longer read
        for (int i = threadIdx.x; i <= 2 * E; i += blockDim.x)
            s_wit[i] = i <= E ? witem[(size_t)wdx * (E + 1) + i] : wfirst[(size_t)wdx * E + (i - E - 1)];
        __syncthreads();
    }
    const long long all = SETS ? 0 : s_wit[E];
    const int first = (int)(all * share / shares), total = (int)(all * (share + 1) / shares);
    const int n_waves = (int)(gridDim.x >> 3) * 4, wave = wave_of(total - first, wave_in_block, n_waves);
    // item jj: its expert is the last e with s_wit[e] <= jj
    auto locate = [&](int jj, int& e, int& item) {
        int lo = 0, hi = E;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (s_wit[mid] <= jj) lo = mid; else hi = mid;
        }
        e = lo;
        item = s_wf[lo] + (jj - s_wit[lo]);
    };
    int j = first + wave;
    SetItem si;  // SETS: the only one
    bool work = j < total;
    if constexpr (SETS) work = si.start(S, E, wave_in_block, UR);
    if (work) {
        int e, item;
        if (SETS) {
            e = si.e;
            item = si.index;
        } else {
            locate(j, e, item);
        }
        // the item's rows that this lane gathers
        auto tokens_of = [&](int it, int (&tok)[NL]) {
            if (SETS) si.tok.list<64, 64>(UR * si.item, s_list, [](int r) { return r; });
            const int32_t* tl = (SETS ? s_list : alist + (size_t)it * UR) + ld_row;
#pragma unroll
            for (int i = 0; i < NL; ++i) tok[i] = tl[8 * i];
        };
        // Rows of the aligned list past the expert's last token hold -1.
        const XRows<NEAR> xrows(x, d);
        uint32_t xoff[NL];
        auto rows_from = [&](const int (&tok)[NL]) {
#pragma unroll
            for (int i = 0; i < NL; ++i)
                xoff[i] = xrows.row(tok[i], ld_piece);
        };
        // The fragments of a 16-neuron tile, without the lanes whose row is padding: experts of 24 neurons in tiles
        // of 32 fetch three quarters of the bytes.  (With the 32-bit rows of x, which save the address
        // arithmetic and the spills: 50432 tokens x 128 experts of 24, d = 768, 117 -> 110 us, 2000 tokens 13.7 -> 12.4;
        // neither does it alone.)
        __amdgpu_buffer_rsrc_t wf[BR];
        const __bf16* wp[BR];
        uint32_t wlane[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
            wlane[mt] = neuron_of_slot(mt, c) < m ? (uint32_t)(mt * NK32 * 1024 + lane * 16) : 0x80000000u;
        auto weights_of = [&](int ee) {
            if constexpr (PTR) {
                wp[0] = wupf + (size_t)ee * MT * NK32 * 512 + lane * 8;
                if (GATED) wp[BR - 1] = wgatef + (size_t)ee * MT * NK32 * 512 + lane * 8;
                return;
            }
            const size_t at = (size_t)__builtin_amdgcn_readfirstlane(ee) * MT * NK32 * 512;
            wf[0] = __builtin_amdgcn_make_buffer_rsrc((void*)(wupf + at), 0, MT * NK32 * 1024, kRawBuffer);
            if (GATED) wf[BR - 1] = __builtin_amdgcn_make_buffer_rsrc((void*)(wgatef + at), 0, MT * NK32 * 1024, kRawBuffer);
        };
        {
            int tok[NL];
            tokens_of(item, tok);
            rows_from(tok);
        }
        weights_of(e);

        bf16x8 xr[NL];
        bf16x8 a0[2][BR][MT], a1[2][BR][MT];
        auto load_x = [&](int kb) {
#pragma unroll
            for (int i = 0; i < NL; ++i) xr[i] = xrows.load(xoff[i], kb);
        };
        auto load_a = [&](int kb, bf16x8 (&a)[2][BR][MT]) {
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int br = 0; br < BR; ++br)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
                        a[ks][br][mt] = PTR ? load8(wp[br] + ((size_t)mt * NK32 + 2 * kb + ks) * 512)
                                            : __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(wf[br], wlane[mt], (2 * kb + ks) * 1024, 0));
        };
        auto store_x = [&](int buf) {
            char* dst = xs + (buf % NBUF) * (UR * kUpRowBytes) + ld_row * kUpRowBytes + ld_piece * 16;
#pragma unroll
            for (int i = 0; i < NL; ++i)
                *reinterpret_cast<bf16x8*>(dst + 8 * i * kUpRowBytes) = xr[i];
        };
        // The first block of an item is requested before the epilogue of the item before it (here:
        // before anything else), so an item starts with its block 0 on the way.
        load_x(0);
        load_a(0, a0);
        for (;;) {
            // the accumulators start at the biases of this lane's neurons (no registers held for
            // them through the K loop)
            f32x4 acc[BR][MT][TT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                f32x4 bias = f32x4{0.f, 0.f, 0.f, 0.f};
                if (!GATED && b_up) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int n = neuron_of_slot(mt, 4 * q + r);
                        bias[r] = (float)b_up[(size_t)e * m + min(n, m - 1)];
                    }
                }
#pragma unroll
                for (int br = 0; br < BR; ++br)
#pragma unroll
                    for (int tt = 0; tt < TT; ++tt) acc[br][mt][tt] = br == 0 ? bias : f32x4{0.f, 0.f, 0.f, 0.f};
            }
            auto compute = [&](int buf, const bf16x8 (&a)[2][BR][MT]) {
                const char* src = xs + (buf % NBUF) * (UR * kUpRowBytes) + c * kUpRowBytes + q * 16;
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {
                    bf16x8 b[TT];
#pragma unroll
                    for (int tt = 0; tt < TT; ++tt)
                        b[tt] = *reinterpret_cast<const bf16x8*>(src + tt * 16 * kUpRowBytes + ks * 64);
#pragma unroll
                    for (int br = 0; br < BR; ++br)
#pragma unroll
                        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                            for (int tt = 0; tt < TT; ++tt)
                                acc[br][mt][tt] = mfma16(a[ks][br][mt], b[tt], acc[br][mt][tt]);
                }
            };

            store_x(0);
            // two K blocks per trip so that the two weight-fragment register sets simply alternate
            for (int kb = 0; kb < NKB - 2; kb += 2) {
                load_x(kb + 1);
                load_a(kb + 1, a1);
                compute(0, a0);
                store_x(1);
                load_x(kb + 2);
                load_a(kb + 2, a0);
                compute(1, a1);
                store_x(0);
            }
            // Last trip: its second set of requests is block 0 of the wavefront's NEXT item (the
            // last item names itself: the block is read and never used), whose list rows are
            // requested together with this item's last block, once its own offsets are done with.
            // (SETS: there is no next one.)
            load_x(NKB - 1);
            load_a(NKB - 1, a1);
            const int jn = j + n_waves;
            const bool more = !SETS && jn < total;
            int en = e, itemn = item;
            if (more) locate(jn, en, itemn);
            int tokn[NL];
            if (!SETS) tokens_of(itemn, tokn);
            compute(0, a0);
            store_x(1);
            if (!SETS) {
                rows_from(tokn);
                weights_of(en);
                load_x(0);
                load_a(0, a0);
            }
            compute(1, a1);

            // lane (q, c) of tile (mt, tt): neurons 16mt + 4q + r of list row 16tt + c
            with_activation(act, [&](auto act_c) {
                constexpr int ACT = decltype(act_c)::value;
#pragma unroll
                for (int tt = 0; tt < TT; ++tt) {
                    __bf16* dst = Hf + ((size_t)item * UR + 16 * tt + c) * (KS * 32) + 8 * q;
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) {
                        bf16x8 hv;
#pragma unroll
                        for (int half = 0; half < 2; ++half) {
                            const int mt = 2 * ks + half;
                            const int n0 = neuron_of_slot(mt, 4 * q);  // + r: consecutive
#pragma unroll
                            for (int r = 0; r < 4; ++r) {
                                float v;
                                if (GATED) {
                                    v = activate_fast(ACT, acc[BR - 1][mt][tt][r]) * acc[0][mt][tt][r];
                                } else {
                                    v = activate_fast(ACT, acc[0][mt][tt][r]);
                                }
                                if (n0 + r >= m) v = 0.0f;
                                hv[half * 4 + r] = (__bf16)v;
                            }
                        }
                        *reinterpret_cast<bf16x8*>(dst + ks * 32) = hv;
                        __builtin_amdgcn_sched_barrier(0);  // eight values at a time
                    }
                }
            });
            if (!more) break;
            j = jn;
            e = en;
            item = itemn;
        }
    }
    }  // windows
}

// Up-projection for experts that fit one 16-row weight tile: at most 16 neurons, or gated with at
// most 8 (the paper's own splits: experts of 6 for its text classifier, 2048 gated experts of 8
// for its language model).  In the general kernel a gated expert of 8 fills a quarter of the rows
// of four weight tiles and a plain one of 6 to 16 half of two; here the expert is ONE tile (gated:
// up rows and gate rows together), so a work item streams a quarter / half of the weight bytes
// and issues a quarter / half of the MFMAs, and what remains is the gather of the x rows.  Same
// work items and x staging as up_bf16_kernel<2, GATED, TT>; the H rows hold only the expert's pieces
// (h_row_neurons).
template <int TT, bool GATED, bool NEAR, bool SETS>
__global__ __launch_bounds__(256) void up_tiny_kernel(
    const __bf16* __restrict__ x, const __bf16* __restrict__ wtf, const __bf16* __restrict__ b_up,
    const int32_t* __restrict__ witem, const int32_t* __restrict__ wfirst, int NW,
    const int32_t* __restrict__ alist, __bf16* __restrict__ Hf, int d, int E, int m, int act, int row_neurons, const SetsArg<SETS> S) {
    constexpr int UR = TT * 16;
    constexpr int NL = TT * 2;
    extern __shared__ char smem[];
    int32_t* s_wit = reinterpret_cast<int32_t*>(smem);  // witem[w][0..E-1], then wfirst[w][0..E-1]
    int32_t* s_wf = s_wit + E;
    const int items_bytes = SETS ? 4 * 64 * 4 : (2 * E * 4 + 15) & ~15;
    const int lane = threadIdx.x & 63, q = lane >> 4, c = lane & 15;
    const int wave_in_block = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int32_t* s_list = s_wit + 64 * wave_in_block;  // SETS: the rows of this wavefront's item
    static_assert(!SETS || UR == 64, "a wavefront's list of rows");
    // one staging buffer per wavefront (its LDS accesses keep their order, so a second one buys
    // nothing): with thousands of experts the work-item table already takes 16 KiB or more, and
    // the LDS left decides how many wavefronts a CU holds
    char* xs = smem + items_bytes + wave_in_block * (UR * kUpRowBytes);
    const int NK32 = d / 32, NKB = d / 64;
    const int ld_row = lane >> 3, ld_piece = lane & 7;

    // (who works on what: see up_bf16_kernel)
    const int xcd = blockIdx.x & 7, shares = NW < 8 ? 8 / NW : 1, share = xcd % shares;
    for (int wdx = SETS ? 0 : xcd / shares; wdx < (SETS ? 1 : NW); wdx += 8) {
    if (!SETS) {
        __syncthreads();  // the previous window's table is no longer read
        for (int i = threadIdx.x; i < 2 * E; i += blockDim.x)
            s_wit[i] = i < E ? witem[(size_t)wdx * (E + 1) + i] : wfirst[(size_t)wdx * E + (i - E)];
    }
    const long long all = SETS ? 0 : witem[(size_t)wdx * (E + 1) + E];
    const int first = (int)(all * share / shares), total = (int)(all * (share + 1) / shares);
    const int n_waves = (int)(gridDim.x >> 3) * 4, wave = wave_of(total - first, wave_in_block, n_waves);
    if (!SETS) __syncthreads();
    SetItem si;  // SETS: the only one
    bool work = first + wave < total;
    if constexpr (SETS) work = si.start(S, E, wave_in_block, UR);
    for (int j = first + wave; work; j += n_waves, work = !SETS && j < total) {
        int e, item;
        if (SETS) {
            e = si.e;
            item = si.index;
            si.tok.list<64, 64>(UR * si.item, s_list, [](int r) { return r; });
        } else {
            int lo = 0, hi = E;  // last e with s_wit[e] <= j
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (s_wit[mid] <= j) lo = mid; else hi = mid;
            }
            e = lo;
            item = s_wf[e] + (j - s_wit[e]);
        }
        const int32_t* tl = (SETS ? s_list : alist + (size_t)item * UR) + ld_row;
        // Valid rows are a prefix of the item and padding rows hold -1.  With thousands of experts
        // most items are part-filled (4096 tokens, 2048 experts, 7 % density: 36 of 64 rows), and
        // what the kernel spends is load instructions: a load whose eight rows are all padding is
        // not issued (`need` has a bit per load instruction; its staging rows are zeroed once).
        const XRows<NEAR> xrows(x, d);
        uint32_t xoff[NL];
        uint32_t need = 0;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int tok = tl[8 * i];
            need |= (__ballot(tok >= 0) != 0 ? 1u : 0u) << i;
            xoff[i] = xrows.row(tok, ld_piece);
        }
        need = __builtin_amdgcn_readfirstlane(need);
        // (SETS: most items of thousands of experts have few rows, so the way without the loads is laid out straight: 130 tokens x 2048
        // gated experts of 8, d = 2048, whole forward 78.0 -> 77.3 us)
        // (without the lanes whose row of the tile is padding: 16384 tokens x 512 experts of 6, d = 768, 94.5 -> 86.4 us)
        const __amdgpu_buffer_rsrc_t wf = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(wtf + (size_t)__builtin_amdgcn_readfirstlane(e) * NK32 * 512), 0, NK32 * 1024, kRawBuffer);
        const uint32_t wlane = (GATED ? (c & 7) : c) < m ? (uint32_t)(lane * 16) : 0x80000000u;

        f32x4 acc[TT];
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) acc[tt] = f32x4{0.f, 0.f, 0.f, 0.f};

        bf16x8 xr[NL];
        bf16x8 a0[2], a1[2];
        auto load_x = [&](int kb) {
#pragma unroll
            for (int i = 0; i < NL; ++i)
                if (SETS ? __builtin_expect((need >> i) & 1u, 0) : (need >> i) & 1u) xr[i] = xrows.load(xoff[i], kb);
        };
        auto load_a = [&](int kb, bf16x8 (&a)[2]) {
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
                a[ks] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(wf, wlane, (2 * kb + ks) * 1024, 0));
        };
        auto store_x = [&]() {
            char* dst = xs + ld_row * kUpRowBytes + ld_piece * 16;
#pragma unroll
            for (int i = 0; i < NL; ++i)
                if (SETS ? __builtin_expect((need >> i) & 1u, 0) : (need >> i) & 1u) *reinterpret_cast<bf16x8*>(dst + 8 * i * kUpRowBytes) = xr[i];
        };
        {   // rows that no load fills: zeros for the whole item
            char* dst = xs + ld_row * kUpRowBytes + ld_piece * 16;
            const bf16x8 zero = {};
#pragma unroll
            for (int i = 0; i < NL; ++i)
                if (!((need >> i) & 1u)) *reinterpret_cast<bf16x8*>(dst + 8 * i * kUpRowBytes) = zero;
        }
        auto compute = [&](const bf16x8 (&a)[2]) {
            const char* src = xs + c * kUpRowBytes + q * 16;
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int tt = 0; tt < TT; ++tt) {
                    const bf16x8 b =
                        *reinterpret_cast<const bf16x8*>(src + tt * 16 * kUpRowBytes + ks * 64);
                    acc[tt] = mfma16(a[ks], b, acc[tt]);
                }
        };

        load_x(0);
        load_a(0, a0);
        store_x();
        for (int kb = 0; kb < NKB; kb += 2) {
            load_x(kb + 1);
            load_a(kb + 1, a1);
            compute(a0);
            store_x();
            const int nb = min(kb + 2, NKB - 1);  // the last trip re-reads a block it will not use
            load_x(nb);
            load_a(nb, a0);
            compute(a1);
            store_x();
        }

        // lane (q, c) of token tile tt holds tile rows 4q + r of list row 16tt + c.
        // Gated: q = 0, 1 the up products of neurons 4q + r, q = 2, 3 the gate products of
        // neurons 4(q - 2) + r.  Plain: neuron 4q + r (plus its bias).
        float bias[4] = {0.f, 0.f, 0.f, 0.f};
        if (!GATED && b_up) {
#pragma unroll
            for (int r = 0; r < 4; ++r) bias[r] = (float)b_up[(size_t)e * m + min(4 * q + r, m - 1)];
        }
        with_activation(act, [&](auto act_c) {
        constexpr int ACT = decltype(act_c)::value;
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
            float v[4], w[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                if (GATED) {
                    const float other = __shfl_xor(acc[tt][r], 32, 64);  // q <-> q ^ 2
                    const float up = q < 2 ? acc[tt][r] : other;
                    const float gate = q < 2 ? other : acc[tt][r];
                    v[r] = activate_fast(ACT, gate) * up;
                    if (4 * (q & 1) + r >= m) v[r] = 0.0f;
                } else {
                    v[r] = activate_fast(ACT, acc[tt][r] + bias[r]);
                    if (4 * q + r >= m) v[r] = 0.0f;
                }
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) w[r] = __shfl_xor(v[r], 16, 64);  // the other half of a piece
            // piece p of the H row = neurons 8p .. 8p+7.  Gated: lane q = 0 has piece 0.  Plain: lane q = 0 has
            // piece 0, q = 2 piece 1.  The others have zeros for the rest of a padded row.
            const bool real = GATED ? q == 0 : (q & 1) == 0;
            const int piece = GATED ? q : (real ? (q >> 1) : 2 + (q >> 1));
            bf16x8 hv;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                hv[r] = (__bf16)(real ? v[r] : 0.0f);
                hv[4 + r] = (__bf16)(real ? w[r] : 0.0f);
            }
            if (8 * piece < row_neurons)
                *reinterpret_cast<bf16x8*>(Hf + ((size_t)item * UR + 16 * tt + c) * row_neurons + 8 * piece) = hv;
        }
        });
    }
    }  // windows
}

// Up-projection for wide experts (8 neuron tiles per K step: gated m = 64; plain m = 128 where x does not allow for
// up_wide_plain_kernel): there the
// weights of an expert are as large as its x rows, so streaming them once per wavefront made the
// kernel a weight stream.  Here a workgroup of four wavefronts owns 4 x 16*TT consecutive list
// rows of one expert and shares each K block of the weight fragments through LDS (double
// buffered, one barrier per block); the x rows stay private to their wavefront as above.
//
// The K blocks of all the items of a workgroup form one stream: while block k is multiplied,
// block k+1 is moved from registers to LDS and the loads of block k+2 are issued -- also
// across the end of an item, so that the first blocks of the next item arrive during the
// activation epilogue of the current one instead of after it (an item is only 12 to 32 blocks
// long, and a round trip beyond L2 takes as long as two or three blocks).  Each register is reloaded
// as soon as its LDS write is issued, between two MFMAs: requests are in flight all the time, and
// neither the writes nor the issue of the loads wait for the end of the block.  (As three phases in
// sequence -- multiply; write; barrier, then request -- 4096 tokens x 256 gated experts of 64, d = 2048, 37 % density
// took 222 us against 197, 333 tokens 53 against 45.)
//
// The order of the items (select.hip) keeps the traffic beyond L2 down: 4096 tokens x 256 gated
// experts of 64, d = 2048, 37 % density: 1.84 -> 0.82 GB from beyond L2 and, with the 32x32x16 MFMA (half
// the instructions of the 16x16x32 one), 276 -> 240 us, both on one card in turn (224 to 253 over
// cards and clocks), before the interleaving above, which lets the workgroups of an XCD drift apart: 0.97 to 1.00 GB since.  Built and
// slower: x rows by LDS-DMA and the weights straight to registers, with a 2 x 2 split over the
// wavefronts (236 us against 220 on the card of that day: LDS instructions down to a sixth, but more bytes and more
// drift between the workgroups, 0.96 GB); rows and weights straight to LDS, one block ahead (up_wide_plain_kernel, below): 420 -> 414 us
// for a whole forward, but 450 -> 473 for the first one on new weights, whose way from HBM is longer than a block; one workgroup
// of 512 rows per CU that way, four blocks of weights ahead, which halves what comes from beyond L2: 412, but 1400 tokens
// 166 -> 186, as nothing works beside a workgroup's epilogue and tail.
template <int MT, bool GATED, int TT>
__global__ __launch_bounds__(256, 2) void up_wide_bf16_kernel(
    const __bf16* __restrict__ x, const __bf16* __restrict__ wupf,
    const __bf16* __restrict__ wgatef, const __bf16* __restrict__ b_up,
    const int32_t* __restrict__ witem, const int2* __restrict__ worder,
    const int32_t* __restrict__ alist, __bf16* __restrict__ Hf, int d, int E, int m, int act) {
    constexpr int BR = GATED ? 2 : 1;
    constexpr int KS = MT / 2;
    constexpr int NT = BR * MT;         // neuron tiles per K step
    constexpr int NJ = NT / 2, TJ = TT / 2;  // tiles of the 32x32x16 MFMA: neurons, list rows
    constexpr int WR = TT * 16;         // rows per wavefront
    constexpr int UR = 4 * WR;          // rows per work item
    constexpr int NL = TT * 2;          // x load instructions per K block
    constexpr int NWF = 2 * NT;         // weight fragments (1 KiB each) per K block
    constexpr int NWL = NWF / 4;        // ... of which each wavefront copies every fourth
    static_assert(NWF % 4 == 0 && MT % 2 == 0, "weight fragments are copied four at a time");
    extern __shared__ char smem[];
    char* wbuf = smem;                                   // [2][NWF][1024]
    const int lane = threadIdx.x & 63, h = lane >> 5, c32 = lane & 31, w = threadIdx.x >> 6;
    char* xs = smem + 2 * NWF * 1024 + w * (WR * kUpRowBytes);   // [WR][kUpRowBytes], private
    float* sbias = reinterpret_cast<float*>(smem + 2 * NWF * 1024 + 4 * (WR * kUpRowBytes));  // [2][MT * 16]
    const int NK32 = d / 32, NKB = d / 64;   // NKB >= 2
    const int ld_row = lane >> 3, ld_piece = lane & 7;
    // this XCD's share of the items (workgroups are dealt round-robin to the 8 XCDs; the grid is a
    // multiple of 8), in the order laid out by the list fill
    const int xcd = blockIdx.x & 7, step = gridDim.x >> 3;
    const int total = xcd_first(witem[E], xcd + 1);
    const int first = xcd_first(witem[E], xcd);
    int j = first + (int)(blockIdx.x >> 3);
    if (j >= total) return;
    // (from the end: an expert's last item, often nearly empty, comes before its full ones, so that the
    // workgroups do not end with items of a wavefront or two)
    auto locate = [&](int jj, int& e, int& item) {
        const int2 v = worder[total - 1 - (jj - first)];
        e = v.x;
        item = v.y;
    };
    // tokens of the x rows this lane fetches; padding rows (-1) read token 0 and produce H rows
    // that nobody merges
    auto rows_of = [&](int item, uint32_t (&xoff)[NL], bool& active) {
        const int32_t* tl = alist + (size_t)item * UR + w * WR;
        active = tl[0] >= 0;  // valid rows are a prefix
#pragma unroll
        for (int i = 0; i < NL; ++i)
            xoff[i] = (uint32_t)max(tl[ld_row + 8 * i], 0);
    };
    // Weight fragment f = (br * MT + mt) * 2 + ks of a K block; this wavefront copies the
    // fragments f = 4 i + w: ks = w & 1, mt = (2 i) % MT + (w >> 1), br = (2 i) / MT.
    const uint32_t woff = (uint32_t)(((w >> 1) * NK32 + (w & 1)) * 512 + lane * 8);
    bf16x8 xr[NL], wr[NWL];
    auto issue_w = [&](int i, int e, int kb) {
        const __bf16* base = (GATED && (2 * i) / MT == BR - 1) ? wgatef : wupf;
        wr[i] = load8(base + (size_t)e * MT * NK32 * 512 + (size_t)kb * 1024 + woff + (size_t)((2 * i) % MT) * NK32 * 512);
    };
    auto issue_x = [&](int i, const uint32_t (&xoff)[NL], int kb) {
        xr[i] = load8(x + ((size_t)xoff[i] * (uint32_t)d + (uint32_t)(8 * ld_piece + 64 * kb)));
    };
    auto park_w = [&](int i, int buf) {
        *reinterpret_cast<bf16x8*>(wbuf + buf * NWF * 1024 + (4 * i + w) * 1024 + lane * 16) = wr[i];
    };
    auto park_x = [&](int i) {
        *reinterpret_cast<bf16x8*>(xs + (ld_row + 8 * i) * kUpRowBytes + ld_piece * 16) = xr[i];
    };
    auto park_bias = [&](int e, int par) {  // plain experts: the item's biases, by neuron
        if (!GATED && (int)threadIdx.x < MT * 16)
            sbias[par * MT * 16 + threadIdx.x] =
                b_up ? (float)b_up[(size_t)e * m + min((int)threadIdx.x, m - 1)] : 0.0f;
    };

    int e, item;
    uint32_t xoff[NL];
    bool active;
    locate(j, e, item);
    rows_of(item, xoff, active);
#pragma unroll
    for (int i = 0; i < NWL; ++i) issue_w(i, e, 0);
#pragma unroll
    for (int i = 0; i < NL; ++i) issue_x(i, xoff, 0);
#pragma unroll
    for (int i = 0; i < NWL; ++i) {
        park_w(i, 0);
        issue_w(i, e, 1);
    }
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        park_x(i);
        issue_x(i, xoff, 1);
    }
    park_bias(e, 0);
    lds_barrier();
    int buf = 0, par = 0;
    for (;;) {
        // the item after this one (the last item names itself: its first blocks are read again
        // and never used)
        const int jn = j + step;
        const bool more = jn < total;
        int en = e, itemn = item;
        if (more) locate(jn, en, itemn);

        f32x16 acc[NJ][TJ];
#pragma unroll
        for (int nj = 0; nj < NJ; ++nj)
#pragma unroll
            for (int tj = 0; tj < TJ; ++tj)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[nj][tj][r] = 0.f;
        // One K block: multiplies block k of this item (in LDS: weight buffer `buf`, x rows staged), parks
        // block k + 1 (requested a block ago) and requests block k + 2, which may be one of the next item (its
        // expert ew, rows xo, block kb2).  xp, xi: whether the rows of k + 1 and of k + 2 are wanted, where this
        // item's are not.
        auto block = [&](int ew, const uint32_t (&xo)[NL], int kb2, bool xp, bool xi) {
            if (active) {
                // operands of k-step s (16 wide): neuron tile nj from the fragments of its two
                // 16-row tiles, token tile tj from the staged rows; the next neuron tile's (and the
                // next k-step's) operands are read while the current tile's MFMAs run
                const char* wsrc_l = wbuf + buf * NWF * 1024 + (c32 >> 4) * 2048 + (h * 16 + (c32 & 15)) * 16;
                const char* xsrc = xs + c32 * kUpRowBytes + h * 16;
                auto read_a = [&](int s, int nj) {
                    return *reinterpret_cast<const bf16x8*>(wsrc_l + nj * 4096 + (s >> 1) * 1024 + (s & 1) * 512);
                };
                auto read_b = [&](int s, int tj) {
                    return *reinterpret_cast<const bf16x8*>(xsrc + tj * 32 * kUpRowBytes + s * 32);
                };
                bf16x8 b[2][TJ], a_next = read_a(0, 0);
#pragma unroll
                for (int tj = 0; tj < TJ; ++tj) b[0][tj] = read_b(0, tj);
#pragma unroll
                for (int s = 0; s < 4; ++s) {
#pragma unroll
                    for (int nj = 0; nj < NJ; ++nj) {
                        const int q = s * NJ + nj;
                        const bf16x8 a = a_next;
                        const int n1 = nj + 1 < NJ ? nj + 1 : 0, s1 = nj + 1 < NJ ? s : s + 1;
                        __builtin_amdgcn_sched_barrier(0);
                        if (s1 < 4) a_next = read_a(s1, n1);
                        if (nj == 0 && s + 1 < 4) {
#pragma unroll
                            for (int tj = 0; tj < TJ; ++tj) b[(s + 1) & 1][tj] = read_b(s + 1, tj);
                        }
#pragma unroll
                        for (int tj = 0; tj < TJ; ++tj) {
                            acc[nj][tj] = mfma32(a, b[s & 1][tj], acc[nj][tj]);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                        if (q >= 1 && q <= NWL) {
                            park_w(q - 1, buf ^ 1);
                            issue_w(q - 1, ew, kb2);
                        }
                        // (the last of this block's rows were read at k-step 2)
                        if (q > 2 * NJ) {
                            constexpr int kSlots = 2 * NJ - 1;
#pragma unroll
                            for (int i = 0; i < NL; ++i)
                                if (i * kSlots / NL == q - 2 * NJ - 1) {
                                    park_x(i);
                                    issue_x(i, xo, kb2);
                                }
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            } else {
#pragma unroll
                for (int i = 0; i < NWL; ++i) {
                    park_w(i, buf ^ 1);
                    issue_w(i, ew, kb2);
                }
                if (xp) {
#pragma unroll
                    for (int i = 0; i < NL; ++i) park_x(i);
                }
                if (xi) {
#pragma unroll
                    for (int i = 0; i < NL; ++i) issue_x(i, xo, kb2);
                }
            }
        };
        for (int kb = 0; kb < NKB - 2; ++kb) {
            block(e, xoff, kb + 2, false, false);
            lds_barrier();
            buf ^= 1;
        }
        // The next item's rows are requested here, two blocks before the end: vector loads return
        // in order, so requested any later they would queue behind the next item's first blocks,
        // and any earlier their wait would hold up this item's start.
        uint32_t xoffn[NL];
        bool activen;
        rows_of(itemn, xoffn, activen);
        block(en, xoffn, 0, false, activen);    // block NKB - 2
        lds_barrier();
        buf ^= 1;
        block(en, xoffn, 1, activen, activen);  // block NKB - 1; the next item's block 0 is parked
        park_bias(en, par ^ 1);
        lds_barrier();
        buf ^= 1;

        if (active) with_activation(act, [&](auto act_c) {
            constexpr int ACT = decltype(act_c)::value;
            const float* sb = sbias + par * MT * 16;
            // lane (h, c) of tile (nj, tj): list row 32 tj + c; registers 0..3 and 8..11 are the eight
            // neurons of piece 4 nj + h of the H row, 4..7 and 12..15 those of piece 4 nj + 2 + h
            // (neuron_of_slot over a pair of 16-row tiles)
#pragma unroll
            for (int tj = 0; tj < TJ; ++tj) {
                __bf16* dst = Hf + ((size_t)item * UR + w * WR + 32 * tj + c32) * (KS * 32);
#pragma unroll
                for (int nj = 0; nj < KS; ++nj) {
#pragma unroll
                    for (int half = 0; half < 2; ++half) {
                        const int n0 = 8 * (4 * nj + 2 * half + h);
                        bf16x8 hv;
#pragma unroll
                        for (int r = 0; r < 8; ++r) {
                            const int i = 4 * half + (r & 3) + 8 * (r >> 2);
                            float v;
                            if (GATED) v = activate_fast(ACT, acc[NJ / 2 + nj][tj][i]) * acc[nj][tj][i];
                            else v = activate_fast(ACT, acc[nj][tj][i] + sb[n0 + r]);
                            if (n0 + r >= m) v = 0.0f;
                            hv[r] = (__bf16)v;
                        }
                        *reinterpret_cast<bf16x8*>(dst + n0) = hv;
                        // eight values at a time: interleaving more of them costs registers the
                        // requests in flight are using
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
        });
        if (!more) break;
        j = jn;
        e = en;
        item = itemn;
        active = activen;
        par ^= 1;
#pragma unroll
        for (int i = 0; i < NL; ++i) xoff[i] = xoffn[i];
    }
}

// The same for plain experts of 65 to 128 neurons.  The K blocks of all the items of a workgroup form one stream: while block k is
// multiplied, the loads of block k+1 go straight to LDS -- also across the end of an item, so that the first block of the
// next item arrives during the activation epilogue of the current one.  A wavefront has the x rows of its block in registers
// before it requests the next ones into their place; the weights, which all four wait for, are requested first.  What
// bounds it: the requests that go beyond the L2s (without any of them 100 us instead of 170), and the vector path.  A ds_write_b128 of staging
// registers takes 35 clocks of a CU per KB beside the 17 of its load, a load to LDS the 17 alone.  24 x 128 experts, d = 768, whole call,
// through registers with two blocks in flight / straight to LDS with one: 50432 tokens at 50 % 377 / 367 us (the first call on new
// buffers 412 / 398), 30000 at 30 % 192 / 187, 12608 at 20 % 94 / 93.  Built and slower: rows before weights (374), everything at the
// block's start (376), one workgroup of 512 rows per CU (388).
// Only for x at a 16-byte address, as loads to LDS want it: at any other the kernel above takes them.  (With rows through registers
// here, x at 8 bytes from such an address, 50432 tokens at 50 % 466 us, loaded at a block's start and written at its end 416, above 387.)
template <int MT, int TT, bool NEAR>
__global__ __launch_bounds__(256, 2) void up_wide_plain_kernel(
    const __bf16* __restrict__ x, const __bf16* __restrict__ wupf, const __bf16* __restrict__ b_up,
    const int32_t* __restrict__ witem, const int2* __restrict__ worder,
    const int32_t* __restrict__ alist, __bf16* __restrict__ Hf, int d, int E, int m, int act) {
    constexpr int KS = MT / 2;
    constexpr int NJ = MT / 2, TJ = TT / 2;  // tiles of the 32x32x16 MFMA: neurons, list rows
    constexpr int WR = TT * 16;         // rows per wavefront
    constexpr int UR = 4 * WR;          // rows per work item
    constexpr int NL = TT * 2;          // x load instructions per K block
    constexpr int NWF = 2 * MT;         // weight fragments (1 KiB each) per K block
    constexpr int NWL = NWF / 4;        // ... of which each wavefront requests every fourth
    static_assert(NWF % 4 == 0 && MT % 2 == 0, "weight fragments are copied four at a time");
    // (arrays of their own: the compiler then sees that reads of one do not wait for loads to another)
    __shared__ __attribute__((aligned(128))) char wbuf0[NWF * 1024];
    __shared__ __attribute__((aligned(128))) char wbuf1[NWF * 1024];
    __shared__ __attribute__((aligned(128))) char xbuf[4 * WR * 128];
    __shared__ float sbias[2 * MT * 16];
    const int lane = threadIdx.x & 63, h = lane >> 5, c32 = lane & 31;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    char* const xs = xbuf + w * (WR * 128);  // [WR][128], private to the wavefront
    const int NK32 = d / 32, NKB = d / 64;   // NKB is even
    const int ld_row = lane >> 3, ld_piece = lane & 7;
    // this XCD's share of the items (workgroups are dealt round-robin to the 8 XCDs; the grid is a
    // multiple of 8), in the order laid out by the list fill
    const int xcd = blockIdx.x & 7, step = gridDim.x >> 3;
    const int total = xcd_first(witem[E], xcd + 1);
    const int first = xcd_first(witem[E], xcd);
    int j = first + (int)(blockIdx.x >> 3);
    if (j >= total) return;
    // (from the end: an expert's last item, often nearly empty, comes before its full ones, so that the
    // workgroups do not end with items of a wavefront or two)
    auto locate = [&](int jj, int& e, int& item) {
        const int2 v = worder[total - 1 - (jj - first)];
        e = v.x;
        item = v.y;
    };
    // tokens of the x rows this lane fetches; padding rows (-1) read token 0 and produce H rows
    // that nobody merges
    const XRows<NEAR> xrows(x, d);
    auto rows_of = [&](int item, uint32_t (&xoff)[NL], bool& active) {
        const int32_t* tl = alist + (size_t)item * UR + w * WR;
        active = __builtin_amdgcn_readfirstlane(tl[0]) >= 0;  // valid rows are a prefix
#pragma unroll
        for (int i = 0; i < NL; ++i)  // piece p of row c lies at p ^ (c / 2): 16 rows' pieces use all the banks
            xoff[i] = xrows.row(max(tl[ld_row + 8 * i], 0), ld_piece ^ (4 * (i & 1) + (ld_row >> 1)));
    };
    // Weight fragment f = mt * 2 + ks of a K block; this wavefront requests the fragments f = 4 i + w: ks = w & 1, mt = 2 i + (w >> 1).
    __amdgpu_buffer_rsrc_t wf;
    auto weights_of = [&](int e) {
        const size_t at = (size_t)__builtin_amdgcn_readfirstlane(e) * MT * NK32 * 512;
        wf = __builtin_amdgcn_make_buffer_rsrc((void*)(wupf + at), 0, MT * NK32 * 1024, kRawBuffer);
    };
    auto request_w = [&](int i, int kb, char* to) {
        buffer_to_lds(wf, lane * 16, ((2 * i + (w >> 1)) * NK32 + 2 * kb + (w & 1)) * 1024, to + (4 * i + w) * 1024);
    };
    auto request_x = [&](int i, const uint32_t (&xoff)[NL], int kb) {
        xrows.to_lds(xoff[i], kb, xs + 1024 * i);
    };
    auto park_bias = [&](int e, int par) {  // the item's biases, by neuron
        if ((int)threadIdx.x < MT * 16)
            sbias[par * MT * 16 + threadIdx.x] =
                b_up ? (float)b_up[(size_t)e * m + min((int)threadIdx.x, m - 1)] : 0.0f;
    };

    int e, item;
    uint32_t xoff[NL];
    bool active;
    locate(j, e, item);
    rows_of(item, xoff, active);
    weights_of(e);
#pragma unroll
    for (int i = 0; i < NWL; ++i) request_w(i, 0, wbuf0);
    if (active) {
#pragma unroll
        for (int i = 0; i < NL; ++i) request_x(i, xoff, 0);
    }
    park_bias(e, 0);
    wait_vmem();
    lds_barrier();
    int par = 0;
    for (;;) {
        // the item after this one (the last item names itself: its first block is read again
        // and never used)
        const int jn = j + step;
        const bool more = jn < total;
        int en = e, itemn = item;
        if (more) locate(jn, en, itemn);

        f32x16 acc[NJ][TJ];
#pragma unroll
        for (int nj = 0; nj < NJ; ++nj)
#pragma unroll
            for (int tj = 0; tj < TJ; ++tj)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[nj][tj][r] = 0.f;
        // One K block: its rows of x to registers, then the requests of the next block (kb; of this item or the next: rows
        // xo, xi whether they are wanted) between the products of this one.  The wait for them and the barrier
        // stand at the end.
        auto block = [&](const char* wb, char* wn, const uint32_t (&xo)[NL], int kb, bool xi) {
            if (active) {
                // operands of k-step s (16 wide): neuron tile nj from the fragments of its two
                // 16-row tiles, token tile tj from the staged rows; the next neuron tile's (and the
                // next k-step's) operands are read while the current tile's MFMAs run
                const char* wsrc_l = wb + (c32 >> 4) * 2048 + (h * 16 + (c32 & 15)) * 16;
                auto read_a = [&](int s, int nj) {
                    return *reinterpret_cast<const bf16x8*>(wsrc_l + nj * 4096 + (s >> 1) * 1024 + (s & 1) * 512);
                };
                constexpr int kAhead = 3;  // weight tiles
                bf16x8 b[4][TJ], a[kAhead + 1];
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int tj = 0; tj < TJ; ++tj)
                        b[s][tj] = *reinterpret_cast<const bf16x8*>(xs + (32 * tj + c32) * 128 + (((2 * s + h) ^ ((c32 >> 1) & 7)) << 4));
#pragma unroll
                for (int q = 0; q < kAhead; ++q) a[q] = read_a(q / NJ, q % NJ);
                __builtin_amdgcn_sched_barrier(0);
                __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the rows are out of the LDS that the requests below fill
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int s = 0; s < 4; ++s) {
#pragma unroll
                    for (int nj = 0; nj < NJ; ++nj) {
                        const int q = s * NJ + nj;
                        __builtin_amdgcn_sched_barrier(0);
                        if (q + kAhead < 4 * NJ) a[(q + kAhead) % (kAhead + 1)] = read_a((q + kAhead) / NJ, (q + kAhead) % NJ);
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int tj = 0; tj < TJ; ++tj) {
                            acc[nj][tj] = mfma32(a[q % (kAhead + 1)], b[s][tj], acc[nj][tj]);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                        if (q < NWL) {
                            request_w(q, kb, wn);
                        } else if (q < NWL + NL / 2) {
                            if (xi) {
                                request_x(2 * (q - NWL), xo, kb);
                                request_x(2 * (q - NWL) + 1, xo, kb);
                            }
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            } else {
                if (xi) {
#pragma unroll
                    for (int i = 0; i < NL; ++i) request_x(i, xo, kb);
                }
#pragma unroll
                for (int i = 0; i < NWL; ++i) request_w(i, kb, wn);
            }
            wait_vmem();
            lds_barrier();
        };
        for (int kb = 0; kb < NKB - 2; kb += 2) {
            block(wbuf0, wbuf1, xoff, kb + 1, active);
            block(wbuf1, wbuf0, xoff, kb + 2, active);
        }
        uint32_t xoffn[NL];
        bool activen;
        rows_of(itemn, xoffn, activen);
        block(wbuf0, wbuf1, xoff, NKB - 1, active);
        park_bias(en, par ^ 1);
        weights_of(en);
        block(wbuf1, wbuf0, xoffn, 0, activen);  // the next item's block 0 is requested

        if (active) with_activation(act, [&](auto act_c) {
            constexpr int ACT = decltype(act_c)::value;
            const float* sb = sbias + par * MT * 16;
            // lane (h, c) of tile (nj, tj): list row 32 tj + c; registers 0..3 and 8..11 are the eight
            // neurons of piece 4 nj + h of the H row, 4..7 and 12..15 those of piece 4 nj + 2 + h
            // (neuron_of_slot over a pair of 16-row tiles)
#pragma unroll
            for (int tj = 0; tj < TJ; ++tj) {
                __bf16* dst = Hf + ((size_t)item * UR + w * WR + 32 * tj + c32) * (KS * 32);
#pragma unroll
                for (int nj = 0; nj < KS; ++nj) {
#pragma unroll
                    for (int half = 0; half < 2; ++half) {
                        const int n0 = 8 * (4 * nj + 2 * half + h);
                        bf16x8 hv;
#pragma unroll
                        for (int r = 0; r < 8; ++r) {
                            const int i = 4 * half + (r & 3) + 8 * (r >> 2);
                            float v = activate_fast(ACT, acc[nj][tj][i] + sb[n0 + r]);
                            if (n0 + r >= m) v = 0.0f;
                            hv[r] = (__bf16)v;
                        }
                        *reinterpret_cast<bf16x8*>(dst + n0) = hv;
                        // eight values at a time: interleaving more of them costs registers the
                        // requests in flight are using
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
        });
        if (!more) break;
        j = jn;
        e = en;
        item = itemn;
        active = activen;
        par ^= 1;
#pragma unroll
        for (int i = 0; i < NL; ++i) xoff[i] = xoffn[i];
    }
}

// The same for a small batch (token_sets.h): a workgroup of eight wavefronts has one item, of 128 TJ rows.  There are few items
// -- one or two an expert -- so that a CU has one workgroup, and what bounds the kernel is how much of the weights is on
// its way from HBM (D K blocks, in registers) and, for an expert of more than 128 rows, the LDS traffic of its rows.
// Wavefront w has the 32-row tiles w & 3 and 4 + (w & 3) of the item, so that a part-filled item keeps all of them busy, and
// half of the neurons; it works on as many tiles as there are.  256 gated experts of 64, d = 2048, against the kernel above: 120
// tokens 35.1 -> 31.1 us (134 MB of weights: half of the workgroups end after 27), 333 tokens (125 rows an expert, up to
// 250) 50.5 -> 43.4 (half end after 29, the fullest after 40), 512 tokens 50.3 -> 49.8; 24 plain ones of 128, 788 tokens 21.4 -> 12.5.
// Slower: four wavefronts with all the neurons (47.5 at 333 tokens); spilled registers (57: a reload waits for all that is on its way).
template <int MT, bool GATED, int TJ>
__global__ __launch_bounds__(512, 2) void up_wide_sets_kernel(
    const __bf16* __restrict__ x, const __bf16* __restrict__ wupf, const __bf16* __restrict__ wgatef,
    const __bf16* __restrict__ b_up, __bf16* __restrict__ Hf, int d, int E, int m, int act, const TokenSets S) {
    constexpr int BR = GATED ? 2 : 1;
    constexpr int KS = MT / 2;
    constexpr int NT = BR * MT;         // neuron tiles (of 16) per K step
    constexpr int NJ = NT / 4;          // ... of 32, per wavefront
    constexpr int WR = 32 * TJ;         // rows per pair of wavefronts
    constexpr int UR = 4 * WR;          // rows per work item
    constexpr int NWF = 2 * NT;         // weight fragments (1 KiB each) per K block
    constexpr int NWL = NWF / 8;        // ... of which each wavefront copies every eighth
    constexpr int D = 4;                // blocks on their way
    static_assert(NJ == 2 && NWL == 2, "eight neuron tiles");
    extern __shared__ char smem[];  // three K blocks
    constexpr int kBuf = NWF * 1024 + 4 * WR * kUpRowBytes;  // a K block: its weights, then the rows of x
    const int lane = threadIdx.x & 63, h = lane >> 5, c32 = lane & 31;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wt = w & 3, wn = w >> 2;
    float* sbias = reinterpret_cast<float*>(smem + 3 * kBuf);  // [MT * 16]
    int32_t* s_list = reinterpret_cast<int32_t*>(sbias + MT * 16) + WR * w;
    const int NK32 = d / 32, NKB = d / 64;   // NKB: a multiple of D
    const int ld_row = lane >> 3, ld_piece = lane & 7;
    const int e = blockIdx.x % E, slot = blockIdx.x / E;
    ExpertTokens tok;
    tok.load(S, E, e, 256, w == 0 && slot == 0);
    const int rows = tok.total - UR * slot;
    if (rows <= 0) return;
    // row 128 tj + 32 wt + c of the item is row 32 tj + c of the pair of wavefronts
    tok.list<WR, UR>(UR * slot, s_list, [&](int r) { return ((r >> 5) & 3) == wt ? 32 * (r >> 7) + (r & 31) : -1; });
    // Weight fragment f = (br * MT + mt) * 2 + ks of a K block; this wavefront copies the
    // fragments f = 8 i + w: ks = w & 1, mt = (4 i) % MT + (w >> 1), br = (4 i) / MT.
    const size_t we = (size_t)e * MT * NK32 * 512 + (size_t)(((w >> 1) * NK32 + (w & 1)) * 512 + lane * 8);
    bf16x8 wr[D][NWL];
    auto issue_w = [&](int i, int kb, bf16x8& r) {
        const __bf16* base = (GATED && (4 * i) / MT == BR - 1) ? wgatef : wupf;
        r = load8(base + we + (size_t)kb * 1024 + (size_t)((4 * i) % MT) * NK32 * 512);
    };
    auto park_w = [&](int i, char* buf, const bf16x8& r) {
        *reinterpret_cast<bf16x8*>(buf + (8 * i + w) * 1024 + lane * 16) = r;
    };
    if (!GATED && (int)threadIdx.x < MT * 16)  // plain experts: the biases, by neuron
        sbias[threadIdx.x] = b_up ? (float)b_up[(size_t)e * m + min((int)threadIdx.x, m - 1)] : 0.0f;
    const size_t row0 = (size_t)e * ((S.T + 255) / 256) * 256 + (size_t)slot * UR;
    // this wavefront's neuron tiles: an up tile and the gate tile of the same neurons, or two neighbouring ones
    auto tile_of = [&](int nj) { return GATED ? 2 * nj + wn : 2 * wn + nj; };

    // all of the item for a wavefront of NTJ tiles
    auto work = [&](auto ntj_c) {
        constexpr int NTJ = decltype(ntj_c)::value, NA = NTJ ? NTJ : 1;
        constexpr int NL = 2 * NTJ, NLA = NL ? NL : 1;  // x load instructions per K block: 8 rows x 128 bytes each
        uint32_t xoff[NLA];  // (none: token 0, rows that nobody merges)
#pragma unroll
        for (int i = 0; i < NL; ++i) xoff[i] = (uint32_t)max(s_list[ld_row + 16 * i + 8 * wn], 0);
        bf16x8 xr[D][NLA];
        auto issue_x = [&](int i, int kb, bf16x8& r) {
            r = load8(x + ((size_t)xoff[i] * (uint32_t)d + (uint32_t)(8 * ld_piece + 64 * kb)));
        };
        auto park_x = [&](int i, char* buf, const bf16x8& r) {
            *reinterpret_cast<bf16x8*>(buf + NWF * 1024 + (wt * WR + ld_row + 16 * i + 8 * wn) * kUpRowBytes + ld_piece * 16) = r;
        };
#pragma unroll
        for (int b = 0; b < D; ++b) {
#pragma unroll
            for (int i = 0; i < NWL; ++i) issue_w(i, b, wr[b][i]);
#pragma unroll
            for (int i = 0; i < NL; ++i) issue_x(i, b, xr[b][i]);
        }
        // operands of k-step s (16 wide)
        struct Step {
            bf16x8 a[NJ], b[NA];
        };
        auto read = [&](const char* buf, int s, Step& o) {
#pragma unroll
            for (int nj = 0; nj < NJ; ++nj)
                o.a[nj] = *reinterpret_cast<const bf16x8*>(buf + (2 * tile_of(nj) + (c32 >> 4)) * 2048 + (s >> 1) * 1024 + (s & 1) * 512 +
                                                           (h * 16 + (c32 & 15)) * 16);
#pragma unroll
            for (int tj = 0; tj < NTJ; ++tj)
                o.b[tj] = *reinterpret_cast<const bf16x8*>(buf + NWF * 1024 + (wt * WR + 32 * tj + c32) * kUpRowBytes + h * 16 + s * 32);
        };
        f32x16 acc[NJ][NA];
#pragma unroll
        for (int nj = 0; nj < NJ; ++nj)
#pragma unroll
            for (int tj = 0; tj < NA; ++tj)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[nj][tj][r] = 0.f;
        auto multiply = [&](const Step& o) {
#pragma unroll
            for (int nj = 0; nj < NJ; ++nj)
#pragma unroll
                for (int tj = 0; tj < NTJ; ++tj) acc[nj][tj] = mfma32(o.a[nj], o.b[tj], acc[nj][tj]);
            __builtin_amdgcn_sched_barrier(0);
        };
        char *cur = smem, *nxt = smem + kBuf, *then = smem + 2 * kBuf;
#pragma unroll
        for (int i = 0; i < NWL; ++i) {
            park_w(i, cur, wr[0][i]);
            issue_w(i, min(D, NKB - 1), wr[0][i]);
        }
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            park_x(i, cur, xr[0][i]);
            issue_x(i, min(D, NKB - 1), xr[0][i]);
        }
        lds_barrier();
        Step o[2];
        read(cur, 0, o[0]);
        // A block: the next one is parked (register set R, into which block kb is then requested; kb < 0: none) while its
        // first half is multiplied; the barrier; operands are read a k-step ahead.  (A wavefront that has passed the
        // barrier may still be reading this block and a faster one parking the block after the next: three buffers.)
        auto block = [&](auto i_c, auto park_c, int kb) {
            constexpr int I = decltype(i_c)::value, R = (I + 1) % D;
            constexpr bool PARK = decltype(park_c)::value;
            __builtin_amdgcn_sched_barrier(0);
            read(cur, 1, o[1]);
            if (PARK) {
#pragma unroll
                for (int i = 0; i < NWL; ++i) {
                    park_w(i, nxt, wr[R][i]);
                    if (kb >= 0) issue_w(i, kb, wr[R][i]);
                }
            }
            multiply(o[0]);
            read(cur, 2, o[0]);
            if (PARK) {
#pragma unroll
                for (int i = 0; i < NL; ++i) {
                    park_x(i, nxt, xr[R][i]);
                    if (kb >= 0) issue_x(i, kb, xr[R][i]);
                }
            }
            multiply(o[1]);
            if (PARK) lds_barrier();
            read(cur, 3, o[1]);
            multiply(o[0]);
            if (PARK) read(nxt, 0, o[0]);
            multiply(o[1]);
            char* const t = cur;
            cur = nxt;
            nxt = then;
            then = t;
        };
        const std::true_type yes;
        const std::integral_constant<int, 0> i0;
        const std::integral_constant<int, 1> i1;
        const std::integral_constant<int, 2> i2;
        const std::integral_constant<int, 3> i3;
        int kb0 = 0;
        for (; kb0 + D < NKB; kb0 += D) {
            block(i0, yes, kb0 + 5);
            block(i1, yes, kb0 + 6);
            block(i2, yes, kb0 + 7);
            block(i3, yes, min(kb0 + 8, NKB - 1));  // (past the end: the last block again, never used)
        }
        block(i0, yes, -1);
        block(i1, yes, -1);
        block(i2, yes, -1);
        block(i3, std::false_type{}, -1);
        if constexpr (NTJ > 0) with_activation(act, [&](auto act_c) {
            constexpr int ACT = decltype(act_c)::value;
            // (which register is which neuron: see up_wide_bf16_kernel)
#pragma unroll
            for (int tj = 0; tj < NTJ; ++tj) {
                __bf16* dst = Hf + (row0 + 128 * tj + 32 * wt + c32) * (KS * 32);
#pragma unroll
                for (int nj = 0; nj < (GATED ? 1 : 2); ++nj) {
#pragma unroll
                    for (int half = 0; half < 2; ++half) {
                        const int n0 = 8 * (4 * tile_of(nj) + 2 * half + h);
                        bf16x8 hv;
#pragma unroll
                        for (int r = 0; r < 8; ++r) {
                            const int i = 4 * half + (r & 3) + 8 * (r >> 2);
                            float v;
                            if (GATED) v = activate_fast(ACT, acc[1][tj][i]) * acc[0][tj][i];
                            else v = activate_fast(ACT, acc[nj][tj][i] + sbias[n0 + r]);
                            if (n0 + r >= m) v = 0.0f;
                            hv[r] = (__bf16)v;
                        }
                        *reinterpret_cast<bf16x8*>(dst + n0) = hv;
                    }
                }
            }
        });
    };
    // (every path has the same barriers)
    if (TJ == 2 && rows > 128 + 32 * wt) work(std::integral_constant<int, TJ>{});
    else if (rows > 32 * wt) work(std::integral_constant<int, 1>{});
    else work(std::integral_constant<int, 0>{});
}

// ---- launchers ---------------------------------------------------------------------------------------
size_t up_lds(const dmoe_layer& L, int TT, int NBUF, bool sets) {  // the item table of a window (or four lists) and the staged rows
    return (sets ? 4 * 64 * 4 : ((2 * (size_t)L.n_experts + 1) * 4 + 15) / 16 * 16) + 4 * NBUF * (size_t)TT * 16 * kUpRowBytes;
}

template <int MT, bool GATED, int TT, int NBUF, bool NEAR, bool PTR = false, bool SETS = false>
void launch_up_t(const dmoe_layer& L, const void* x, const PackedLayout& P, const int32_t* witem,
                 const int32_t* wfirst, int NW, const int32_t* alist, TokenSets S, void* H, int grid,
                 hipStream_t s) {
    if (SETS) grid = sets_grid(S, L.n_experts, 16 * TT, 256 * (NBUF == 1 ? 3 : 2));
    const size_t lds = up_lds(L, TT, NBUF, SETS);
    static std::once_flag attr_once;  // kernel attributes: once per process, thread-safe
    std::call_once(attr_once, [&] {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&up_bf16_kernel<MT, GATED, TT, NBUF, NEAR, PTR, SETS>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    });
    const char* pk = static_cast<const char*>(L.packed);
    launch_kernel(up_bf16_kernel<MT, GATED, TT, NBUF, NEAR, PTR, SETS>, grid, 256, lds, s, 
        (const __bf16*)x, (const __bf16*)(pk + P.wupf), (const __bf16*)(pk + P.wgatef),
        (const __bf16*)L.b_up, witem, wfirst, NW, alist, (__bf16*)H, L.d_model, L.n_experts,
        L.expert_size, L.act, S);
}

template <int MT, bool GATED, int TT>
void launch_up_wide_t(const dmoe_layer& L, const void* x, const PackedLayout& P,
                      const int32_t* witem, const void* worder, const int32_t* alist,
                      void* H, int grid, hipStream_t s) {
    constexpr int NWF = 2 * (GATED ? 2 : 1) * MT;
    const size_t lds = 2 * NWF * 1024 + 4 * (size_t)TT * 16 * kUpRowBytes + 2 * MT * 16 * sizeof(float);
    static std::once_flag attr_once;  // kernel attributes: once per process, thread-safe
    std::call_once(attr_once, [&] {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&up_wide_bf16_kernel<MT, GATED, TT>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    });
    const char* pk = static_cast<const char*>(L.packed);
    launch_kernel(up_wide_bf16_kernel<MT, GATED, TT>, grid, 256, lds, s,
        (const __bf16*)x, (const __bf16*)(pk + P.wupf), (const __bf16*)(pk + P.wgatef),
        (const __bf16*)L.b_up, witem, (const int2*)worder, alist, (__bf16*)H, L.d_model, L.n_experts,
        L.expert_size, L.act);
}

template <int MT, int TT, bool NEAR>
void launch_up_wide_plain_t(const dmoe_layer& L, const void* x, const PackedLayout& P,
                            const int32_t* witem, const void* worder, const int32_t* alist,
                            void* H, int grid, hipStream_t s) {
    launch_kernel(up_wide_plain_kernel<MT, TT, NEAR>, grid, 256, 0, s, (const __bf16*)x,
        (const __bf16*)(static_cast<const char*>(L.packed) + P.wupf), (const __bf16*)L.b_up, witem, (const int2*)worder,
        alist, (__bf16*)H, L.d_model, L.n_experts, L.expert_size, L.act);
}

template <int MT, bool GATED, int TJ>
void launch_up_wide_sets_t(const dmoe_layer& L, const void* x, const PackedLayout& P, const TokenSets& S, void* H, hipStream_t s) {
    constexpr int NWF = 2 * (GATED ? 2 : 1) * MT;
    const size_t lds = 3 * (NWF * 1024 + 4 * (size_t)TJ * 32 * kUpRowBytes) + MT * 16 * sizeof(float) + 8 * 32 * TJ * sizeof(int32_t);
    static_assert(3 * (NWF * 1024 + 4 * TJ * 32 * kUpRowBytes) + MT * 16 * 4 + 8 * 32 * TJ * 4 <= 160 * 1024, "LDS");
    static std::once_flag attr_once;  // kernel attributes: once per process, thread-safe
    std::call_once(attr_once, [&] {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&up_wide_sets_kernel<MT, GATED, TJ>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    });
    const char* pk = static_cast<const char*>(L.packed);
    launch_kernel(up_wide_sets_kernel<MT, GATED, TJ>, L.n_experts * div_up(S.T, 128 * TJ), 512, lds, s, (const __bf16*)x,
                  (const __bf16*)(pk + P.wupf), (const __bf16*)(pk + P.wgatef), (const __bf16*)L.b_up, (__bf16*)H, L.d_model,
                  L.n_experts, L.expert_size, L.act, S);
}

template <int MT, bool GATED>
void launch_up_wide_sets(const dmoe_layer& L, const void* x, const PackedLayout& P, const TokenSets& S, void* H, hipStream_t s) {
    // With few experts items of 128 rows, as long as every one has a CU: 24 x 128 experts, 788 tokens, a quarter of them per token, 12.5 us
    // against 17.7.  Otherwise the experts of more than 128 rows would wait for a second round: 256 x 64, 200 tokens 41.6 against 36.6.
    if (L.n_experts * div_up(S.T, 128) <= 256) launch_up_wide_sets_t<MT, GATED, 1>(L, x, P, S, H, s);
    else launch_up_wide_sets_t<MT, GATED, 2>(L, x, P, S, H, s);
}

}  // namespace

bool experts_bf16_supported(const dmoe_layer& L) {
    const int mp = m_pad_of(L.expert_size);
    if (!(mp == 32 || mp == 64 || mp == 128)) return false;
    if (L.gated && mp == 128) return false;  // accumulators of both branches would not fit
    return down_bf16_supported(L) && L.n_experts <= kMaxExperts;
}

void launch_pack_bf16(const dmoe_layer& L, void* packed, hipStream_t s) {
    LaunchTimer tm(kSlotPack, s);
    const PackedLayout P = packed_layout(L);
    const int mp = m_pad_of(L.expert_size);
    char* pk = static_cast<char*>(packed);
    const int fp8 = weights_fp8(L);
    const int E = L.n_experts, m = L.expert_size, d = L.d_model;
    const float* scales = nullptr;   // the snapped copy inside the packed buffer
    if (fp8) {
        launch_kernel(snap_scales_kernel, div_up(3 * E, 256), 256, 0, s, L.w_scales,
                      (float*)(pk + P.scales), 3 * E);
        scales = (const float*)(pk + P.scales);
    }
    launch_pack_columns(L, scales, (__bf16*)(pk + P.w2f), SmallDownMap{mp / 32, E * (mp / 32)}, s);
    launch_pack_down_bf16(L, pk + P.w2g, s);
    if (down_quad_w_bytes(L)) launch_pack_down_quad(L, packed, s);
    launch_kernel(pack_up_kernel<__bf16>, 2048, 256, 0, s, L.w_up, scales, fp8, 0, (__bf16*)(pk + P.wupf), E,
                                                m, d, mp / 16, 1);
    if (L.gated)
        launch_kernel(pack_up_kernel<__bf16>, 2048, 256, 0, s, L.w_gate, scales, fp8, 1,
                                                    (__bf16*)(pk + P.wgatef), E, m, d, mp / 16, 1);
    if (up_tiny_supported(L))
        launch_kernel(pack_up_tiny_kernel, 2048, 256, 0, s, L.w_up, L.w_gate, scales, fp8,
                                                 (__bf16*)(pk + P.wtinyf), E, m, d, L.gated);
    if (fp8) {  // byte fragments for the small-token kernels
        launch_pack_columns(L, scales, (uint8_t*)(pk + P.w2f8), SmallDownMap{mp / 32, E * (mp / 32)}, s);
        launch_kernel(pack_up_kernel<uint8_t>, 2048, 256, 0, s, L.w_up, scales, 1, 0, (uint8_t*)(pk + P.wupf8),
                                                     E, m, d, mp / 16, 1);
        if (L.gated)
            launch_kernel(pack_up_kernel<uint8_t>, 2048, 256, 0, s, L.w_gate, scales, 1, 1,
                                                         (uint8_t*)(pk + P.wgatef8), E, m, d, mp / 16, 1);
    }
    if (up_x8_supported(L)) launch_pack_x8(L, packed, s);  // operands of the 8-bit up-projection
    if (down_x8_shape(L)) launch_pack_down_x8(L, packed, s);  // ... and of the 8-bit down-projection
    // the router matrices use the same fragment format: "one expert" whose rows are the hidden
    // units (r_w1) or the experts (r_w2)
    const int dh = L.router_hidden;
    if (L.r_w1 && L.r_w2 && dh > 0 && dh % 32 == 0 && L.d_model % 32 == 0) {
        launch_kernel(pack_up_kernel<__bf16>, 512, 256, 0, s, L.r_w1, nullptr, 0, 0, (__bf16*)(pk + P.r1f), 1, dh,
                                                   L.d_model, dh / 16, 0);
        launch_kernel(pack_up_kernel<__bf16>, 512, 256, 0, s, L.r_w2, nullptr, 0, 0, (__bf16*)(pk + P.r2f), 1,
                                                   L.n_experts, dh, div_up(L.n_experts, 16), 0);
    }
}

// Where the weights of all experts fit an L2 or so, every XCD may as well read all of them and keep
// to its own tokens; else the weights are what must not be read by every XCD.
bool up_items_by_experts(const dmoe_layer& L) {
    const size_t bytes = (size_t)L.n_experts * (L.gated ? 2 : 1) * m_pad_of(L.expert_size) * L.d_model *
                         (up_x8_supported(L) ? 1 : 2);
    return bytes > ((size_t)8 << 20);
}

// Groups of 64 tokens per up-projection window: the x rows of a window (about 3 MB) should stay
// in the 4 MB L2 of the XCD that works on it, and the number of windows is a multiple of 8, or
// divides 8, so that every XCD gets the same share.
int up_window_groups(const dmoe_layer& L, int T) {
    const int NG = std::max(1, div_up(T, kGroup));
    // wide experts: per window the XCD would stream every expert's weights (far more than its
    // L2) through the same cache, and the 256-row items span more than a window; measured slower
    if (up_rows_bf16(L) != 64) return std::max(1, NG);
    const double x_bytes = 2.0 * (double)NG * kGroup * L.d_model;
    // Small batches: 1, 2, 4 or 8 windows, the XCDs of a window sharing the experts -- the number with
    // which the least comes from beyond the L2s (the weights once per window, x once per share), while
    // the x rows of a window are not much more than an L2 holds; a little more is taken where the
    // weights are the larger part.  (Up-projection, us, with 1 / 2 / 4 / 8 windows: 2048 gated experts of
    // 8, d = 2048, 1800 tokens 106 / 111 / 128 / 139, 4096 tokens 261 / 223 / 191 / 216; 512 experts of
    // 6, d = 768, 5000 tokens 36 / 34 / 34 / 40, 16384 tokens 172 / 136 / 104 / 95; 128 experts of 24,
    // 16384 tokens 76 / 62 / 50 / 47.)
    const double rows = up_tiny_supported(L) ? 16 : (L.gated ? 2 : 1) * m_pad_of(L.expert_size);
    const double w_bytes = 2.0 * L.n_experts * rows * L.d_model, most = w_bytes > x_bytes ? 8.0e6 : 6.0e6;
    if (x_bytes <= 8 * most) {
        int best = 8;
        for (int a = 4; a >= 1; a /= 2)
            if (x_bytes <= a * most && a * w_bytes + 8 / a * x_bytes < best * w_bytes + 8 / best * x_bytes) best = a;
        // (whole groups per window: where that does not come out as a number of windows that divides the
        // XCDs, one window)
        const int groups = div_up(NG, best);
        return 8 % div_up(NG, groups) == 0 ? groups : std::max(1, NG);
    }
    const double window_bytes = 3.2 * 1048576.0;
    const int n_windows = 8 * std::max(1, (int)ceil(x_bytes / (8.0 * window_bytes)));
    return std::max(1, div_up(NG, n_windows));
}

void launch_up_bf16(const dmoe_layer& L, const void* x, int T, const int32_t* witem,
                    const int32_t* wfirst, const void* worder, const int32_t* alist, const TokenSets& S, void* H,
                    hipStream_t s) {
    LaunchTimer tm(kSlotUp, s);
    const PackedLayout P = packed_layout(L);
    const int NW = div_up(div_up(T, kGroup), up_window_groups(L, T));
    // persistent workgroups, capped at what a CU holds; with few items at most one wavefront each has
    // one (wave_of); a multiple of 8 so that every XCD runs the same number
    const long long worst = (long long)T * L.n_experts / up_rows_bf16(L) + L.n_experts;
    const int grid = round_up((int)std::min<long long>(worst, 256 * 2), 8);
    const int mt = m_pad_of(L.expert_size) / 16;
    const bool near = (size_t)T * L.d_model * 2 < ((size_t)1 << 31);  // (XRows)
    if (up_rows_bf16(L) == 256) {  // wide experts: weights shared through LDS
        const int wgrid = round_up(
            (int)std::min<long long>((long long)T * L.n_experts / 256 + L.n_experts, 512), 8);
        if (S.sets && L.gated) launch_up_wide_sets<4, true>(L, x, P, S, H, s);
        else if (S.sets) launch_up_wide_sets<8, false>(L, x, P, S, H, s);
        else if (L.gated) launch_up_wide_t<4, true, 4>(L, x, P, witem, worder, alist, H, wgrid, s);
        else if (reinterpret_cast<uintptr_t>(x) & 15) launch_up_wide_t<8, false, 4>(L, x, P, witem, worder, alist, H, wgrid, s);
        else if (near) launch_up_wide_plain_t<8, 4, true>(L, x, P, witem, worder, alist, H, wgrid, s);
        else launch_up_wide_plain_t<8, 4, false>(L, x, P, witem, worder, alist, H, wgrid, s);
        return;
    }
    if (up_tiny_supported(L)) {
        constexpr int TT = 4;
        const size_t lds = (S.sets ? 4 * 64 * 4 : (2 * (size_t)L.n_experts * 4 + 15) / 16 * 16) +
                           4 * (size_t)TT * 16 * kUpRowBytes;
        // as many workgroups per CU as LDS allows, at most the three that the registers allow
        // (squeezed into a fourth wavefront per SIMD's share of registers the kernel got slower)
        const int per_cu = std::max(1, std::min(3, (int)(160 * 1024 / lds)));
        TokenSets Sg = S;
        const int grid = S.sets ? sets_grid(Sg, L.n_experts, 64, 256 * per_cu)
                                : round_up((int)std::min<long long>(worst, 256 * per_cu), 8);
        const char* pk = static_cast<const char*>(L.packed);
        auto go = [&](auto kernel, std::once_flag& attr_once) {
            std::call_once(attr_once, [&] {  // kernel attributes: once per process, thread-safe
                (void)hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                          hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
            });
            launch_kernel(kernel, grid, 256, lds, s, (const __bf16*)x, (const __bf16*)(pk + P.wtinyf),
                          L.gated ? nullptr : (const __bf16*)L.b_up, witem, wfirst, NW, alist, (__bf16*)H, L.d_model,
                          L.n_experts, L.expert_size, L.act, h_row_neurons(L), Sg);
        };
        static std::once_flag once[6];
        if (S.sets) {  // (so few tokens that x is always near)
            if (L.gated) go(up_tiny_kernel<TT, true, true, true>, once[4]);
            else go(up_tiny_kernel<TT, false, true, true>, once[5]);
        } else if (L.gated) {
            if (near) go(up_tiny_kernel<TT, true, true, false>, once[0]);
            else go(up_tiny_kernel<TT, true, false, false>, once[1]);
        } else {
            if (near) go(up_tiny_kernel<TT, false, true, false>, once[2]);
            else go(up_tiny_kernel<TT, false, false, false>, once[3]);
        }
        return;
    }
    // (gated experts of 64 and plain ones of 128 are wide)
    auto go = [&](auto near_c, auto sets_c) {
        constexpr bool kNear = decltype(near_c)::value, kSets = decltype(sets_c)::value;
        if (L.gated) {
            // One workgroup per CU, for want of LDS beside the item table (more than 820 experts): then the registers that keep a second
            // one away are free.  992 tokens x 1627 experts of 32, d = 2048, all selected 1073 / 1002 us.  But by address padding rows
            // move as well: 737 x 1436 of 16, d = 1024, 60 % 183 / 238; 49 x 114 of 16, d = 3072 37.7 / 42.1.  Elsewhere two
            // share a CU: 4096 tokens x 256 of 32, d = 2048, 30 % 122 / 164; 300 tokens 34 / 57.
            if (up_lds(L, 4, 2, kSets) > 80 * 1024 && L.expert_size > 24) launch_up_t<2, true, 4, 2, false, true>(L, x, P, witem, wfirst, NW, alist, S, H, grid, s);
            else launch_up_t<2, true, 4, 2, kNear, false, kSets>(L, x, P, witem, wfirst, NW, alist, S, H, grid, s);
        } else if (mt == 2) {
            // 32-neuron rows: one staging buffer, three workgroups per CU
            const int grid3 = round_up((int)std::min<long long>(worst, 256 * 3), 8);
            launch_up_t<2, false, 4, 1, kNear, false, kSets>(L, x, P, witem, wfirst, NW, alist, S, H, grid3, s);
        } else {
            launch_up_t<4, false, 4, 2, kNear, false, kSets>(L, x, P, witem, wfirst, NW, alist, S, H, grid, s);
        }
    };
    if (S.sets) go(std::true_type{}, std::true_type{});  // (so few tokens that x is always near)
    else if (near) go(std::true_type{}, std::false_type{});
    else go(std::false_type{}, std::false_type{});
}

}  // namespace dmoe
