// Expert up-projection on 8-bit operands (weight format DMOE_W_FP8_E4M3_X8; the lower-precision
// layers of Appendix C, with the 8-bit floating-point format of the gfx950 matrix cores in place
// of int8).
//
//   quantise  one wavefront per token: the row maximum, the power-of-two scale
//             s_t = 2^ceil(log2(max / 448)), and every element rounded to the nearest E4M3 value
//             of x / s_t (ties to the even mantissa): by integer arithmetic on the fp32 bits where
//             the quantised value is wanted as well, by the hardware converter where only the
//             code is (it gives that arithmetic's code for every input it can meet here; see
//             e4m3_codes8).
//   up        the wide-expert kernel of ffn_bf16.hip (a workgroup owns 256 list rows of one
//             expert, the weights of a K block go through LDS once per workgroup, every
//             wavefront stages its own 64 gathered x rows) on v_mfma_f32_32x32x64_f8f6f4: a K block
//             is 128 wide, so per element of K the kernel gathers, stages and reads half the
//             bytes and issues a quarter of the matrix instructions at twice their rate.
//             The instruction adds the products of a 32-wide block with less than fp32
//             precision (measured: within 3e-4 of the block's largest product); the scales
//             s_t * w_scale enter once, on the accumulators, before the activation.
//
// Operand layout with both formats E4M3 (lane = 32h + c): the lane holds 32 bytes of row c of A, or column
// c of B; D as in the other 32 x 32 MFMAs.  Only "the same k in the same (h, byte) of A and B" matters
// for the sum, so lane half h of k-step s works on the k values 32 (2s + h) .. + 31 of the K block.
//   The packed weights are in tiles of 16 rows (lane = 16q + c), q = 2s + h:
//   wupx8[E][m_pad/16][d/128][64][32]: lane (q, c) of block (e, neuron tile mt, K block) holds
//   w[e][neuron_of_slot(mt, c)][128 kb + 32q ..], zero bytes for neurons >= m.
#include <algorithm>
#include <type_traits>

#include "pack.h"
#include "quantize.h"
#include "token_sets.h"

namespace dmoe {

namespace {

typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

constexpr int kScaleOne = 0x7f7f7f7f;   // E8M0 block scales of 1.0: the MFMA runs unscaled

// (lane (h, c) holds 32 k of row or column c; with unit scales any 32, as long as A and B agree)
__device__ __forceinline__ f32x16 mfma64(i32x8 a, i32x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, kScaleOne, 0, kScaleOne);
}

// ---- row-wise quantisation of x ----------------------------------------------------------------
__global__ __launch_bounds__(256) void quantize_x_kernel(const __bf16* __restrict__ x, int T, int d, const QuantX q) {
    const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (t < T) quantize_row(x, t, d, q.x8, q.xscale, q.xhat);
}

// ---- one-time packing -----------------------------------------------------------------------------
__global__ void pack_up_x8_kernel(const uint8_t* __restrict__ w, uint8_t* __restrict__ out, int E,
                                  int m, int d, int MT) {
    const size_t n = (size_t)E * MT * 2 * d;  // eight bytes each (see pack.h)
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; i < n; i += stride) {
        const int j8 = (int)(i & 15), c = (int)((i >> 4) & 15), q = j8 >> 2;  // bytes 8 j8 .. of row c: lane (q, c)
        const size_t block = i >> 8;
        size_t f = block;
        const int kb = (int)(f % (d / 128));
        f /= (d / 128);
        const int mt = (int)(f % MT), e = (int)(f / MT);
        const int neuron = neuron_of_slot(mt, c);
        const u8x8 v = neuron < m ? Packed8<uint8_t>::load(w, nullptr, 1, 0, e, ((size_t)e * m + neuron) * d + 128 * kb + 8 * j8)
                                  : u8x8{};
        *reinterpret_cast<u8x8*>(out + (block * 64 + 16 * q + c) * 32 + 8 * (j8 & 3)) = v;
    }
}

constexpr int kX8RowBytes = 144;   // 128 bytes of one x row + 16 bytes of bank skew

// ---- up-projection ----------------------------------------------------------------------------------
// Workgroup = (expert, 4 x 16*TT consecutive list rows); NT = neuron tiles of both branches.
// H8OUT: the hidden rows go out quantised for the 8-bit down-projection (DMOE_W_FP8_E4M3_A8):
// rounded to bf16 as usual, then the row's power-of-two scale and E4M3 codes, H8[row][16 MT] and
// hs8[row], instead of the bf16 row.
template <int MT, bool GATED, int TT, bool H8OUT>
__global__ __launch_bounds__(256, 2) void up_wide_x8_kernel(
    const uint8_t* __restrict__ x8, const float* __restrict__ xscale,
    const uint8_t* __restrict__ wupx, const uint8_t* __restrict__ wgatex,
    const float* __restrict__ w_scales, const __bf16* __restrict__ b_up,
    const int32_t* __restrict__ witem, const int2* __restrict__ worder,
    const int32_t* __restrict__ alist, __bf16* __restrict__ Hf, uint8_t* __restrict__ H8,
    uint8_t* __restrict__ hs8, int d, int E, int m, int act) {
    constexpr int BR = GATED ? 2 : 1;
    constexpr int KS = MT / 2;
    constexpr int NT = BR * MT;         // neuron tiles (2 KiB of weights each) per K block
    constexpr int NJ = NT / 2, TJ = TT / 2;  // tiles of the 32x32x64 MFMA: neurons, list rows
    constexpr int WR = TT * 16;         // rows per wavefront
    constexpr int UR = 4 * WR;          // rows per work item
    constexpr int NL = TT * 2;          // x load instructions per K block: 8 rows x 128 bytes each
    constexpr int NWL = NT / 2;         // weight load instructions per thread and K block
    static_assert(NT % 2 == 0, "the weights of a K block are copied 4 KiB at a time");
    extern __shared__ char smem[];
    char* wbuf = smem;                                            // [2][NT][64][32]
    const int lane = threadIdx.x & 63, h = lane >> 5, c = lane & 31, w = threadIdx.x >> 6;
    char* xs = smem + 2 * NT * 2048 + w * (WR * kX8RowBytes);     // [WR][kX8RowBytes], private
    float* sbias = reinterpret_cast<float*>(smem + 2 * NT * 2048 + 4 * (WR * kX8RowBytes));  // [2][MT * 16]
    const int NKB = d / 128;   // >= 2
    const int ld_row = lane >> 3, ld_piece = lane & 7;
    // this XCD's share of the items (workgroups are dealt round-robin to the 8 XCDs; the grid is a
    // multiple of 8), in the order laid out by the list fill
    const int xcd = blockIdx.x & 7, step = gridDim.x >> 3;
    const int total = xcd_first(witem[E], xcd + 1);
    const int first = xcd_first(witem[E], xcd);
    int j = first + (int)(blockIdx.x >> 3);
    if (j >= total) return;
    auto locate = [&](int jj, int& e, int& item) {
        const int2 v = worder[total - 1 - (jj - first)];  // (from the end: see up_wide_bf16_kernel)
        e = v.x;
        item = v.y;
    };
    // tokens of the x rows this lane fetches; padding rows (-1) read token 0 and produce H rows
    // that nobody merges
    auto rows_of = [&](int item, uint32_t (&xtok)[NL], bool& active) {
        const int32_t* tl = alist + (size_t)item * UR + w * WR;
        active = tl[0] >= 0;  // valid rows are a prefix
#pragma unroll
        for (int i = 0; i < NL; ++i) xtok[i] = (uint32_t)max(tl[ld_row + 8 * i], 0);
    };
    // The K block's weights are NT tiles of 2 KiB; this thread copies the 16-byte pieces
    // tid, tid + 256, ...: piece 256 i + tid belongs to tile 2i + (tid >> 7), the first MT of
    // which are up rows and the rest gate rows -- one base per matrix plus i times a stride.
    const uint32_t wlane = (uint32_t)((threadIdx.x >> 7) * NKB * 2048 + (threadIdx.x & 127) * 16);
    const size_t wstride = (size_t)2 * NKB * 2048;   // two neuron tiles on
    i32x4 xr[NL], wr[NWL];
    auto issue_w = [&](int i, int e, int kb) {
        const size_t we = (size_t)e * MT * NKB * 2048 + (size_t)kb * 2048 + wlane;
        wr[i] = *reinterpret_cast<const i32x4*>(((GATED && i >= MT / 2) ? wgatex : wupx) + we + (i % (MT / 2)) * wstride);
    };
    auto issue_x = [&](int i, const uint32_t (&xtok)[NL], int kb) {
        xr[i] = *reinterpret_cast<const i32x4*>(x8 + ((size_t)xtok[i] * (uint32_t)d + (uint32_t)(16 * ld_piece + 128 * kb)));
    };
    // in LDS a tile is two planes of 64 x 16 bytes, the first and the second half of every lane's 32
    // (read in one go at a lane stride of 32 bytes they would meet in the banks)
    char* const wdst = wbuf + (threadIdx.x >> 7) * 2048 + (threadIdx.x & 1) * 1024 + ((threadIdx.x & 127) >> 1) * 16;
    auto park_w = [&](int i, int buf) { *reinterpret_cast<i32x4*>(wdst + buf * NT * 2048 + i * 4096) = wr[i]; };
    auto park_x = [&](int i) {
        *reinterpret_cast<i32x4*>(xs + (ld_row + 8 * i) * kX8RowBytes + ld_piece * 16) = xr[i];
    };
    auto park_bias = [&](int e, int par) {  // plain experts: the item's biases, by neuron
        if (!GATED && (int)threadIdx.x < MT * 16)
            sbias[par * MT * 16 + threadIdx.x] =
                b_up ? (float)b_up[(size_t)e * m + min((int)threadIdx.x, m - 1)] : 0.0f;
    };

    // The K blocks of all the items of the workgroup form one stream, also across the end of an item: while
    // block k is multiplied, block k + 1 goes from registers to LDS and block k + 2 is requested, each
    // register as soon as it is free, between two MFMAs (see up_wide_bf16_kernel).  As phases in sequence and with
    // the 16x16x128 MFMA: 4096 tokens x 256 gated experts of 64, d = 2048, 37 % density 134 us, with this 115 (116 with
    // the 16x16x128 one, which holds 16 more operand registers: 128 neurons, d = 768: 53 against 48), with the
    // activations of mfma.h 107.
    int e, item;
    uint32_t xtok[NL];
    bool active;
    locate(j, e, item);
    rows_of(item, xtok, active);
#pragma unroll
    for (int i = 0; i < NWL; ++i) issue_w(i, e, 0);
#pragma unroll
    for (int i = 0; i < NL; ++i) issue_x(i, xtok, 0);
#pragma unroll
    for (int i = 0; i < NWL; ++i) {
        park_w(i, 0);
        issue_w(i, e, 1);
    }
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        park_x(i);
        issue_x(i, xtok, 1);
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
        const int32_t* tl = alist + (size_t)item * UR + w * WR;

        f32x16 acc[NJ][TJ];
#pragma unroll
        for (int nj = 0; nj < NJ; ++nj)
#pragma unroll
            for (int tj = 0; tj < TJ; ++tj)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[nj][tj][r] = 0.f;
        // One K block (see up_wide_bf16_kernel): multiplies block k, parks block k + 1 and requests
        // block k + 2 (weights of expert ew, rows xo, block kb2), between the MFMAs.
        auto block = [&](int ew, const uint32_t (&xo)[NL], int kb2, bool xp, bool xi) {
            if (active) {
                // k-step s of 64: lane (h, c) works on the 32 bytes 32 (2 s + h) .. of row c -- of the weights,
                // which are laid out for tiles of 16 rows, that is lane 16 (2 s + h) + c % 16 of tile c / 16
                const char* wsrc_l = wbuf + buf * NT * 2048 + (c >> 4) * 2048 + (16 * h + (c & 15)) * 16;
                const char* xsrc = xs + c * kX8RowBytes + h * 32;
                auto read_b = [&](int s, int tj) {
                    const char* p = xsrc + tj * 32 * kX8RowBytes + s * 64;
                    const i32x4 b0 = *reinterpret_cast<const i32x4*>(p), b1 = *reinterpret_cast<const i32x4*>(p + 16);
                    return i32x8{b0[0], b0[1], b0[2], b0[3], b1[0], b1[1], b1[2], b1[3]};
                };
                auto read_a = [&](int s, int nj) {
                    const char* p = wsrc_l + nj * 4096 + s * 512;
                    const i32x4 a0 = *reinterpret_cast<const i32x4*>(p), a1 = *reinterpret_cast<const i32x4*>(p + 1024);
                    return i32x8{a0[0], a0[1], a0[2], a0[3], a1[0], a1[1], a1[2], a1[3]};
                };
                i32x8 b[TJ], a_next = read_a(0, 0);
#pragma unroll
                for (int tj = 0; tj < TJ; ++tj) b[tj] = read_b(0, tj);
#pragma unroll
                for (int s = 0; s < 2; ++s) {
#pragma unroll
                    for (int nj = 0; nj < NJ; ++nj) {
                        const int q = s * NJ + nj;
                        const i32x8 a = a_next;
                        __builtin_amdgcn_sched_barrier(0);
                        if (q + 1 < 2 * NJ) a_next = read_a((q + 1) / NJ, (q + 1) % NJ);
#pragma unroll
                        for (int tj = 0; tj < TJ; ++tj) {
                            acc[nj][tj] = mfma64(a, b[tj], acc[nj][tj]);
                            __builtin_amdgcn_sched_barrier(0);
                            if (q == NJ - 1) b[tj] = read_b(1, tj);
                            if (tj == 0 && q >= 1 && q <= NWL) {
                                park_w(q - 1, buf ^ 1);
                                issue_w(q - 1, ew, kb2);
                            }
                            // (this block's rows are all read before its second k-step)
                            if (s == 1) {
#pragma unroll
                                for (int i = 0; i < NL; ++i)
                                    if (i * (TJ * NJ - 1) / NL == nj * TJ + tj) {
                                        park_x(i);
                                        issue_x(i, xo, kb2);
                                    }
                            }
                            __builtin_amdgcn_sched_barrier(0);
                        }
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
            block(e, xtok, kb + 2, false, false);
            lds_barrier();
            buf ^= 1;
        }
        // The next item's rows and this item's row scales are requested here, two blocks before
        // the end: vector loads return in order, so requested any later they would queue behind
        // the next item's first blocks, and any earlier their wait would hold up this item's start.
        uint32_t xtokn[NL];
        bool activen;
        rows_of(itemn, xtokn, activen);
        int tok_c[TJ];
#pragma unroll
        for (int tj = 0; tj < TJ; ++tj) tok_c[tj] = max(tl[32 * tj + c], 0);
        block(en, xtokn, 0, false, activen);    // block NKB - 2
        lds_barrier();
        buf ^= 1;
        float s_xr[TJ];
#pragma unroll
        for (int tj = 0; tj < TJ; ++tj) s_xr[tj] = xscale[tok_c[tj]];
        block(en, xtokn, 1, activen, activen);  // block NKB - 1; the next item's block 0 is parked
        park_bias(en, par ^ 1);
        lds_barrier();
        buf ^= 1;

        if (active) with_activation(act, [&](auto act_c) {
            constexpr int ACT = decltype(act_c)::value;
            // lane (h, c) of tile (nj, tj): list row 32 tj + c; registers 0..3 and 8..11 are the eight
            // neurons of piece 4 nj + h of the H row, 4..7 and 12..15 those of piece 4 nj + 2 + h.
            // The accumulators are sums of code products: times the row's scale and the
            // matrix's scale they are the pre-activations.
            const float s_up = w_scales[3 * e + 0], s_gate = w_scales[3 * e + 1];
#pragma unroll
            for (int tj = 0; tj < TJ; ++tj) {
                const float s_x = s_xr[tj];
                const size_t row = (size_t)item * UR + w * WR + 32 * tj + c;
                bf16x8 hv[KS][2];
#pragma unroll
                for (int nj = 0; nj < KS; ++nj) {
#pragma unroll
                    for (int half = 0; half < 2; ++half) {
                        const int n0 = 8 * (4 * nj + 2 * half + h);
#pragma unroll
                        for (int r = 0; r < 8; ++r) {
                            const int i = 4 * half + (r & 3) + 8 * (r >> 2);
                            float v;
                            if (GATED)
                                v = activate_fast(ACT, acc[NJ / 2 + nj][tj][i] * (s_x * s_gate)) * (acc[nj][tj][i] * (s_x * s_up));
                            else
                                v = activate_fast(ACT, acc[nj][tj][i] * (s_x * s_up) + sbias[par * MT * 16 + n0 + r]);
                            if (n0 + r >= m) v = 0.0f;
                            hv[nj][half][r] = (__bf16)v;
                        }
                    }
                }
                if (!H8OUT) {
                    __bf16* dst = Hf + row * (KS * 32) + 8 * h;
#pragma unroll
                    for (int nj = 0; nj < KS; ++nj)
#pragma unroll
                        for (int half = 0; half < 2; ++half)
                            *reinterpret_cast<bf16x8*>(dst + 32 * nj + 16 * half) = hv[nj][half];
                } else {
                    // the row's neurons are spread over the two lanes (h) of column c
                    float amax = 0.0f;
#pragma unroll
                    for (int nj = 0; nj < KS; ++nj)
#pragma unroll
                        for (int half = 0; half < 2; ++half)
#pragma unroll
                            for (int i = 0; i < 8; ++i) amax = fmaxf(amax, fabsf((float)hv[nj][half][i]));
                    amax = fmaxf(amax, __shfl_xor(amax, 32, 64));
                    int s_exp = 0;
                    if (amax > 0.0f && amax < INFINITY) {
                        int ex;
                        const float f = frexpf(amax, &ex);
                        s_exp = f <= 0.875f ? ex - 9 : ex - 8;
                        s_exp = min(max(s_exp, -100), 100);
                    }
#pragma unroll
                    for (int nj = 0; nj < KS; ++nj)
#pragma unroll
                        for (int half = 0; half < 2; ++half) {
                            float sv[8];
#pragma unroll
                            for (int i = 0; i < 8; ++i) sv[i] = ldexpf((float)hv[nj][half][i], -s_exp);
                            // piece 4 nj + 2 half + h of the row: eight neurons, one byte each
                            *reinterpret_cast<uint2*>(H8 + row * (KS * 32) + 8 * (4 * nj + 2 * half + h)) = e4m3_codes8(sv);
                        }
                    if (h == 0) hs8[row] = (uint8_t)(127 + s_exp);
                }
                // one list row at a time: interleaving more of them costs registers that the
                // requests in flight are using
                __builtin_amdgcn_sched_barrier(0);
            }
        });
        if (!more) break;
        j = jn;
        e = en;
        item = itemn;
        active = activen;
        par ^= 1;
#pragma unroll
        for (int i = 0; i < NL; ++i) xtok[i] = xtokn[i];
    }
}

// A lane's half (h) of the hidden row `row`, whose sums of code products are up[] and gate[]: times the row's scale and
// the matrix's they are the pre-activations.  H8OUT: quantised (see up_wide_x8_kernel, whose
// epilogue it is; called there it cost 8-bit layers of 4096 tokens 11 us by the registers that it moves).
template <int MT, bool GATED, bool H8OUT, int ACT>
__device__ __forceinline__ void hidden_row_x8(const f32x16 (&up)[MT / 2], const f32x16 (&gate)[MT / 2], float s_up, float s_gate,
                                              const float* bias, int m, int h, size_t row, __bf16* __restrict__ Hf,
                                              uint8_t* __restrict__ H8, uint8_t* __restrict__ hs8) {
    constexpr int KS = MT / 2;
    bf16x8 hv[KS][2];
#pragma unroll
    for (int nj = 0; nj < KS; ++nj) {
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int n0 = 8 * (4 * nj + 2 * half + h);
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const int i = 4 * half + (r & 3) + 8 * (r >> 2);
                float v;
                if (GATED) v = activate_fast(ACT, gate[nj][i] * s_gate) * (up[nj][i] * s_up);
                else v = activate_fast(ACT, up[nj][i] * s_up + bias[n0 + r]);
                if (n0 + r >= m) v = 0.0f;
                hv[nj][half][r] = (__bf16)v;
            }
        }
    }
    if (!H8OUT) {
        __bf16* dst = Hf + row * (KS * 32) + 8 * h;
#pragma unroll
        for (int nj = 0; nj < KS; ++nj)
#pragma unroll
            for (int half = 0; half < 2; ++half)
                *reinterpret_cast<bf16x8*>(dst + 32 * nj + 16 * half) = hv[nj][half];
        return;
    }
    // the row's neurons are spread over the two lanes (h) of its column
    float amax = 0.0f;
#pragma unroll
    for (int nj = 0; nj < KS; ++nj)
#pragma unroll
        for (int half = 0; half < 2; ++half)
#pragma unroll
            for (int i = 0; i < 8; ++i) amax = fmaxf(amax, fabsf((float)hv[nj][half][i]));
    amax = fmaxf(amax, __shfl_xor(amax, 32, 64));
    int s_exp = 0;
    if (amax > 0.0f && amax < INFINITY) {
        int ex;
        const float f = frexpf(amax, &ex);
        s_exp = f <= 0.875f ? ex - 9 : ex - 8;
        s_exp = min(max(s_exp, -100), 100);
    }
#pragma unroll
    for (int nj = 0; nj < KS; ++nj)
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            float sv[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) sv[i] = ldexpf((float)hv[nj][half][i], -s_exp);
            // piece 4 nj + 2 half + h of the row: eight neurons, one byte each
            *reinterpret_cast<uint2*>(H8 + row * (KS * 32) + 8 * (4 * nj + 2 * half + h)) = e4m3_codes8(sv);
        }
    if (h == 0) hs8[row] = (uint8_t)(127 + s_exp);
}

// The same for a small batch: one item of 256 rows per workgroup, D K blocks in flight, the item's tiles
// dealt to the wavefronts (see up_wide_sets_kernel in ffn_bf16.hip).
constexpr int kSetsTiles = 2;  // tiles of 32 rows a wavefront
template <int MT, bool GATED, bool H8OUT, int D>
__global__ __launch_bounds__(256, 1) void up_wide_sets_x8_kernel(
    const uint8_t* __restrict__ x8, const float* __restrict__ xscale, const uint8_t* __restrict__ wupx,
    const uint8_t* __restrict__ wgatex, const float* __restrict__ w_scales, const __bf16* __restrict__ b_up,
    __bf16* __restrict__ Hf, uint8_t* __restrict__ H8, uint8_t* __restrict__ hs8, int d, int E, int m, int act, const TokenSets S) {
    constexpr int BR = GATED ? 2 : 1;
    constexpr int KS = MT / 2;
    constexpr int NT = BR * MT;         // neuron tiles (2 KiB of weights each) per K block
    constexpr int NJ = NT / 2;          // ... of 32 rows
    constexpr int TJ = kSetsTiles;
    constexpr int WR = 32 * TJ;         // rows per wavefront
    constexpr int UR = 4 * WR;          // rows per work item
    constexpr int NWL = NT / 2;         // weight load instructions per thread and K block
    static_assert(D % 2 == 0 && NWL < 2 * NJ, "weight buffers alternate; copied within a block");
    extern __shared__ char smem[];
    char* wbuf = smem;                                            // [2][NT][64][32]
    const int lane = threadIdx.x & 63, h = lane >> 5, c = lane & 31;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    char* xs = smem + 2 * NT * 2048 + w * (WR * kX8RowBytes);     // [WR][kX8RowBytes], private
    float* sbias = reinterpret_cast<float*>(smem + 2 * NT * 2048 + 4 * (WR * kX8RowBytes));  // [MT * 16]
    int32_t* s_list = reinterpret_cast<int32_t*>(sbias + MT * 16) + WR * w;
    const int NKB = d / 128;   // a multiple of D
    const int ld_row = lane >> 3, ld_piece = lane & 7;
    const int e = blockIdx.x % E, slot = blockIdx.x / E;
    ExpertTokens tok;
    tok.load(S, E, e, 256, w == 0 && slot == 0);
    const int rows = tok.total - UR * slot;
    if (rows <= 0) return;
    // row 128 tj + 32 w + c of the item is row 32 tj + c of wavefront w
    tok.list<WR, UR>(UR * slot, s_list, [&](int r) { return ((r >> 5) & 3) == w ? 32 * (r >> 7) + (r & 31) : -1; });
    // (the copies of the weights: see up_wide_x8_kernel)
    const size_t we = (size_t)e * MT * NKB * 2048 + (threadIdx.x >> 7) * (size_t)NKB * 2048 + (threadIdx.x & 127) * 16;
    const size_t wstride = (size_t)2 * NKB * 2048;
    i32x4 wr[D][NWL];
    auto issue_w = [&](int i, int kb, i32x4& r) {
        r = *reinterpret_cast<const i32x4*>(((GATED && i >= MT / 2) ? wgatex : wupx) + we + (size_t)kb * 2048 + (i % (MT / 2)) * wstride);
    };
    char* const wdst = wbuf + (threadIdx.x >> 7) * 2048 + (threadIdx.x & 1) * 1024 + ((threadIdx.x & 127) >> 1) * 16;
    auto park_w = [&](int i, int buf, const i32x4& r) { *reinterpret_cast<i32x4*>(wdst + buf * NT * 2048 + i * 4096) = r; };
    if (!GATED && (int)threadIdx.x < MT * 16)  // plain experts: the biases, by neuron
        sbias[threadIdx.x] = b_up ? (float)b_up[(size_t)e * m + min((int)threadIdx.x, m - 1)] : 0.0f;
    const size_t row0 = (size_t)e * ((S.T + 255) / 256) * 256 + (size_t)slot * UR;

    // all of the item for a wavefront of NTJ tiles
    auto work = [&](auto ntj_c) {
        constexpr int NTJ = decltype(ntj_c)::value, NA = NTJ ? NTJ : 1;
        constexpr int NL = 4 * NTJ, NLA = NL ? NL : 1;  // x load instructions per K block: 8 rows x 128 bytes each
        uint32_t xtok[NLA];
#pragma unroll
        for (int i = 0; i < NL; ++i) xtok[i] = (uint32_t)max(s_list[ld_row + 8 * i], 0);  // (none: token 0, rows that nobody merges)
        float s_x[NA];
#pragma unroll
        for (int tj = 0; tj < NTJ; ++tj) s_x[tj] = xscale[max(s_list[32 * tj + c], 0)];
        i32x4 xr[D][NLA];
        auto issue_x = [&](int i, int kb, i32x4& r) {
            r = *reinterpret_cast<const i32x4*>(x8 + ((size_t)xtok[i] * (uint32_t)d + (uint32_t)(16 * ld_piece + 128 * kb)));
        };
        auto park_x = [&](int i, const i32x4& r) {
            *reinterpret_cast<i32x4*>(xs + (ld_row + 8 * i) * kX8RowBytes + ld_piece * 16) = r;
        };
#pragma unroll
        for (int b = 0; b < D; ++b) {
#pragma unroll
            for (int i = 0; i < NWL; ++i) issue_w(i, b, wr[b][i]);
#pragma unroll
            for (int i = 0; i < NL; ++i) issue_x(i, b, xr[b][i]);
        }
#pragma unroll
        for (int i = 0; i < NWL; ++i) {
            park_w(i, 0, wr[0][i]);
            issue_w(i, min(D, NKB - 1), wr[0][i]);
        }
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            park_x(i, xr[0][i]);
            issue_x(i, min(D, NKB - 1), xr[0][i]);
        }
        lds_barrier();
        f32x16 acc[NJ][NA];
#pragma unroll
        for (int nj = 0; nj < NJ; ++nj)
#pragma unroll
            for (int tj = 0; tj < NA; ++tj)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[nj][tj][r] = 0.f;
        // K block k = kb - D - 1, in weight buffer BUF; parks block k + 1 from its register set and requests block kb into it
        auto block = [&](auto buf_c, auto park_c, auto issue_c, i32x4 (&wk)[NWL], i32x4 (&xk)[NLA], int kb) {
            constexpr int BUF = decltype(buf_c)::value;
            constexpr bool PARK = decltype(park_c)::value, ISSUE = decltype(issue_c)::value;
            if constexpr (NTJ > 0) {
                const char* wsrc_l = wbuf + BUF * NT * 2048 + (c >> 4) * 2048 + (16 * h + (c & 15)) * 16;
                const char* xsrc = xs + c * kX8RowBytes + h * 32;
                auto read_b = [&](int s, int tj) {
                    const char* p = xsrc + tj * 32 * kX8RowBytes + s * 64;
                    const i32x4 b0 = *reinterpret_cast<const i32x4*>(p), b1 = *reinterpret_cast<const i32x4*>(p + 16);
                    return i32x8{b0[0], b0[1], b0[2], b0[3], b1[0], b1[1], b1[2], b1[3]};
                };
                auto read_a = [&](int s, int nj) {
                    const char* p = wsrc_l + nj * 4096 + s * 512;
                    const i32x4 a0 = *reinterpret_cast<const i32x4*>(p), a1 = *reinterpret_cast<const i32x4*>(p + 1024);
                    return i32x8{a0[0], a0[1], a0[2], a0[3], a1[0], a1[1], a1[2], a1[3]};
                };
                i32x8 b[NA], a_next = read_a(0, 0);
#pragma unroll
                for (int tj = 0; tj < NTJ; ++tj) b[tj] = read_b(0, tj);
#pragma unroll
                for (int s = 0; s < 2; ++s) {
#pragma unroll
                    for (int nj = 0; nj < NJ; ++nj) {
                        const int q = s * NJ + nj;
                        const i32x8 a = a_next;
                        __builtin_amdgcn_sched_barrier(0);
                        if (q + 1 < 2 * NJ) a_next = read_a((q + 1) / NJ, (q + 1) % NJ);
#pragma unroll
                        for (int tj = 0; tj < NTJ; ++tj) {
                            acc[nj][tj] = mfma64(a, b[tj], acc[nj][tj]);
                            __builtin_amdgcn_sched_barrier(0);
                            if (q == NJ - 1) b[tj] = read_b(1, tj);
                            if (tj == 0 && q >= 1 && q <= NWL) {
                                if (PARK) park_w(q - 1, BUF ^ 1, wk[q - 1]);
                                if (ISSUE) issue_w(q - 1, kb, wk[q - 1]);
                            }
                            // (this block's rows are all read before its second k-step)
                            if (s == 1) {
#pragma unroll
                                for (int i = 0; i < NL; ++i)
                                    if (i * (NTJ * NJ - 1) / NL == nj * NTJ + tj) {
                                        if (PARK) park_x(i, xk[i]);
                                        if (ISSUE) issue_x(i, kb, xk[i]);
                                    }
                            }
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    }
                }
            } else {
#pragma unroll
                for (int i = 0; i < NWL; ++i) {
                    if (PARK) park_w(i, BUF ^ 1, wk[i]);
                    if (ISSUE) issue_w(i, kb, wk[i]);
                }
            }
            lds_barrier();
        };
        const std::true_type yes;
        const std::false_type no;
        auto trip = [&](auto more_c, int kb0) {
            constexpr bool MORE = decltype(more_c)::value;
            auto one = [&](auto i_c) {
                constexpr int I = decltype(i_c)::value;
                constexpr int R = (I + 1) % D;
                // (past the end: the last block again, never used)
                if constexpr (MORE) block(std::integral_constant<int, I & 1>{}, yes, yes, wr[R], xr[R], min(kb0 + I + 1 + D, NKB - 1));
                else if constexpr (I + 1 < D) block(std::integral_constant<int, I & 1>{}, yes, no, wr[R], xr[R], 0);
                else block(std::integral_constant<int, I & 1>{}, no, no, wr[R], xr[R], 0);
            };
            one(std::integral_constant<int, 0>{});
            one(std::integral_constant<int, 1>{});
            if constexpr (D > 2) {
                one(std::integral_constant<int, 2>{});
                one(std::integral_constant<int, 3>{});
            }
        };
        int kb0 = 0;
        for (; kb0 + D < NKB; kb0 += D) trip(yes, kb0);
        trip(no, kb0);
        if constexpr (NTJ > 0) with_activation(act, [&](auto act_c) {
            const float s_up = w_scales[3 * e + 0], s_gate = w_scales[3 * e + 1];
#pragma unroll
            for (int tj = 0; tj < NTJ; ++tj) {
                f32x16 up[KS], gate[KS];
#pragma unroll
                for (int nj = 0; nj < KS; ++nj) {
                    up[nj] = acc[nj][tj];
                    gate[nj] = acc[GATED ? NJ / 2 + nj : nj][tj];
                }
                hidden_row_x8<MT, GATED, H8OUT, decltype(act_c)::value>(up, gate, s_x[tj] * s_up, s_x[tj] * s_gate, sbias, m, h,
                                                                        row0 + 128 * tj + 32 * w + c, Hf, H8, hs8);
                __builtin_amdgcn_sched_barrier(0);
            }
        });
    };
    // (every path has the same barriers)
    if (rows > 128 + 32 * w) work(std::integral_constant<int, TJ>{});
    else if (rows > 32 * w) work(std::integral_constant<int, 1>{});
    else work(std::integral_constant<int, 0>{});
}

template <int MT, bool GATED, int TT, bool H8OUT>
void launch_up_x8_t(const dmoe_layer& L, const PackedLayout& P, const uint8_t* x8,
                    const float* xscale, const int32_t* witem, const void* worder,
                    const int32_t* alist, void* H, uint8_t* H8, uint8_t* hs8, int grid,
                    hipStream_t s) {
    constexpr int NT = (GATED ? 2 : 1) * MT;
    const size_t lds = 2 * NT * 2048 + 4 * (size_t)TT * 16 * kX8RowBytes + 2 * MT * 16 * sizeof(float);
    static std::once_flag attr_once;  // kernel attributes: once per process, thread-safe
    std::call_once(attr_once, [&] {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&up_wide_x8_kernel<MT, GATED, TT, H8OUT>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    });
    const char* pk = static_cast<const char*>(L.packed);
    launch_kernel(up_wide_x8_kernel<MT, GATED, TT, H8OUT>, grid, 256, lds, s, x8, xscale,
                  (const uint8_t*)(pk + P.wupx8), (const uint8_t*)(pk + P.wgatex8),
                  (const float*)(pk + P.scales), (const __bf16*)L.b_up, witem, (const int2*)worder, alist,
                  (__bf16*)H, H8, hs8, L.d_model, L.n_experts, L.expert_size, L.act);
}

template <int MT, bool GATED, bool H8OUT, int D>
void launch_up_x8_sets_t(const dmoe_layer& L, const PackedLayout& P, const uint8_t* x8, const float* xscale, const TokenSets& S,
                         void* H, uint8_t* H8, uint8_t* hs8, hipStream_t s) {
    constexpr int NT = (GATED ? 2 : 1) * MT, TJ = kSetsTiles;
    const size_t lds = 2 * NT * 2048 + 4 * (size_t)TJ * 32 * kX8RowBytes + MT * 16 * sizeof(float) + 4 * 32 * TJ * sizeof(int32_t);
    static std::once_flag attr_once;  // kernel attributes: once per process, thread-safe
    std::call_once(attr_once, [&] {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&up_wide_sets_x8_kernel<MT, GATED, H8OUT, D>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    });
    const char* pk = static_cast<const char*>(L.packed);
    launch_kernel(up_wide_sets_x8_kernel<MT, GATED, H8OUT, D>, L.n_experts * div_up(S.T, 128 * TJ), 256, lds, s, x8, xscale,
                  (const uint8_t*)(pk + P.wupx8), (const uint8_t*)(pk + P.wgatex8), (const float*)(pk + P.scales),
                  (const __bf16*)L.b_up, (__bf16*)H, H8, hs8, L.d_model, L.n_experts, L.expert_size, L.act, S);
}

template <int MT, bool GATED, bool H8OUT>
void launch_up_x8_sets(const dmoe_layer& L, const PackedLayout& P, const uint8_t* x8, const float* xscale, const TokenSets& S,
                       void* H, uint8_t* H8, uint8_t* hs8, hipStream_t s) {
    if (L.d_model % 512) launch_up_x8_sets_t<MT, GATED, H8OUT, 2>(L, P, x8, xscale, S, H, H8, hs8, s);  // (whole trips)
    else launch_up_x8_sets_t<MT, GATED, H8OUT, 4>(L, P, x8, xscale, S, H, H8, hs8, s);
}

}  // namespace

void launch_quantize_x(const dmoe_layer& L, const void* x, int T, const QuantX& q, hipStream_t s) {
    LaunchTimer tm(kSlotQuantX, s);
    launch_kernel(quantize_x_kernel, div_up(T, 4), 256, 0, s, (const __bf16*)x, T, L.d_model, q);
}

void launch_pack_x8(const dmoe_layer& L, void* packed, hipStream_t s) {
    const PackedLayout P = packed_layout(L);
    char* pk = static_cast<char*>(packed);
    const int mt = m_pad_of(L.expert_size) / 16;
    launch_kernel(pack_up_x8_kernel, 2048, 256, 0, s, (const uint8_t*)L.w_up, (uint8_t*)(pk + P.wupx8),
                  L.n_experts, L.expert_size, L.d_model, mt);
    if (L.gated)
        launch_kernel(pack_up_x8_kernel, 2048, 256, 0, s, (const uint8_t*)L.w_gate,
                      (uint8_t*)(pk + P.wgatex8), L.n_experts, L.expert_size, L.d_model, mt);
}

void launch_up_x8(const dmoe_layer& L, const uint8_t* x8, const float* xscale, int T,
                  const int32_t* witem, const void* worder, const int32_t* alist, const TokenSets& S, void* H,
                  uint8_t* H8, uint8_t* hs8, hipStream_t s) {
    LaunchTimer tm(kSlotUp, s);
    const PackedLayout P = packed_layout(L);
    const int grid = round_up(
        (int)std::min<long long>((long long)T * L.n_experts / 256 + L.n_experts, 512), 8);
    if (S.sets) {
        if (L.gated && H8) launch_up_x8_sets<4, true, true>(L, P, x8, xscale, S, H, H8, hs8, s);
        else if (L.gated) launch_up_x8_sets<4, true, false>(L, P, x8, xscale, S, H, H8, hs8, s);
        else if (H8) launch_up_x8_sets<8, false, true>(L, P, x8, xscale, S, H, H8, hs8, s);
        else launch_up_x8_sets<8, false, false>(L, P, x8, xscale, S, H, H8, hs8, s);
        return;
    }
    if (L.gated && H8) launch_up_x8_t<4, true, 4, true>(L, P, x8, xscale, witem, worder, alist, H, H8, hs8, grid, s);
    else if (L.gated) launch_up_x8_t<4, true, 4, false>(L, P, x8, xscale, witem, worder, alist, H, nullptr, nullptr, grid, s);
    else if (H8) launch_up_x8_t<8, false, 4, true>(L, P, x8, xscale, witem, worder, alist, H, H8, hs8, grid, s);
    else launch_up_x8_t<8, false, 4, false>(L, P, x8, xscale, witem, worder, alist, H, nullptr, nullptr, grid, s);
}

}  // namespace dmoe
