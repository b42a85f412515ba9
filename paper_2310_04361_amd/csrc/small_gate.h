// Pieces of the dynamic-k gate for at most 16 tokens (Sec. 3.4 Eq. 4): device functions shared by the
// stand-alone gate kernels (select.hip) and by the small-token forward (ffn_small.hip).
#pragma once

#include "dmoe_internal.h"
#include "mfma.h"

namespace dmoe {

// Maximum of token t's score row, by the wavefront that owns the token (lanes stride the experts).
__device__ __forceinline__ float small_row_max(const float* __restrict__ row, int E) {
    const int lane = threadIdx.x & 63;
    float mx = -INFINITY;
    for (int e = lane; e < E; e += 64) mx = fmaxf(mx, row[e]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
    return mx;
}

// The comparison of Eq. 4, exact: the fp64 product of two fp32 numbers is exact.
__device__ __forceinline__ bool small_keeps(float s, float tau, float mx) {
    return tau == 0.0f || (double)s >= (double)tau * (double)mx;
}

// T <= 16, one workgroup of 16 wavefronts: wavefront t = token t with lanes striding the experts,
// so the score row is read coalesced, the maximum is a wavefront reduction and a ballot IS a mask
// word.  The transpose to per-expert token sets (colmask) and counts then goes through LDS
// (mw[16][W]).
__device__ __forceinline__ void select_small_body(const float* __restrict__ scores,
                                                  uint64_t* __restrict__ mw,
                                                  uint64_t* __restrict__ mask,
                                                  int32_t* __restrict__ k_per_token,
                                                  int32_t* __restrict__ group_cnt,
                                                  uint64_t* __restrict__ colmask, int T, int E,
                                                  int W, float tau) {
    const int lane = threadIdx.x & 63, t = threadIdx.x >> 6;
    if (t < T) {
        const float* row = scores + (size_t)t * E;
        const float mx = small_row_max(row, E);
        int kt = 0;
        for (int w = 0; w < W; ++w) {
            const int e = 64 * w + lane;
            const bool keep = e < E && small_keeps(row[min(e, E - 1)], tau, mx);
            const uint64_t word = __ballot(keep);
            kt += __popcll(word);
            if (lane == 0) {
                mw[t * W + w] = word;
                mask[(size_t)t * W + w] = word;
            }
        }
        if (lane == 0 && k_per_token) k_per_token[t] = kt;
    }
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += 1024) {
        uint64_t col = 0;
        for (int tt = 0; tt < T; ++tt) col |= ((mw[tt * W + (e >> 6)] >> (e & 63)) & 1ull) << tt;
        group_cnt[e] = __popcll(col);
        if (colmask) colmask[e] = col;
    }
}

}  // namespace dmoe
