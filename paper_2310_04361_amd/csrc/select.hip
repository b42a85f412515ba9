// Dynamic-k gate and per-expert bucketing (Sec. 3.4 Eq. 4; the metadata of Appendix C built by
// dedicated kernels instead of a full argsort).
//
// Data flow:  scores -> [tau_mask | topk_mask, count_from_mask] -> mask bits + per-(group, expert) counts
//             -> [scan_groups] prefix over token groups per expert
//             -> [fill] prefix over experts (list offsets, up-projection work items) and the
//                ascending per-expert token lists, compact and work-item aligned.
// A group is 64 consecutive tokens handled by one wavefront with lane = token; the 64x64 bit
// transpose between "experts of a token" and "tokens of an expert" is done with ballots.
#include "dmoe_internal.h"
#include "mfma.h"
#include "small_gate.h"

#include <type_traits>

namespace dmoe {

namespace {

constexpr int kWave = 64;

__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

// Inclusive prefix sum over the 64 lanes of a wavefront.
__device__ __forceinline__ int wave_inclusive_scan(int v) {
    const int lane = lane_id();
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        int n = __shfl_up(v, off, kWave);
        if (lane >= off) v += n;
    }
    return v;
}

// 64 x 64 bits over a wavefront: bit b of lane a becomes bit a of lane b.
__device__ __forceinline__ uint64_t transpose64(uint64_t v, int lane) {
    uint64_t out = 0;
#pragma unroll 8
    for (int b = 0; b < 64; ++b) {
        const uint64_t bal = __ballot((v >> b) & 1ull);
        if (lane == b) out = bal;
    }
    return out;
}

// The group's tokens that keep expert e: their number to row g of the table, or (sets, see token_sets.h) they
// themselves, 16 tokens a row, to the rows 4 g .. 4 g + 3 of it.
__device__ __forceinline__ void store_group(int32_t* __restrict__ cnt, int g, int T, int E, int e, uint64_t col, bool sets) {
    if (!sets) {
        cnt[(size_t)g * E + e] = __popcll(col);
        return;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (16 * (4 * g + i) < T) cnt[(size_t)(4 * g + i) * E + e] = (int32_t)((col >> (16 * i)) & 0xffffu);
}

// Per-group expert counts from the mask words: one wavefront per (group of 64 tokens, mask word),
// lane = token.  The ballot transpose gives, for every expert of the word, the 64-bit set of the
// group's tokens that keep it: its population count goes to group_cnt[g][e], the set itself to
// colmask[g][e] if wanted.
__global__ __launch_bounds__(256) void count_from_mask_kernel(const uint64_t* __restrict__ mask,
                                                              int32_t* __restrict__ group_cnt,
                                                              uint64_t* __restrict__ colmask,
                                                              int T, int E, int W, bool sets) {
    const int lane = lane_id();
    const int wave = (blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    const int NG = (T + kGroup - 1) / kGroup;
    const int g = wave / W, w = wave - g * W;
    if (g >= NG) return;  // uniform per wavefront
    const int t = g * kGroup + lane;
    // lane b: which tokens of the group keep expert 64w + b
    const uint64_t col = transpose64(t < T ? mask[(size_t)t * W + w] : 0ull, lane);
    const int e = 64 * w + lane;
    if (e < E) {
        store_group(group_cnt, g, T, E, e, col, sets);
        if (colmask) colmask[(size_t)g * E + e] = col;
    }
}

// Dynamic-k gate (Sec. 3.4 Eq. 4) with one wavefront per token and the lanes striding the
// experts: the score row is read coalesced and once (CH = ceil(E / 64) values per lane, all
// loads in flight together), the maximum is a wavefront reduction and a ballot IS a mask word.
// The per-group expert counts are then taken from the mask words by count_from_mask_kernel.
template <int CH>
__global__ __launch_bounds__(256) void tau_mask_kernel(const float* __restrict__ scores,
                                                       uint64_t* __restrict__ mask,
                                                       int32_t* __restrict__ k_per_token, int T,
                                                       int E, int W, float tau) {
    const int lane = lane_id();
    const int t = (blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    if (t >= T) return;  // uniform per wavefront
    const float* row = scores + (size_t)t * E;
    float v[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int e = 64 * c + lane;
        v[c] = e < E ? row[e] : -INFINITY;
    }
    float mx = -INFINITY;
#pragma unroll
    for (int c = 0; c < CH; ++c) mx = fmaxf(mx, v[c]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, kWave));
    const double thr = (double)tau * (double)mx;  // exact: at most 48 significant bits
    int kt = 0;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int e = 64 * c + lane;
        const bool keep = e < E && (tau == 0.0f || (double)v[c] >= thr);
        const uint64_t word = __ballot(keep);
        kt += __popcll(word);
        if (lane == 0 && c < W) mask[(size_t)t * W + c] = word;
    }
    if (lane == 0 && k_per_token) k_per_token[t] = kt;
}

// The same gate and the counts of its decisions in one launch: workgroup = 16 tokens, a wavefront each, and a row of
// the count table.  The mask words also go to LDS, from which a lane then counts its expert's bits.  What bounds
// it is reading the scores.
template <int CH>
__global__ __launch_bounds__(1024) void gate_counts_kernel(const float* __restrict__ scores, uint64_t* __restrict__ mask,
                                                           int32_t* __restrict__ cnt, int T, int E, int W, float tau, bool sets) {
    extern __shared__ uint64_t words[];  // [16][W]
    const int lane = lane_id();
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), t = blockIdx.x * 16 + w;
    if (t < T) {  // uniform
        const float* row = scores + (size_t)t * E;
        float v[CH];
#pragma unroll
        for (int c = 0; c < CH; ++c) v[c] = row[min(64 * c + lane, E - 1)];
        float mx = v[0];
#pragma unroll
        for (int c = 1; c < CH; ++c) mx = fmaxf(mx, v[c]);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, kWave));
        const double thr = (double)tau * (double)mx;  // exact: at most 48 significant bits
        const bool keep_all = tau == 0.0f;
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            const bool keep = (64 * c + lane < E) & (keep_all | ((double)v[c] >= thr));
            const uint64_t word = __ballot(keep);
            if (lane == 0 && c < W) {
                mask[(size_t)t * W + c] = word;
                words[w * W + c] = word;
            }
        }
    } else {
        for (int c = lane; c < W; c += kWave) words[w * W + c] = 0ull;
    }
    __syncthreads();
    for (int c = w; c < W; c += 16) {
        const int e = 64 * c + lane;
        int set = 0;
#pragma unroll
        for (int i = 0; i < 16; ++i) set |= ((int)(words[i * W + c] >> lane) & 1) << i;
        if (e < E) cnt[(size_t)blockIdx.x * E + e] = sets ? set : __popc(set);
    }
}

// Top-k gate (the conventional rule that Sec. 3.3 / 3.4 compare against): keep the k largest
// scores of each token, ties at the k-th value going to the lower expert index, so that exactly
// k are kept.  One wavefront per token with the lanes striding the experts (coalesced row read).
// The k-th largest value is found by a radix descent over the 32 bits of an order-preserving
// integer image of the scores (one ballot per 64 experts and bit); the experts equal to it are
// then admitted in index order until k are reached.  CH = ceil(E / 64) values per lane.
template <int CH>
__global__ __launch_bounds__(256) void topk_mask_kernel(const float* __restrict__ scores,
                                                        uint64_t* __restrict__ mask,
                                                        int32_t* __restrict__ k_per_token, int T,
                                                        int E, int W, int k) {
    const int lane = lane_id();
    const int t = (blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    if (t >= T) return;  // uniform per wavefront
    const float* row = scores + (size_t)t * E;
    uint32_t key[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int e = 64 * c + lane;
        // -0 and +0 compare equal, as they do as numbers; then flip so that unsigned order =
        // numeric order (sign bit set: all bits flipped, else only the sign bit)
        const uint32_t b = e < E ? __float_as_uint(row[e] + 0.0f) : 0x80000000u;  // padding: -0 -> below
        key[c] = (b & 0x80000000u) ? ~b : (b | 0x80000000u);
        if (e >= E) key[c] = 0u;  // below every real score
    }
    // largest x with #{key >= x} >= k
    uint32_t x = 0u;
    if (k > 0) {
        for (int bit = 31; bit >= 0; --bit) {
            const uint32_t cand = x | (1u << bit);
            int cnt = 0;
#pragma unroll
            for (int c = 0; c < CH; ++c) cnt += __popcll(__ballot(key[c] >= cand));
            if (cnt >= k) x = cand;  // uniform
        }
    }
    int above = 0;
#pragma unroll
    for (int c = 0; c < CH; ++c) above += __popcll(__ballot(key[c] > x));
    int need = k - above;  // how many of the experts equal to x are admitted, lowest index first
    int kt = 0;
#pragma unroll
    for (int c = 0; c < CH; ++c) {
        const int e = 64 * c + lane;
        const bool eq = key[c] == x && e < E;
        const uint64_t eqb = __ballot(eq);
        const bool take = eq && (int)__popcll(eqb & ((1ull << lane) - 1ull)) < need;
        const uint64_t word = __ballot(k > 0 && ((key[c] > x && e < E) || take));
        need -= min(need, (int)__popcll(eqb));
        if (c < W) kt += __popcll(word);
        if (lane == 0 && c < W) mask[(size_t)t * W + c] = word;
    }
    if (lane == 0 && k_per_token) k_per_token[t] = kt;
}

__global__ __launch_bounds__(1024) void select_small_kernel(const float* __restrict__ scores,
                                                            uint64_t* __restrict__ mask,
                                                            int32_t* __restrict__ k_per_token,
                                                            int32_t* __restrict__ group_cnt,
                                                            uint64_t* __restrict__ colmask, int T,
                                                            int E, int W, float tau) {
    extern __shared__ uint64_t mw[];  // [16][W]
    select_small_body(scores, mw, mask, k_per_token, group_cnt, colmask, T, E, W, tau);
}

// the same gate for every layer of a group (blockIdx.z = layer), each with its own tau
__global__ __launch_bounds__(1024) void select_small_group_kernel(const SmallGroup G, int T, int E,
                                                                  int W) {
    extern __shared__ uint64_t mw[];  // [16][W]
    const SmallMod& M = G.m[blockIdx.z];
    select_small_body(M.scores, mw, M.mask, nullptr, M.group_cnt, M.colmask, T, E, W, M.tau);
}

// Caller-supplied lists -> mask words and group counts, in three launches (clear, scatter, finish) and in one of two
// ways, which the number of positions on the device decides:
//   by bytes: a byte per (expert, token), bytes[E][Tp]; an expert's positions go to one row of workgroups.  No atomics, but
//   all E T bytes are written and read.
//   by bits: an atomic OR per position into the mask words, lines that all XCDs write, and a count afterwards.
// Entries outside [0, T) are dropped, duplicates meet in one byte or bit.  Bits / bytes, us: 605000 positions of 24
// experts at 50432 tokens 19.0 / 12.5, 300000 of 2048 experts at 2000 tokens 25 / 13.6; 2048 experts, 50432 tokens, 0.05 / 0.3 /
// 1 % of E T: 34 / 46 / 75 and 48 / 49 / 58; 256 experts, 66000 tokens, 0.3 / 1 / 3 %: 14 / 19 / 35 and 21 / 21 / 21.
// CHOOSE: up to bits_max positions go by bits, and all where there are no bytes; otherwise all go by bytes.
template <bool CHOOSE>
__device__ __forceinline__ bool lists_by_bytes(const int32_t* offsets, int T, int E, const void* bytes, long long bits_max) {
    if (!CHOOSE) return true;
    return bytes && min((long long)offsets[E], (long long)T * E) - max((long long)offsets[0], 0ll) > bits_max;
}

template <bool CHOOSE>
__global__ __launch_bounds__(256) void lists_clear_kernel(const int32_t* __restrict__ offsets, int T, int E,
                                                          uint64_t* __restrict__ mask, size_t n_mask,
                                                          uint64_t* __restrict__ bytes, size_t n_bytes, long long bits_max) {
    const bool by_bytes = lists_by_bytes<CHOOSE>(offsets, T, E, bytes, bits_max);
    uint64_t* p = by_bytes ? bytes : mask;
    const size_t n = by_bytes ? n_bytes : n_mask, stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = 0ull;
}

// blockIdx.y = expert (by bytes)
template <bool CHOOSE>
__global__ __launch_bounds__(256) void lists_scatter_kernel(const int32_t* __restrict__ offsets,
                                                            const int32_t* __restrict__ lists, int T, int E, int W,
                                                            int Tp, uint8_t* __restrict__ bytes,
                                                            unsigned long long* __restrict__ mask, long long bits_max) {
    const long long cap = (long long)T * E, begin = max((long long)offsets[0], 0ll), end = min((long long)offsets[E], cap);
    if (lists_by_bytes<CHOOSE>(offsets, T, E, bytes, bits_max)) {
        const int e = blockIdx.y;
        const long long first = max(begin, (long long)offsets[e]), last = min(end, (long long)offsets[e + 1]);
        uint8_t* row = bytes + (size_t)e * Tp;
        constexpr int kN = 8;  // positions in flight: one expert may have most of them
        const long long stride = (long long)gridDim.x * 256;
        for (long long p = first + (long long)blockIdx.x * 256 + threadIdx.x; p < last; p += kN * stride) {
            int t[kN];
#pragma unroll
            for (int k = 0; k < kN; ++k) t[k] = lists[min(p + k * stride, last - 1)];
#pragma unroll
            for (int k = 0; k < kN; ++k)
                if (p + k * stride < last && (unsigned)t[k] < (unsigned)T) row[t[k]] = 1;
        }
        return;
    }
    const long long stride = (long long)gridDim.x * gridDim.y * 256;
    for (long long p = begin + (long long)(blockIdx.y * gridDim.x + blockIdx.x) * 256 + threadIdx.x; p < end; p += stride) {
        // expert of position p: the last e with offsets[e] <= p
        int lo = 0, hi = E;  // answer in [lo, hi)
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if ((long long)offsets[mid] <= p) lo = mid; else hi = mid;
        }
        if (p >= (long long)offsets[lo + 1]) continue;  // non-monotone offsets: drop
        const int t = lists[p];
        if ((unsigned)t < (unsigned)T)
            atomicOr(&mask[(size_t)t * W + (lo >> 6)], 1ull << (lo & 63));
    }
}

// One wavefront per (group of 64 tokens, mask word).  By bytes: lane b turns the group's 64 bytes of expert 64 w + b
// into its 64-bit token set, and the ballots over a token's bit of all the sets are the mask words.  By bits: the other
// way round (count_from_mask_kernel).
template <bool CHOOSE>
__global__ __launch_bounds__(256) void lists_finish_kernel(const int32_t* __restrict__ offsets,
                                                           const uint8_t* __restrict__ bytes, int T, int E, int W,
                                                           int Tp, uint64_t* __restrict__ mask,
                                                           int32_t* __restrict__ group_cnt, bool sets, long long bits_max) {
    const int lane = lane_id();
    const int wave = (blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    const int NG = (T + kGroup - 1) / kGroup;
    const int g = wave / W, w = wave - g * W;
    if (g >= NG) return;  // uniform per wavefront
    const int e = 64 * w + lane, t = g * kGroup + lane;
    if (!lists_by_bytes<CHOOSE>(offsets, T, E, bytes, bits_max)) {
        const uint64_t set = transpose64(t < T ? mask[(size_t)t * W + w] : 0ull, lane);
        if (e < E) store_group(group_cnt, g, T, E, e, set, sets);
        return;
    }
    uint64_t set = 0;
    if (e < E) {
        const ulonglong2* src = reinterpret_cast<const ulonglong2*>(bytes + (size_t)e * Tp + g * kGroup);
        ulonglong2 v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = src[i];
#pragma unroll
        for (int i = 0; i < 4; ++i) {  // eight bytes of 0 or 1 -> eight bits
            set |= ((v[i].x * 0x0102040810204080ull) >> 56) << (16 * i);
            set |= ((v[i].y * 0x0102040810204080ull) >> 56) << (16 * i + 8);
        }
        store_group(group_cnt, g, T, E, e, set, sets);
    }
    const uint64_t word = transpose64(set, lane);
    if (t < T) mask[(size_t)t * W + w] = word;
}

// The same in one launch, for so few positions that every workgroup may look at all those of its experts: workgroup = 256 tokens
// and one mask word (64 experts), whose bits it collects in LDS.
constexpr int kListsTokens = 256;
__global__ __launch_bounds__(1024) void lists_small_kernel(const int32_t* __restrict__ offsets, const int32_t* __restrict__ lists,
                                                           int T, int E, int W, uint64_t* __restrict__ mask,
                                                           int32_t* __restrict__ group_cnt, uint64_t* __restrict__ colmask, bool sets) {
    __shared__ uint32_t bits[64][kListsTokens / 32 + 1];  // [expert][32 tokens]
    __shared__ int s_off[128];  // from ne on: the end
    __shared__ int s_ordered;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int w = blockIdx.y, e0 = 64 * w, ne = min(64, E - e0), t0 = blockIdx.x * kListsTokens;
    if (tid == 0) s_ordered = 1;
    for (int i = tid; i < 64 * (kListsTokens / 32 + 1); i += 1024) (&bits[0][0])[i] = 0u;
    const long long cap = (long long)T * E, begin = max((long long)offsets[0], 0ll), end = min((long long)offsets[E], cap);
    if (tid < 128) s_off[tid] = (int)min(max((long long)offsets[e0 + min(tid, ne)], begin), max(begin, end));
    __syncthreads();
    if (tid < ne && s_off[tid] > s_off[tid + 1]) s_ordered = 0;
    __syncthreads();
    constexpr int kN = 8;  // positions in flight
    auto mark = [&](int e, int t) {
        if ((unsigned)t < (unsigned)T && (unsigned)(t - t0) < (unsigned)kListsTokens)
            atomicOr(&bits[e][(t - t0) >> 5], 1u << ((t - t0) & 31));
    };
    if (s_ordered) {  // the positions of all the experts as one range
        const int last = s_off[ne];
        for (int p = s_off[0] + tid; p < last; p += kN * 1024) {
            int t[kN];
#pragma unroll
            for (int k = 0; k < kN; ++k) t[k] = lists[min(p + k * 1024, last - 1)];
            int e[kN] = {};  // their experts: the last with s_off[e] <= position, all searches side by side
#pragma unroll
            for (int step = 32; step > 0; step >>= 1)
#pragma unroll
                for (int k = 0; k < kN; ++k) e[k] += s_off[e[k] + step] <= p + k * 1024 ? step : 0;
#pragma unroll
            for (int k = 0; k < kN; ++k)
                if (p + k * 1024 < last) mark(e[k], t[k]);
        }
    } else {  // offsets that fall: expert by expert
        for (int e = wave; e < ne; e += 16)
            for (int p = s_off[e] + lane; p < s_off[e + 1]; p += 64) mark(e, lists[p]);
    }
    __syncthreads();
    if (wave >= kListsTokens / kGroup) return;
    const int g = t0 / kGroup + wave, t = g * kGroup + lane;  // wavefront = group of 64 tokens
    if (g * kGroup >= T) return;  // uniform
    const uint64_t set = bits[lane][2 * wave] | (uint64_t)bits[lane][2 * wave + 1] << 32;  // lane = expert
    if (lane < ne) {
        store_group(group_cnt, g, T, E, e0 + lane, set, sets);
        if (colmask) colmask[(size_t)g * E + e0 + lane] = set;
    }
    const uint64_t word = transpose64(set, lane);
    if (t < T) mask[(size_t)t * W + w] = word;
}

// One wavefront per expert: exclusive prefix sum of group_cnt[.][e] over the groups, in place;
// row NG receives the total.  With sub != nullptr the counts of group g are read as the sum of
// the rows split * g .. split * g + split - 1 of sub (n_sub rows in all).
__global__ __launch_bounds__(256) void scan_groups_kernel(int32_t* __restrict__ group_cnt, int NG,
                                                          int E, const int32_t* __restrict__ sub,
                                                          int split, int n_sub) {
    const int lane = lane_id();
    const int e = (blockIdx.x * blockDim.x + threadIdx.x) / kWave;
    if (e >= E) return;
    // eight chunks of 64 groups per pass with all their loads in flight together (one memory round
    // trip per 512 groups instead of one per 64)
    // (the parts of a group too: one after the other they were 1.4 of 5.6 us, 4096 tokens, 256 and 512 experts)
    int carry = 0;
    for (int base = 0; base < NG; base += 8 * kWave) {
        int v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int g = base + k * kWave + lane;
            v[k] = 0;
            if (base + k * kWave >= NG) continue;  // uniform
            if (sub) {
                int part[4];  // (split is at most 4)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    part[j] = sub[(size_t)min(split * g + min(j, split - 1), n_sub - 1) * E + e];
#pragma unroll
                for (int j = 0; j < 4; ++j) v[k] += j < split && split * g + j < n_sub ? part[j] : 0;
            } else {
                v[k] = g < NG ? group_cnt[(size_t)g * E + e] : 0;
            }
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int g = base + k * kWave + lane;
            if (base + k * kWave >= NG) break;  // uniform
            const int incl = wave_inclusive_scan(v[k]);
            if (g < NG) group_cnt[(size_t)g * E + e] = carry + incl - v[k];
            carry += __shfl(incl, kWave - 1, kWave);
        }
    }
    if (lane == 0) group_cnt[(size_t)NG * E + e] = carry;
}

// Prefix sums over the experts plus the list fill, one launch.
//
// Every workgroup first redoes the (tiny) scan over the per-expert totals in LDS:
//   s_off[e]  = start of expert e in the compact lists (offsets),
//   s_item[e] = first up-projection work item of expert e when an item covers rows_per_item list
//               rows; s_item[E] = number of items.
// Workgroup 0 also publishes counts / offsets / item_start.
// Then one wavefront per group of 64 tokens (lane = token) turns mask words into list entries:
// for every expert, the lanes whose token keeps it write their token id at
//   lists[offsets[e] + group_off[g][e] + rank]                 compact, ascending (caller-visible)
//   alist[item_start[e] * rows_per_item + group_off[g][e] + rank]   aligned copy for the kernels
// where rank counts the group's keepers below the lane.  In the aligned copy every expert starts
// on a work-item boundary -- the same indexing as the rows of H -- and the slack behind its last
// token holds -1.
//
// FOLD: the scan over the token groups happens here as well.  The raw counts come as `sub_rows`
// rows of sub (split rows per group, as the router wrote them); every workgroup adds the rows up
// for itself -- at most kFoldRows independent loads per expert -- and workgroup (g, 0) publishes
// row g of group_off.  With few groups that is much cheaper than a kernel of its own in front of
// this one: 128 x 24 experts, 512 tokens: 5.5 + 6.1 us as two launches.
//
// MANY (more than 256 experts): a thread has several experts, so the chains that a thread goes through one after
// the other bound the launch: the loads of up to four experts are in flight together, and the window table takes
// one scan over the threads' sums instead of one, with two barriers, per 256 experts.  2048 experts, 128 / 300
// tokens 18.1 / 18.5 -> 12.4 / 12.5 us, 1000 tokens 13.6 -> 11.8; 512 experts, 128 / 512 tokens 8.4 / 10.3 -> 7.5 / 9.4.
// With fewer experts the same code was 0.3 us slower (its staging through LDS).
template <bool FOLD, bool MANY>
__global__ __launch_bounds__(256) void fill_lists_kernel(
    const uint64_t* __restrict__ mask, int T, int E, int W, int32_t* __restrict__ group_off,
    const int32_t* __restrict__ sub, int split, int sub_rows,
    int row_shift, int32_t* __restrict__ counts, int32_t* __restrict__ offsets,
    int32_t* __restrict__ item_start, int32_t* __restrict__ lists, int32_t* __restrict__ alist,
    int GW, int NW, int32_t* __restrict__ witem, int32_t* __restrict__ wfirst,
    int2* __restrict__ worder, int by_experts) {
    extern __shared__ int32_t sm[];
    int32_t* s_off = sm;                 // [E + 1]
    int32_t* s_item = sm + (E + 1);      // [E + 1]
    int32_t* s_tot = s_item + (E + 1);   // [E] tokens per expert
    int32_t* s_pre = s_tot + E;          // FOLD: [E] of them in the groups before this one
    int32_t* s_lo = s_pre + E;           // FOLD: [E] ... before this workgroup's window
    int32_t* s_hi = s_lo + E;            // FOLD: [E] ... before its end
    // [E] items of the window, in the place of what they come from: the totals are afterwards the differences of
    // s_off.  (In a place of their own, a fourth array, 2048 experts leave LDS for one workgroup less per CU: 20000 tokens
    // 45.3 us against 34.7, 4096 experts 133.9 against 104.8.)
    int32_t* s_n = FOLD ? s_lo : s_tot;
    __shared__ int s_part[2][4];
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const int NG = (T + kGroup - 1) / kGroup;
    const int g = blockIdx.x, wdx = blockIdx.x;
    const int rows_per_item = 1 << row_shift;

    // Totals to LDS (coalesced, the loads of eight experts -- FOLD: of sixteen to 32 counts -- in flight
    // together), then every thread adds up K consecutive experts and ONE scan runs over the
    // threads: taking 256 experts at a time with a scan each, this was 15 of 20 us for 2048.
    const int K = (E + 255) >> 8, e_first = tid * K;
    if (FOLD) {
        const int n_pre = g * split, n_lo = wdx * GW * split, n_hi = (wdx * GW + GW) * split;
        auto add_up = [&](auto experts, auto rows) {
            constexpr int NE = decltype(experts)::value, NR = decltype(rows)::value;
            for (int e0 = tid; e0 < E; e0 += NE * 256) {
                int cnt[NE] = {}, pre[NE] = {}, lo[NE] = {}, hi[NE] = {};
                for (int r0 = 0; r0 < sub_rows; r0 += NR) {
                    int v[NR][NE];
#pragma unroll
                    for (int j = 0; j < NR; ++j)
#pragma unroll
                        for (int k = 0; k < NE; ++k)
                            v[j][k] = r0 + j < sub_rows ? sub[(size_t)(r0 + j) * E + min(e0 + 256 * k, E - 1)] : 0;  // (uniform)
#pragma unroll
                    for (int j = 0; j < NR; ++j) {
                        const int r = r0 + j;
#pragma unroll
                        for (int k = 0; k < NE; ++k) {
                            cnt[k] += v[j][k];
                            pre[k] += r < n_pre ? v[j][k] : 0;
                            lo[k] += r < n_lo ? v[j][k] : 0;
                            hi[k] += r < n_hi ? v[j][k] : 0;
                        }
                    }
                }
#pragma unroll
                for (int k = 0; k < NE; ++k) {
                    const int e = e0 + 256 * k;
                    if (e >= E) break;
                    s_tot[e] = cnt[k];
                    s_pre[e] = pre[k];
                    s_lo[e] = lo[k];
                    s_hi[e] = hi[k];
                    if (blockIdx.y == 0) {
                        group_off[(size_t)g * E + e] = pre[k];
                        if (g == NG - 1) group_off[(size_t)NG * E + e] = cnt[k];
                    }
                }
            }
        };
        if (!MANY) add_up(std::integral_constant<int, 1>{}, std::integral_constant<int, 16>{});
        else if (E <= 512) add_up(std::integral_constant<int, 2>{}, std::integral_constant<int, 8>{});
        else add_up(std::integral_constant<int, 4>{}, std::integral_constant<int, 8>{});
    } else {
        for (int e0 = tid; e0 < E; e0 += 8 * 256) {
            int v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = group_off[(size_t)NG * E + min(e0 + 256 * k, E - 1)];
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (e0 + 256 * k < E) s_tot[e0 + 256 * k] = v[k];
        }
    }
    __syncthreads();
    int sum = 0, isum = 0;
    for (int k = 0; k < K && e_first + k < E; ++k) {
        const int cnt = s_tot[e_first + k];
        s_off[e_first + k] = sum;
        s_item[e_first + k] = isum;
        sum += cnt;
        isum += (cnt + rows_per_item - 1) >> row_shift;
    }
    {
        const int incl = wave_inclusive_scan(sum), iincl = wave_inclusive_scan(isum);
        if (lane == kWave - 1) {
            s_part[0][wave] = incl;
            s_part[1][wave] = iincl;
        }
        __syncthreads();
        int before = incl - sum, ibefore = iincl - isum;
        for (int w2 = 0; w2 < wave; ++w2) {
            before += s_part[0][w2];
            ibefore += s_part[1][w2];
        }
        for (int k = 0; k < K && e_first + k < E; ++k) {
            s_off[e_first + k] += before;
            s_item[e_first + k] += ibefore;
        }
        if (tid == 255) {  // the last thread: everything up to E
            s_off[E] = before + sum;
            s_item[E] = ibefore + isum;
        }
    }
    __syncthreads();

    // gridDim.y workgroups share the mask words of one group; those with y = 0 also do the
    // per-launch work
    const bool first_y = blockIdx.y == 0;
    if (blockIdx.x == 0 && first_y) {
        for (int e = tid; e <= E; e += 256) {
            offsets[e] = s_off[e];
            if (item_start) item_start[e] = s_item[e];
            if (e < E && counts) counts[e] = s_tot[e];
        }
    }
    // Window table for the up-projection (block w lays out window w = GW consecutive groups):
    // the work items of expert e that window w works on are wfirst[w][e] .. + n (those whose
    // rows mostly belong to tokens of the window); witem[w][e] is the exclusive prefix of n over
    // the experts.
    if (witem && wdx < NW && first_y) {
        const int32_t* r_lo = group_off + (size_t)(wdx * GW) * E;
        const int32_t* r_hi = group_off + (size_t)min(wdx * GW + GW, NG) * E;
        auto items_of = [&](int e, int& first) {
            // the expert's items are dealt to the windows in proportion to its rows there
            // (cutting at ceil(row / rows_per_item) would hand every expert's first,
            // rounded-up item to window 0 and overload its XCD)
            // (in double: exact far beyond any real size, monotone in the row, and identical for
            // the shared boundary of two neighbouring windows -- a 64-bit integer division
            // costs hundreds of instructions)
            const int cnt = s_tot[e];
            const int lo = FOLD ? s_lo[e] : r_lo[e], hi = FOLD ? s_hi[e] : r_hi[e];
            const int items = (cnt + rows_per_item - 1) >> row_shift;
            const double scale = cnt ? (double)items / (double)cnt : 0.0;
            const int k0 = min(items, (int)((double)lo * scale + 0.5));
            const int k1 = hi >= cnt ? items : min(items, (int)((double)hi * scale + 0.5));
            first = s_item[e] + k0;
            return k1 - k0;
        };
        int n = 0;  // items of the thread's own experts
        if (MANY) {
#pragma unroll 4
            for (int e = tid; e < E; e += 256) {
                int first;
                s_n[e] = items_of(e, first);
                wfirst[(size_t)wdx * E + e] = first;
            }
            __syncthreads();
            for (int k = 0; k < K && e_first + k < E; ++k) n += s_n[e_first + k];
        } else if (tid < E) {
            int first;
            n = items_of(tid, first);
            wfirst[(size_t)wdx * E + tid] = first;
        }
        const int incl = wave_inclusive_scan(n);
        __syncthreads();  // s_part from the scan above has been read
        if (lane == kWave - 1) s_part[0][wave] = incl;
        __syncthreads();
        int before = incl - n;
        for (int w2 = 0; w2 < wave; ++w2) before += s_part[0][w2];
        if (MANY) {
            for (int k = 0; k < K && e_first + k < E; ++k) {
                witem[(size_t)wdx * (E + 1) + e_first + k] = before;
                before += s_n[e_first + k];
            }
        } else {
            if (tid < E) witem[(size_t)wdx * (E + 1) + tid] = before;
            before += n;
        }
        if (tid == 255) witem[(size_t)wdx * (E + 1) + E] = before;
    }
    if (alist) {  // -1 behind each expert's last token, up to its next work-item boundary
        const int n = E << row_shift, stride = gridDim.x * gridDim.y * 256;
        for (int i = (blockIdx.y * gridDim.x + blockIdx.x) * 256 + tid; i < n; i += stride) {
            const int e = i >> row_shift;
            const int p = (s_item[e] << row_shift) + s_off[e + 1] - s_off[e] + (i & (rows_per_item - 1));
            if (p < s_item[e + 1] << row_shift) alist[p] = -1;
        }
    }

    // Order of the wide up-projection's work items.  XCD k takes the items k N / 8 .. of the order
    // below; the workgroups of an XCD walk them side by side, so what those in flight share comes
    // out of its L2.  Items are ordered by where their tokens lie (item i of an expert's n covers
    // about the tokens i T / n .. (i + 1) T / n), so that the experts working on one stretch of
    // tokens gather the same x rows: over all items (every XCD works on its own stretch with all
    // the experts), or, by_experts, over the items of the XCD's own share of the experts (each
    // XCD goes over all the tokens, but no two read the same weights).
    // Where the workgroups have three items and more each, three neighbouring items of an expert count as one of three
    // times the size: they run side by side and share the weights.  Up-projection, one by one / in threes: 512 gated
    // experts of 64, d = 1024, 4096 / 8192 tokens 189 / 182 and 228 / 219 us, 8-bit 125 / 119 and 147 / 139; 400 experts of 128,
    // d = 2048, 4096 tokens 334 / 322; 256 gated experts of 64, d = 2048, 4096 tokens 196 / 194 (8-bit 111 / 111) with 1.00 GB
    // from beyond the L2 instead of 1.05 (8-bit 0.48 instead of 0.56); 25 more sizes within 2 % either way.  The order itself
    // takes 0.3 to 0.7 us longer to work out.  With 1.6 to 2.2 items the last ones run longer (pairs: 94 us instead
    // of 90), and where all XCDs have all the experts (50432 tokens x 24 of 128) pairs were 1 % slower.
    if (worder) {
        const int N = s_item[E], run = by_experts && N >= 3 * 512 ? 3 : 1;
        auto expert_of = [&](int n) {  // the last e with s_item[e] <= n
            int lo = 0, hi = E;
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (s_item[mid] <= n) lo = mid; else hi = mid;
            }
            return lo;
        };
        // one wavefront per item, its lanes over the experts that share the item's range
        const int waves = gridDim.x * gridDim.y * 4;
        for (int n = (blockIdx.y * gridDim.x + blockIdx.x) * 4 + wave; n < N; n += waves) {
            int lo = 0, hi = N;
            if (by_experts) {
                int k = 0;
                while (k < 7 && n >= xcd_first(N, k + 1)) ++k;
                lo = xcd_first(N, k);
                hi = xcd_first(N, k + 1);
            }
            // (the three searches are one walk of three lanes)
            const int found = expert_of(lane == 0 ? n : (lane == 1 ? lo : hi - 1));
            const int e = __shfl(found, 0, kWave), e0 = __shfl(found, 1, kWave), e1 = __shfl(found, 2, kWave);
            const double ne = (double)((s_item[e + 1] - s_item[e] + run - 1) / run), key = (double)(2 * ((n - s_item[e]) / run) + 1);
            const double inv = 0.5 / ne;
            int rank = 0;
            for (int o = e0 + lane; o <= e1; o += kWave) {  // items of expert o in [lo, hi) that come before
                const int no = s_item[o + 1] - s_item[o];
                const int c0 = max(0, lo - s_item[o]), c1 = min(no, hi - s_item[o]);
                // (2 i' + 1) / no < (2 i + 1) / ne, at equality the lower expert first
                // (floor of an integer over 2 ne; the half added keeps the quotient off the integers,
                // which makes the rounding of the multiplication harmless)
                const double num = key * (double)((no + run - 1) / run) + ne - 1.0 + (o < e ? 1.0 : 0.0);
                rank += max(0, min(c1, o == e ? n - s_item[e] : (int)((num + 0.5) * inv) * run) - c0);
            }
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) rank += __shfl_xor(rank, off, kWave);
            if (lane == 0) worder[lo + rank] = make_int2(e, n);
        }
    }

    // one workgroup per group of 64 tokens (lane = token); wavefront w takes the experts
    // 64*word + 16w .. +15 of every mask word
    if (g >= NG || (!lists && !alist)) return;
    const int t = g * kGroup + lane;
    const bool valid = t < T;
    const uint64_t below = (1ull << lane) - 1ull;
    for (int w = blockIdx.y; w < W; w += gridDim.y) {
        const uint64_t word = valid ? mask[(size_t)t * W + w] : 0ull;
        // lane b keeps the three bases of expert 64w + b; b is uniform in the loop below, so each
        // read of them is a broadcast through the scalar unit
        const int e_l = 64 * w + lane;
        const int goff_l = e_l < E ? (FOLD ? s_pre[e_l] : group_off[(size_t)g * E + e_l]) : 0;
        const int cbase_l = e_l < E ? s_off[e_l] + goff_l : 0;
        const int abase_l = e_l < E ? (s_item[e_l] << row_shift) + goff_l : 0;
        const int nb = min(64, E - 64 * w);
#pragma unroll
        for (int bi = 0; bi < 16; ++bi) {
            const int b = 16 * wave + bi;
            const uint64_t bal = __ballot(((word >> b) & 1ull) != 0 && b < nb);
            if (bal != 0ull) {  // uniform
                const int cbase = __builtin_amdgcn_readlane(cbase_l, b);
                const int abase = __builtin_amdgcn_readlane(abase_l, b);
                if ((word >> b) & 1ull) {
                    const int rank = __popcll(bal & below);
                    if (lists) lists[cbase + rank] = t;
                    if (alist) alist[abase + rank] = t;
                }
            }
        }
    }
}

}  // namespace

void launch_mask_from_scores(const float* scores, int T, int E, float tau, uint64_t* mask,
                             int32_t* k_per_token, int32_t* group_off, uint64_t* colmask, bool sets,
                             hipStream_t s) {
    const int W = div_up(E, 64), NG = div_up(T, kGroup);
    LaunchTimer tm(kSlotMask, s);
    if (T <= 16) {
        launch_kernel(select_small_kernel, 1, 1024, sizeof(uint64_t) * 16 * W, s, 
            scores, mask, k_per_token, group_off, colmask, T, E, W, tau);
        return;
    }
    const int grid = div_up(T, 4);
    if (W <= 1) launch_kernel(tau_mask_kernel<1>, grid, 256, 0, s, scores, mask, k_per_token, T, E, W, tau);
    else if (W <= 2) launch_kernel(tau_mask_kernel<2>, grid, 256, 0, s, scores, mask, k_per_token, T, E, W, tau);
    else if (W <= 4) launch_kernel(tau_mask_kernel<4>, grid, 256, 0, s, scores, mask, k_per_token, T, E, W, tau);
    else if (W <= 8) launch_kernel(tau_mask_kernel<8>, grid, 256, 0, s, scores, mask, k_per_token, T, E, W, tau);
    else if (W <= 16) launch_kernel(tau_mask_kernel<16>, grid, 256, 0, s, scores, mask, k_per_token, T, E, W, tau);
    else if (W <= 32) launch_kernel(tau_mask_kernel<32>, grid, 256, 0, s, scores, mask, k_per_token, T, E, W, tau);
    else launch_kernel(tau_mask_kernel<64>, grid, 256, 0, s, scores, mask, k_per_token, T, E, W, tau);
    if (!group_off && !colmask) return;  // nobody reads the counts
    launch_kernel(count_from_mask_kernel, div_up(NG * W, 4), 256, 0, s, mask, group_off, colmask, T, E, W, sets);
}

// 16 tokens per workgroup, four rows of counts per group: where the scan over the groups is a launch of its own anyway
// (up to 192 groups, for which the workspace has room).  2048 experts, gate and counts in two launches against one, us: 700
// tokens 9.5 / 7.7, 2000 tokens 10.5 / 8.4, 4096 tokens 14.6 / 11.4.  Below, whole groups would have to be one
// row: 24.6 us at 300 tokens, against 8.9.
bool gate_counts_supported(int T, int E) {
    return !fold_scan(T, E, 1) && div_up(T, kGroup) < 192;
}

void launch_gate_counts(const float* scores, int T, int E, float tau, uint64_t* mask, int32_t* cnt, bool sets, hipStream_t s) {
    const int W = div_up(E, 64);
    LaunchTimer tm(kSlotMask, s);
    auto go = [&](auto kernel) {
        launch_kernel(kernel, div_up(T, 16), 1024, sizeof(uint64_t) * 16 * W, s, scores, mask, cnt, T, E, W, tau, sets);
    };
    if (W <= 16) go(gate_counts_kernel<16>);
    else if (W <= 32) go(gate_counts_kernel<32>);
    else go(gate_counts_kernel<64>);
}

void launch_select_small_group(const dmoe_layer& L, const SmallGroup& G, int n_layers, int T,
                               hipStream_t s) {
    const int E = L.n_experts, W = div_up(E, 64);
    LaunchTimer tm(kSlotMask, s);
    launch_kernel(select_small_group_kernel, dim3(1, 1, n_layers), 1024, sizeof(uint64_t) * 16 * W, s, G, T, E, W);
}

void launch_counts_from_mask(const uint64_t* mask, int T, int E, int32_t* group_off, uint64_t* colmask, bool sets,
                             hipStream_t s) {
    const int W = div_up(E, 64), NG = div_up(T, kGroup);
    LaunchTimer tm(kSlotMask, s);
    launch_kernel(count_from_mask_kernel, div_up(NG * W, 4), 256, 0, s, mask, group_off, colmask, T, E, W, sets);
}

void launch_mask_from_lists(const int32_t* offsets, const int32_t* lists, int T, int E,
                            uint64_t* mask, int32_t* group_off, uint64_t* colmask, bool sets, void* scratch,
                            size_t scratch_bytes, hipStream_t s) {
    const int W = div_up(E, 64), Tp = round_up(T, kGroup);
    // In one launch, forward us against three: 24 experts of 128, 40 tokens 23.7 / 21.3, 197 tokens (5 and 50 % per expert) 34.7 / 31.7
    // and 36.9 / 35.5, 788 tokens 39.0 / 36.8 and 41.6 / 41.3; beyond, what every workgroup reads of the lists decides: 3152
    // tokens 69.8 / 66.9 and 75.1 / 78.9.
    if (group_off && (long long)T * std::min(E, 64) <= 20000) {
        LaunchTimer tm(kSlotListsToMask, s);
        launch_kernel(lists_small_kernel, dim3(div_up(T, kListsTokens), W), 1024, 0, s, offsets, lists, T, E, W, mask, group_off, colmask, sets);
        return;
    }
    // by bytes where there is room for them and the counts are all that is wanted besides the mask words
    uint8_t* bytes = !colmask && group_off && (size_t)E * Tp <= scratch_bytes ? (uint8_t*)scratch : nullptr;
    // Up to 8 MB of bytes that way costs no more at any density, and looking at the number of positions in three
    // launches costs 0.5 to 1 us (300 tokens x 256 experts of 64 77.3 us a call, 78.0 with the look).
    const bool choose = !bytes || (size_t)E * Tp > ((size_t)8 << 20);
    const long long bits_max = (long long)T * E / 192;
    const size_t n_mask = (size_t)T * W, n_bytes = (size_t)E * Tp / 8, n = bytes ? n_bytes : n_mask;
    const int clear_grid = (int)std::min<size_t>(1024, (n + 255) / 256), finish_grid = div_up(div_up(T, kGroup) * W, 4);
    const dim3 scatter_grid(std::max(1, std::min(div_up(T, 256), 1024 / E)), E);
    LaunchTimer tm(kSlotListsToMask, s);
    auto go = [&](auto choose_c) {
        constexpr bool kChoose = decltype(choose_c)::value;
        launch_kernel(lists_clear_kernel<kChoose>, clear_grid, 256, 0, s, offsets, T, E, mask, n_mask, (uint64_t*)bytes, n_bytes,
                      bits_max);
        launch_kernel(lists_scatter_kernel<kChoose>, scatter_grid, 256, 0, s, offsets, lists, T, E, W, Tp, bytes,
                      reinterpret_cast<unsigned long long*>(mask), bits_max);
        if (bytes)
            launch_kernel(lists_finish_kernel<kChoose>, finish_grid, 256, 0, s, offsets, bytes, T, E, W, Tp, mask, group_off,
                          sets, bits_max);
        else
            launch_counts_from_mask(mask, T, E, group_off, colmask, sets, s);
    };
    if (choose) go(std::true_type{});
    else go(std::false_type{});
}

void launch_mask_topk(const float* scores, int T, int E, int k, uint64_t* mask,
                      int32_t* k_per_token, int32_t* group_off, uint64_t* colmask, bool sets, hipStream_t s) {
    const int W = div_up(E, 64), NG = div_up(T, kGroup);
    LaunchTimer tm(kSlotMask, s);
    const int grid = div_up(T, 4);
    if (W <= 1) launch_kernel(topk_mask_kernel<1>, grid, 256, 0, s, scores, mask, k_per_token, T, E, W, k);
    else if (W <= 2) launch_kernel(topk_mask_kernel<2>, grid, 256, 0, s, scores, mask, k_per_token, T, E, W, k);
    else if (W <= 4) launch_kernel(topk_mask_kernel<4>, grid, 256, 0, s, scores, mask, k_per_token, T, E, W, k);
    else if (W <= 8) launch_kernel(topk_mask_kernel<8>, grid, 256, 0, s, scores, mask, k_per_token, T, E, W, k);
    else if (W <= 16) launch_kernel(topk_mask_kernel<16>, grid, 256, 0, s, scores, mask, k_per_token, T, E, W, k);
    else if (W <= 32) launch_kernel(topk_mask_kernel<32>, grid, 256, 0, s, scores, mask, k_per_token, T, E, W, k);
    else launch_kernel(topk_mask_kernel<64>, grid, 256, 0, s, scores, mask, k_per_token, T, E, W, k);
    if (!group_off && !colmask) return;  // nobody reads the counts
    // counts per (group, expert) and, if wanted, the per-expert token sets
    launch_kernel(count_from_mask_kernel, div_up(NG * W, 4), 256, 0, s, mask, group_off, colmask, T, E, W, sets);
}

bool fold_scan(int T, int E, int split) {
    const int rows = div_up(T, kGroup / split);
    return rows <= kFoldRows && (size_t)rows * E <= 16384;
}

void launch_scan_and_fill(const uint64_t* mask, int T, int E, int32_t* group_off, int32_t* counts,
                          int32_t* offsets, int32_t* item_start, int rows_per_item,
                          int32_t* token_lists, int32_t* aligned_lists, int window_groups,
                          int32_t* witem, int32_t* wfirst, hipStream_t s, const int32_t* sub_cnt,
                          int split, void* worder, bool by_experts) {
    const int W = div_up(E, 64), NG = div_up(T, kGroup);
    const int NW = witem ? div_up(NG, window_groups) : 0;
    const bool fold = sub_cnt && NG > 0 && fold_scan(T, E, split);
    if (!fold) {
        LaunchTimer tm(kSlotScanGroups, s);
        launch_kernel(scan_groups_kernel, div_up(E, 4), 256, 0, s, group_off, NG, E, sub_cnt, split,
                                                        div_up(T, kGroup / split));
    }
    LaunchTimer tm(kSlotFill, s);
    const size_t lds = sizeof(int32_t) * ((fold ? 6 : 3) * (size_t)E + 2);
    static std::once_flag attr_once;  // kernel attributes: once per process, thread-safe
    std::call_once(attr_once, [&] {
        for (const void* f : {reinterpret_cast<const void*>(&fill_lists_kernel<false, true>),
                              reinterpret_cast<const void*>(&fill_lists_kernel<true, true>)})
            (void)hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024);
    });
    // With few token groups and many experts the mask words of a group are split over several
    // workgroups (each repeats the prefix sums over the experts).  Further workgroups only help to
    // pad the aligned list, which with few tokens is mostly padding (256 x 64 gated experts at 48
    // tokens: 64 K entries; 53 us with the four workgroups of its one group).
    int ny = std::max(1, std::min(W, div_up(1024, std::max(1, NG))));
    if (aligned_lists) {
        const long long pad = (long long)E * rows_per_item;
        ny = std::max(ny, (int)std::min<long long>(div_up(256, std::max(1, NG)), pad / (1024LL * std::max(1, NG))));
    }
    const bool many = E > 256;
    auto kernel = fold ? (many ? fill_lists_kernel<true, true> : fill_lists_kernel<true, false>)
                       : (many ? fill_lists_kernel<false, true> : fill_lists_kernel<false, false>);
    int row_shift = 0;
    while ((1 << row_shift) < rows_per_item) ++row_shift;
    launch_kernel(kernel, dim3(std::max(1, NG), ny), 256, lds, s,
        mask, T, E, W, group_off, sub_cnt, split, div_up(T, kGroup / split), row_shift, counts, offsets,
        item_start, token_lists, aligned_lists, window_groups, NW, witem, wfirst, (int2*)worder, by_experts ? 1 : 0);
}

}  // namespace dmoe
