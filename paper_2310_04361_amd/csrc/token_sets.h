// Small batches without token lists: the gate leaves, per 16 tokens and expert, the set of the tokens that keep the
// expert, and a wavefront of an up-projection makes the rows of its work item out of its expert's sets.
//
// With lists a batch of some hundred tokens spends a launch of 6 to 10 us (13 with the scan over the groups in front of it) on
// a few kilobytes, in a forward of 40 to 120 us; the wavefront reads one column of the sets in the time it
// would read its list rows in.  An expert's H rows start at a fixed row (the most items that it can have, times its
// number), which takes no counts to know and no more room than the workspace has for every token keeping every expert.
// One wavefront per expert leaves what the down-projections read: the first rank of every group of 64 tokens
// (group_off) and the expert's first item (item_start).
#pragma once

#include <type_traits>

#include "dmoe_internal.h"

namespace dmoe {

// Inclusive prefix sum over the 64 lanes.
__device__ __forceinline__ int wave_prefix(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);  // row_shr 1, 2, 4, 8: within 16 lanes
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast 15: lane 15 of the row below
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast 31
    return v;
}

// One expert's tokens, over the lanes of a wavefront: lane l has the 16 C tokens from 16 C l on, C = 1, 2 or 4.
struct ExpertTokens {
    uint32_t set[4];  // which of them, 16 in each
    int C;            // (uniform)
    int first;        // how many come before them
    int total;        // all of the expert's (uniform)

    // leave: this wavefront writes the expert's group_off and item_start (rows_per_item rows an item).
    __device__ __forceinline__ void load(const TokenSets& S, int E, int e, int rows_per_item, bool leave) {
        const int lane = threadIdx.x & 63, rows = (S.T + 15) >> 4;
        int n = 0;
        C = S.T <= 1024 ? 1 : (S.T <= 2048 ? 2 : 4);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            set[c] = 0u;
            if (c < C) set[c] = (uint32_t)S.sets[(size_t)min(lane * C + c, rows - 1) * E + e];  // (uniform)
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (lane * C + c >= rows) set[c] = 0u;
            n += __popc(set[c]);
        }
        const int incl = wave_prefix(n);
        first = incl - n;
        total = __builtin_amdgcn_readlane(incl, 63);
        if (leave) {
            const int NG = (S.T + kGroup - 1) / kGroup, items = (S.T + rows_per_item - 1) / rows_per_item;
            const int per_group = 4 / C, g = lane / per_group;  // (lanes to a group)
            if (lane % per_group == 0 && g < NG) S.group_off[(size_t)g * E + e] = first;
            if (lane == 1) S.group_off[(size_t)NG * E + e] = total;
            if (lane == 2) S.item_start[e] = e * items;
            if (lane == 3 && e == E - 1) S.item_start[E] = E * items;
        }
    }
    // The tokens of ranks lo + r, 0 <= r < RANKS, to list[at(r)] (LDS of this wavefront) where 0 <= at(r) < N; -1 where there is none.
    template <int N, int RANKS, class At>
    __device__ __forceinline__ void list(int lo, int32_t* list, At&& at) const {
        const int lane = threadIdx.x & 63;
        if (lane < N) list[lane] = -1;
        int rank = first - lo;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (c >= C) break;  // (uniform)
            const int n = __popc(set[c]);
            if (__ballot(rank < RANKS && rank + n > 0) != 0ull) {
                int r = rank;
#pragma unroll
                for (int b = 0; b < 16; ++b) {
                    const uint32_t in = (set[c] >> b) & 1u;
                    const int i = at(r);
                    if (in != 0u && (unsigned)r < (unsigned)RANKS && (unsigned)i < (unsigned)N) list[i] = 16 * (lane * C + c) + b;
                    r += (int)in;
                }
            }
            rank += n;
        }
    }
};

// The work item (of rows_per_item rows) of a wavefront, four to a workgroup: wavefront i has item i / E of expert i % E, so
// that the first items of all experts, which there always are, come first.  There is a wavefront for every item that an
// expert can have.  Where the chip holds them all (at most `resident` workgroups) the first items go over all the CUs before
// a CU gets a second one, otherwise they go to the workgroups that start first.
inline int sets_grid(TokenSets& S, int E, int rows_per_item, int resident) {
    const int grid = (int)(((long long)E * div_up(S.T, rows_per_item) + 3) / 4);
    S.wave_step = grid > resident ? 1 : grid;
    S.block_step = grid > resident ? 4 : 1;
    return grid;
}
struct SetItem {
    int e, item;  // the expert and which of its items
    int index;    // the item's place among all that there can be
    ExpertTokens tok;
    // false: no such item.  The first wavefront of an expert leaves its group_off and item_start.
    __device__ __forceinline__ bool start(const TokenSets& S, int E, int wave, int rows_per_item) {
        const int i = S.wave_step * wave + S.block_step * (int)blockIdx.x;
        e = i % E;
        item = i / E;
        index = e * ((S.T + rows_per_item - 1) / rows_per_item) + item;
        tok.load(S, E, e, rows_per_item, item == 0);
        return item * rows_per_item < tok.total;
    }
};

// The sets as an argument of a kernel that has an instance for lists, which has no such argument: 32 bytes more of them cost the
// up-projection of every batch with lists 0.3 to 0.6 us (forward, 16384 tokens x 128 experts of 24, d = 768, with them 122.5, without 121.9).
struct NoSets {
    NoSets(const TokenSets&) {}
};
template <bool SETS>
using SetsArg = std::conditional_t<SETS, TokenSets, NoSets>;

}  // namespace dmoe
