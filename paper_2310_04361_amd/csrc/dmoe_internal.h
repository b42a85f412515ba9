// Internal declarations shared by the HIP translation units of libdmoe (not installed).
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>

#include <mutex>

#include "../../include/dmoe.h"

namespace dmoe {

// ---- fixed granularities -------------------------------------------------------------------
constexpr int kGroup = 64;        // tokens per select group (one wavefront, lane = token)
constexpr int kChunkGroups = 2;   // groups per down-projection token chunk
constexpr int kChunk = kGroup * kChunkGroups;   // 128 tokens whose outputs live in LDS together
constexpr int kTilePad = 64;      // entries the expert kernels may read past the end of the lists

inline int round_up(int a, int b) { return (a + b - 1) / b * b; }
inline int div_up(int a, int b) { return (a + b - 1) / b; }
// Hidden units per H row: 32, 64 or 128 (the widths the expert kernels are compiled for), so
// experts of 65 .. 96 neurons take 128.
inline int m_pad_of(int m) {
    const int p = round_up(m, 32);
    return p == 96 ? 128 : p;
}

// List rows per up-projection work item (a multiple of 16); every expert's region of H starts
// at a multiple of this many rows.
inline int up_rows_bf16(const dmoe_layer& L) {
    // wide experts (8 neuron tiles per K step) use the kernel that shares the weights of a 256-row
    // item through LDS; everything else uses one wavefront per 64 rows
    const int tiles = (L.gated ? 2 : 1) * (m_pad_of(L.expert_size) / 16);
    return tiles == 8 ? 256 : 64;
}

// H capacity in 16-row fragments for T tokens: every expert may round up to a whole work item,
// and the down kernel reads one fragment past the last one.
inline size_t h_fragments(const dmoe_layer& L, int T) {
    return ((size_t)T * L.n_experts + (size_t)L.n_experts * up_rows_bf16(L)) / 16 + 4;
}

// 8-bit expert weights (both 8-bit formats); 8-bit expert inputs as well.
inline bool weights_fp8(const dmoe_layer& L) {
    return L.weight_format == DMOE_W_FP8_E4M3 || L.weight_format == DMOE_W_FP8_E4M3_X8 ||
           L.weight_format == DMOE_W_FP8_E4M3_A8;
}
inline bool acts_fp8(const dmoe_layer& L) {
    return L.weight_format == DMOE_W_FP8_E4M3_X8 || L.weight_format == DMOE_W_FP8_E4M3_A8;
}
// 8-bit hidden activations as well (every H row quantised before the down-projection) ...
inline bool hidden_fp8(const dmoe_layer& L) { return L.weight_format == DMOE_W_FP8_E4M3_A8; }
// ... and whether the 8-bit matrix-core down-projection covers the shape (H rows of 64 or 128
// neurons, 256-column slices); other shapes quantise H in place and run the bf16 kernels.
inline bool down_x8_shape(const dmoe_layer& L) {
    return hidden_fp8(L) && m_pad_of(L.expert_size) >= 64 && L.d_model % 256 == 0;
}
// ... and whether the 8-bit matrix-core up-projection covers the shape (the 256-row work items of
// the wide-expert kernel); other shapes run the bf16 kernels on the quantised input.
inline bool up_x8_supported(const dmoe_layer& L) { return acts_fp8(L) && up_rows_bf16(L) == 256; }

// Experts that fit ONE 16-row weight tile -- at most 16 neurons, or gated with at most 8 (up rows
// and gate rows together) -- take the up-projection kernel built around that tile.
inline bool up_tiny_supported(const dmoe_layer& L) {
    return L.dtype == DMOE_BF16 && L.expert_size <= (L.gated ? 8 : 16);
}

// Neurons per H row as the kernels lay it out: experts of one tile keep just their one or two pieces of eight
// (their pairs are many, and the rows of one expert and group, which follow each other, then share
// cache lines.  4096 tokens x 2048 gated experts of 8: up 190 -> 179 us, down 166 -> 154).  Fully 8-bit layers of such experts quantise
// padded rows in place.
inline int h_row_neurons(const dmoe_layer& L) {
    return up_tiny_supported(L) && !hidden_fp8(L) ? (L.expert_size <= 8 ? 8 : 16) : m_pad_of(L.expert_size);
}

// Sub-buffers of the packed-weights buffer (bytes from its start).
struct PackedLayout {
    size_t w2f, w2g, w2s, wupf, wgatef, r1f, r2f, w2f8, wupf8, wgatef8, wtinyf, scales, wupx8, wgatex8, w2x8, wsc8, total;
};
size_t down_quad_w_bytes(const dmoe_layer& L);  // 0: no such operands
inline PackedLayout packed_layout(const dmoe_layer& L) {
    PackedLayout P{};
    if (L.dtype != DMOE_BF16) return P;
    const size_t one =
        (2 * (size_t)L.n_experts * L.d_model * m_pad_of(L.expert_size) + 255) / 256 * 256;
    // the 32x32x16 down fragments pack the experts' real 8-neuron pieces in stages of one or two
    // experts: never more than m_pad neurons per expert, but a last half-filled stage counts as
    // two experts
    const size_t one_g =
        (2 * ((size_t)L.n_experts + 1) * L.d_model * m_pad_of(L.expert_size) + 255) / 256 * 256;
    P.w2f = 0;          // down-projection, 16x16x32 fragments (small-token path)
    P.w2g = one;        // down-projection, 32x32x16 fragments (down_bf16.hip)
    P.wupf = one + one_g;
    P.wgatef = P.wupf + one;
    size_t o = P.wupf + (L.gated ? 2 : 1) * one;
    // router weights as fragments: r1f[d_h/16][d/32][64][8], r2f[ceil(E/16)][d_h/32][64][8]
    P.r1f = o;
    o += (2 * (size_t)round_up(L.router_hidden > 0 ? L.router_hidden : 0, 16) * L.d_model + 255) / 256 * 256;
    P.r2f = o;
    o += (2 * (size_t)round_up(L.n_experts, 16) * round_up(L.router_hidden > 0 ? L.router_hidden : 0, 32) + 255) / 256 * 256;
    // 8-bit expert weights: the same fragments with one byte per weight for the small-token
    // kernels (w2f8, wupf8, wgatef8: half of `one` each)
    P.w2f8 = P.wupf8 = P.wgatef8 = o;
    if (weights_fp8(L)) {
        const size_t half = (one / 2 + 255) / 256 * 256;
        P.w2f8 = o;
        P.wupf8 = o + half;
        P.wgatef8 = o + 2 * half;
        o += (L.gated ? 3 : 2) * half;
    }
    // experts of one 16-row weight tile (at most 16 neurons; gated: 8 up rows + 8 gate rows)
    // (ffn_bf16.hip, up_tiny_kernel): wtinyf[E][d/32][64][8]
    P.wtinyf = o;
    if (up_tiny_supported(L)) o += (2 * (size_t)L.n_experts * 16 * L.d_model + 255) / 256 * 256;
    // 8-bit weights: the caller's scales snapped to powers of two, [E][3] fp32 -- the copy every
    // kernel uses, so that all paths compute the same layer whatever the caller passed
    P.scales = o;
    if (weights_fp8(L)) o += (sizeof(float) * 3 * (size_t)L.n_experts + 255) / 256 * 256;
    // 8-bit inputs: the up (and gate) matrices as operands of the 8-bit MFMA,
    // wupx8[E][m_pad/16][d/128][64][32] (ffn_x8.hip), one byte per weight
    P.wupx8 = P.wgatex8 = o;
    if (up_x8_supported(L)) {
        const size_t half = (one / 2 + 255) / 256 * 256;
        P.wupx8 = o;
        P.wgatex8 = o + half;
        o += (L.gated ? 2 : 1) * half;
    }
    // 8-bit hidden activations: the down matrices as operands of the 32x32x64 8-bit MFMA,
    // w2x8[E * units][d/32][64][32] (down_x8.hip; a unit = 64 neurons of an expert), and the E8M0
    // byte of every unit's down scale
    P.w2x8 = P.wsc8 = o;
    if (down_x8_shape(L)) {
        const size_t units = (size_t)L.n_experts * (m_pad_of(L.expert_size) / 64);
        P.w2x8 = o;
        o += (units * (L.d_model / 32) * 2048 + 255) / 256 * 256;
        P.wsc8 = o;
        o += (units + 255) / 256 * 256;
    }
    // down-projection of sparse selections: operands of the structured-sparse 32x32x32 MFMA
    // (down_quad_bf16.hip)
    P.w2s = o;
    o += (down_quad_w_bytes(L) + 255) / 256 * 256;
    P.total = o;
    return P;
}

// ---- kernel timing slots --------------------------------------------------------------------
enum Slot {
    kSlotRouter = 0,
    kSlotMask,
    kSlotListsToMask,
    kSlotScanGroups,
    kSlotFill,
    kSlotUp,
    kSlotDown,
    kSlotDownRmw,
    kSlotFfnF32,
    kSlotSmallUp,
    kSlotSmallDown,
    kSlotPack,
    kSlotQuantX,
    kSlotQuantH,
    kSlotCount
};

// Scope of the kernel launches that are accounted to one timing slot (see dmoe_timing_enable).
// With timing enabled, launch_kernel() inside the scope has the launch itself stamp an event pair
// with the start and the end of the kernel on the device, so what is summed is kernel time, not
// the gaps around event records.  One scope counts as one launch of its slot however many
// kernels it holds.
struct LaunchTimer {
    LaunchTimer(int slot, hipStream_t stream);
    ~LaunchTimer();
    int slot_;
    int index_;          // event pair reserved for the first launch, -1: timing off
    bool used_;          // that pair has been handed to a launch
    LaunchTimer* prev_;
    hipStream_t stream_;
};
// Event pair for the next launch of the calling thread's innermost scope (false: launch untimed).
bool timer_events_for_launch(hipEvent_t* start, hipEvent_t* stop);

// Every kernel of the library is launched through here.
template <typename... KArgs, typename... Args>
inline void launch_kernel(void (*kernel)(KArgs...), dim3 grid, dim3 block, size_t lds, hipStream_t s,
                          Args&&... args) {
    hipEvent_t ev0, ev1;
    if (timer_events_for_launch(&ev0, &ev1))
        hipExtLaunchKernelGGL(kernel, grid, block, (uint32_t)lds, s, ev0, ev1, 0u,
                              static_cast<KArgs>(args)...);
    else
        kernel<<<grid, block, lds, s>>>(static_cast<KArgs>(args)...);
}

// ---- select / bucket (select.hip) -----------------------------------------------------------
// group_off is [(NG+1)][E] int32 with NG = ceil(T/64): after the scans, group_off[g][e] is the
// number of tokens < 64*g that selected expert e, and row NG holds the per-expert totals.
// (For more than 16 tokens group_off may be null, if colmask is: then nothing is counted.)
// colmask (nullable) is [NG][E] u64: bit j of colmask[g][e] = token 64g + j keeps expert e.
// sets, in these launchers: the rows are token sets (token_sets.h), of 16 tokens each, instead of counts.
void launch_mask_from_scores(const float* scores, int T, int E, float tau, uint64_t* mask,
                             int32_t* k_per_token, int32_t* group_off, uint64_t* colmask, bool sets,
                             hipStream_t s);
// Top-k gate: exactly k experts per token, ties at the k-th score to the lower expert index.
void launch_mask_topk(const float* scores, int T, int E, int k, uint64_t* mask,
                      int32_t* k_per_token, int32_t* group_off, uint64_t* colmask, bool sets, hipStream_t s);
// Counts per (group, expert) and, if wanted, the per-expert token sets from mask bits.
void launch_counts_from_mask(const uint64_t* mask, int T, int E, int32_t* group_off, uint64_t* colmask, bool sets,
                             hipStream_t s);
// scratch: E * 64 ceil(T / 64) bytes (16-byte aligned) for the way without atomics, which is not taken with fewer.
void launch_mask_from_lists(const int32_t* offsets, const int32_t* lists, int T, int E,
                            uint64_t* mask, int32_t* group_off, uint64_t* colmask, bool sets, void* scratch,
                            size_t scratch_bytes, hipStream_t s);
// sub_cnt (nullable): the counts come as `split` rows per group (ceil(T * split / 64) rows) that
// are added up into group_off on the way; with few such rows (fold_scan) the list fill does that
// itself and there is no scan launch, so the counts of small batches should come this way.
constexpr int kFoldRows = 32;
bool fold_scan(int T, int E, int split);
// Dynamic-k gate on stored scores and the counts of its decisions, four rows per group, in one launch.
bool gate_counts_supported(int T, int E);
void launch_gate_counts(const float* scores, int T, int E, float tau, uint64_t* mask, int32_t* cnt, bool sets, hipStream_t s);
// What the up-projections of a small batch read instead of lists, and what they write for the
// down-projections (token_sets.h); sets == nullptr: there are lists.
constexpr int kSetTokens = 3072;  // (a lane of a wavefront holds up to four rows)
struct TokenSets {
    const int32_t* sets;   // [ceil(T / 16)][E]: bit j of row r: token 16 r + j keeps the expert
    int32_t* group_off;    // [ceil(T / 64) + 1][E]
    int32_t* item_start;   // [E + 1]
    int T;
    int wave_step, block_step;  // (sets_grid)
};
void launch_scan_and_fill(const uint64_t* mask, int T, int E, int32_t* group_off, int32_t* counts,
                          int32_t* offsets, int32_t* item_start, int rows_per_item,
                          int32_t* token_lists, int32_t* aligned_lists, int window_groups,
                          int32_t* witem, int32_t* wfirst, hipStream_t s,
                          const int32_t* sub_cnt = nullptr, int split = 1, void* worder = nullptr,
                          bool by_experts = false);
// First of the N work items of the wide up-projection (in the order of worder) that XCD k takes.
__host__ __device__ inline int xcd_first(int N, int k) { return (int)((long long)N * k / 8); }
// Whether an XCD takes a share of the experts (and all the tokens) rather than a stretch of tokens
// (and all the experts): see the order of the work items in select.hip.
bool up_items_by_experts(const dmoe_layer& L);
// The up-projection walks its work items window by window (window = window_groups consecutive
// 64-token groups, window w on XCD w % 8) so that the x rows an XCD gathers stay in its L2:
// witem[NW][E+1], wfirst[NW][E] are built with the lists (nullable: no tables).  Of fewer
// than 8 windows each is shared by several XCDs; wide experts (whose weight stream would flush the
// rows anyway) have a single one.
int up_window_groups(const dmoe_layer& L, int T);
constexpr int kMaxExperts = 4096;  // the list fill keeps 2 ints per expert in LDS

// ---- router (router.hip) ----------------------------------------------------------------------
void launch_router_f32(const dmoe_layer& L, const float* x, int T, float* scores, hipStream_t s);
void launch_router_bf16(const dmoe_layer& L, const void* x, int T, float* scores, hipStream_t s);
// Fused router + gate + group counts (router_fused.hip); mask == nullptr runs the router alone,
// which has no limit on the number of experts (router_fused_scores_supported).
bool router_fused_supported(const dmoe_layer& L);
bool router_fused_scores_supported(const dmoe_layer& L);
// split = 1, 2 or 4 workgroups per group of 64 tokens (router_fused_split: more where the groups
// alone would leave most of the chip idle).  With the gate and split > 1, group_cnt is a table
// of split rows per group -- row r holds the counts of the tokens 64 r / split .. -- that
// launch_scan_and_fill adds up.
int router_fused_split(const dmoe_layer& L, int T);
// Large routers (2 MB of matrices or more) without the gate: two launches with the matrices split
// over the workgroups; hid is a [T][d_h] bf16 scratch buffer.
bool router_sliced(const dmoe_layer& L);
void launch_router_sliced(const dmoe_layer& L, const void* x, int T, void* hid, float* scores,
                          hipStream_t s);
// ... and with the dynamic-k gate and the counts of its decisions, four rows per group or token sets (513 to 2048 experts).
bool scores_gate_supported(const dmoe_layer& L, int T);
void launch_router_gate_sliced(const dmoe_layer& L, const void* x, int T, void* hid, float* scores, float tau, uint64_t* mask,
                               int32_t* cnt, bool sets, hipStream_t s);
// (sets, here and below: the gate leaves the token sets of token_sets.h in the rows of counts)
// Small and medium batches of a router whose first matrix takes 512 KB or more: the hidden rows (a [T][d_h] bf16 buffer) in one launch, the
// scores and the gate in another; the bits of launch_router_fused with the gate.
bool router_two_launches(const dmoe_layer& L, int T);
// q (nullable): the rows of x are quantised as well, beside the hidden rows; false: not here.
struct QuantX {
    uint8_t* x8;      // [T][d] codes
    float* xscale;    // [T]
    __bf16* xhat;     // [T][d] the quantised rows as bf16 numbers, or null
};
bool launch_router_two(const dmoe_layer& L, const void* x, int T, int split, void* hid, float* scores, float tau,
                       uint64_t* mask, int32_t* group_cnt, bool sets, const QuantX* q, hipStream_t s);
void launch_router_fused(const dmoe_layer& L, const void* x, int T, int split, float* scores,
                         float tau, uint64_t* mask, int32_t* group_cnt, bool sets, hipStream_t s);

// ---- small-token path (use_small_path in api.hip): up to kGroupMax layers of one shape per launch ------
// The attention projections Q, K and V are three converted layers with the same input (Sec. 3.5),
// and at 16 tokens a forward is a few launches that each last a few microseconds: every
// small-token kernel therefore takes the per-layer pointers of a whole group and works on layer
// blockIdx.z.  A single layer is a group of one.
constexpr int kGroupMax = 4;
struct SmallMod {
    const __bf16 *r1f, *r_b1, *r2f, *r_b2;                 // packed router matrices, biases
    const __bf16 *wupf, *wgatef, *b_up, *w2f, *b_down;     // packed expert matrices, biases
    const uint8_t *wupf8, *wgatef8, *w2f8;                 // the same fragments, one E4M3 byte per weight
    const float* w_scales;                                 // [E][3] (up, gate, down); null: bf16 weights
    __bf16 *hid, *Hs, *y;                                  // router hidden tile, H fragments, output
    float *scores, *partial;                               // scores [T][E]; per-expert-group partial outputs
    uint64_t *mask, *colmask;                              // mask [T][W]; colmask [E]
    int32_t* group_cnt;                                    // [E] tokens per expert
    void *sync, *tickets;                                  // exchange area and counters of a call (ffn_small.hip)
    float tau;
};
struct SmallGroup {
    SmallMod m[kGroupMax];
};
// Router as a weight stream over many workgroups (same support conditions as the fused kernel);
// hid is a 16 x d_h bf16 scratch buffer per layer.  The gate runs separately.
void launch_router_small(const dmoe_layer& L, const SmallGroup& G, int n_layers, const void* x,
                         int T, hipStream_t s);
// Dynamic-k gate of every layer of the group on its stored scores (mask, colmask, group_cnt).
void launch_select_small_group(const dmoe_layer& L, const SmallGroup& G, int n_layers, int T,
                               hipStream_t s);

// ---- small-token forward (ffn_small.hip): T <= kSmallBatch -----------------------------------------
constexpr int kSmallTokens = 16;      // one MFMA column tile
constexpr int kSmallMaxTiles = 4;
constexpr int kSmallBatch = 16 * kSmallMaxTiles;
constexpr int kSmallMaxGroups = 32;   // expert groups whose shares are summed at the end
constexpr int kSmallGateMaxE = 1024;  // experts up to which the router and the gate ride in the up-projection
bool small_bf16_supported(const dmoe_layer& L);
size_t small_sync_bytes(const dmoe_layer& L);
size_t small_ticket_bytes(const dmoe_layer& L);
// Hs: E * (m_pad/32) * ceil(T/16) KiB of fragments; partial: at most 16 kSmallMaxGroups rows of d floats.
// gate: router, dynamic-k gate (M.tau) and up-projection in one launch, which writes M.mask, M.colmask and,
// if not null, M.scores; otherwise M.colmask comes from a gate that ran before.  x_router: the
// router's input; x: the experts' (another one only in layers with 8-bit inputs).
void launch_small_bf16(const dmoe_layer& L, const SmallGroup& G, int n_layers, const void* x_router,
                       const void* x, int T, bool gate, hipStream_t s);
void small_give_up(int every);  // dmoe_small_give_up

// ---- experts ----------------------------------------------------------------------------------
void launch_ffn_f32(const dmoe_layer& L, const float* x, int T, const uint64_t* mask, float* y,
                    hipStream_t s);
// Small fp32 layers: router, dynamic-k gate and experts in one launch (mask, scores_out: nullable outputs).
bool layer_f32_fused(const dmoe_layer& L);
void launch_layer_f32(const dmoe_layer& L, const float* x, int T, float tau, uint64_t* mask, float* scores_out,
                      float* y, hipStream_t s);
void launch_pack_bf16(const dmoe_layer& L, void* packed, hipStream_t s);
// H holds one row of m_pad hidden activations per list row (layout: see ffn_bf16.hip).
// alist is the work-item-aligned token list (see select.hip); its index is the row index of H.
void launch_up_bf16(const dmoe_layer& L, const void* x, int T, const int32_t* witem,
                    const int32_t* wfirst, const void* worder, const int32_t* alist, const TokenSets& S, void* H, hipStream_t s);
// Down-projection and merge (down_bf16.hip): mask is the token-major selection bitmask that the
// lists were built from; group_off[g][e] = rows of expert e that belong to tokens before group g.
bool down_bf16_supported(const dmoe_layer& L);
bool down_bf16_addressable(const dmoe_layer& L, int T);
void launch_pack_down_bf16(const dmoe_layer& L, void* w2g, hipStream_t s);
// Two kernels, both launched where the first can win: offsets[E] (the executed pairs) decides on the device
// which one works -- at most max_pairs pairs (down_quad_max_pairs; 0: not launched): the one for sparse
// selections (down_quad_bf16.hip), more: the dense one (down_bf16.hip).  Sizes beyond the 32-bit
// buffer offsets of both: down_rmw_bf16.hip.
void launch_down_bf16(const dmoe_layer& L, int T, const int32_t* item_start,
                      const int32_t* group_off, const uint64_t* mask, const int32_t* offsets,
                      const void* H, void* y, float* partial, long long max_pairs,
                      hipStream_t s);
bool down_bf16_wide(const dmoe_layer& L, int T);  // workgroups of 384 columns
double down_walk_us(const dmoe_layer& L, int T);  // estimate of one workgroup's walk over the experts
double down_walk_us(const dmoe_layer& L);         // ... where it is not divided
void launch_pack_down_quad(const dmoe_layer& L, void* packed, hipStream_t s);
long long down_quad_max_pairs(const dmoe_layer& L, int T);
void launch_down_quad(const dmoe_layer& L, int T, const int32_t* item_start, const int32_t* group_off,
                      const int32_t* alist, const uint64_t* mask, const int32_t* offsets, const void* H, void* y,
                      float* partial, long long max_pairs, hipStream_t s);
void launch_down_rmw_bf16(const dmoe_layer& L, int T, const int32_t* item_start,
                          const int32_t* group_off, const int32_t* alist, const void* H, void* y, hipStream_t s);

// Batches too small to fill the chip: the walk over the experts is split over this many workgroups
// per tile of outputs, whose fp32 shares (down_partial_floats of workspace) are added at the end.
// down_parts_limit: as many as the chip and the workspace hold.
int down_parts(const dmoe_layer& L, int T);
int down_parts_limit(const dmoe_layer& L, int T);
size_t down_partial_floats(const dmoe_layer& L, int T);
void launch_down_finish(const dmoe_layer& L, int T, const float* partial, void* y, int parts, hipStream_t s);
// Loop trips of one part: even, so that a part never starts at the last trip of a batch of experts.
__host__ __device__ inline int down_part_trips(int trips, int parts) {
    return parts <= 1 ? trips : ((trips + parts - 1) / parts + 1) / 2 * 2;
}
// Which 128-token chunk, column slice and part a workgroup of the matrix-core down kernels works
// on (workgroups are dealt round-robin to the 8 XCDs).  Undivided walks: the column slices of one
// chunk share its H rows, so they sit on one XCD and next to each other in launch order.  Divided
// walks: with few chunks the weights are the traffic, so the chunks that read the same slice of the
// same experts follow each other, and every XCD takes an eighth of that order.  (Whole slices dealt to
// the XCDs in turn put 38 workgroups on each of four XCDs and 19 on each of the others for 19 chunks
// of 768 columns in 4 parts: 76 us a forward of 128 x 24 experts, 63 this way.)  part == parts: no work.
// xs (undivided; divides NS and 8): the XCDs as xs groups of slices x 8 / xs groups of chunks.
struct DownTile {
    int chunk, slice, part;
};
__host__ __device__ inline DownTile down_tile(int block, int NS, int NC, int parts, int xs = 1) {
    const int xcd = block & 7, k = block >> 3;
    if (parts <= 1) {
        const int xc = 8 / xs, per = NS / xs;
        return DownTile{(k / per) * xc + xcd % xc, (xcd / xc) * per + k % per, 0};
    }
    const int n = NC * NS * parts, first = xcd_first(n, xcd);
    if (first + k >= xcd_first(n, xcd + 1)) return DownTile{0, 0, parts};
    const int i = first + k, combo = i / NC;
    return DownTile{i % NC, combo % NS, combo / NS};
}
inline int down_grid(int NC, int NS, int parts) {
    return parts <= 1 ? round_up(NC, 8) * NS : round_up(NC * NS * parts, 8);
}

// ---- 8-bit hidden activations (down_x8.hip) -------------------------------------------------------
// Row-wise quantisation of the H rows that the up-projection wrote (see DMOE_W_FP8_E4M3_A8 in
// dmoe.h; the number of rows is item_start[E] * rows per item): to codes H8[row][64] and E8M0
// scale bytes hs8[row] for the 8-bit down-projection, or in place (the quantised rows as bf16
// numbers) for the bf16 down-projections.
void launch_pack_down_x8(const dmoe_layer& L, void* packed, hipStream_t s);
bool down_x8_addressable(const dmoe_layer& L, int T);
void launch_h_rows_to_e4m3(const dmoe_layer& L, const int32_t* item_start, const void* H,
                           uint8_t* H8, uint8_t* hs8, hipStream_t s);
void launch_h_rows_quantize(const dmoe_layer& L, const int32_t* item_start, void* H, hipStream_t s);
void launch_down_x8(const dmoe_layer& L, int T, const int32_t* item_start, const int32_t* group_off,
                    const uint64_t* mask, const uint8_t* H8, const uint8_t* hs8, void* y,
                    float* partial, hipStream_t s);

// ---- 8-bit expert inputs (ffn_x8.hip) -------------------------------------------------------------
// Row-wise quantisation of x (see DMOE_W_FP8_E4M3_X8 in dmoe.h): x8[T][d] E4M3 codes, xscale[T]
// the power-of-two scales, xhat[T][d] (nullable) the quantised rows as bf16 numbers.
void launch_quantize_x(const dmoe_layer& L, const void* x, int T, const QuantX& q, hipStream_t s);
void launch_pack_x8(const dmoe_layer& L, void* packed, hipStream_t s);
// Up-projection on 8-bit operands; same work items, lists and H rows as launch_up_bf16.
// H8 / hs8 non-null: the rows go out quantised for the 8-bit
// down-projection instead of as bf16 rows in H.
void launch_up_x8(const dmoe_layer& L, const uint8_t* x8, const float* xscale, int T,
                  const int32_t* witem, const void* worder, const int32_t* alist, const TokenSets& S, void* H,
                  uint8_t* H8, uint8_t* hs8, hipStream_t s);

bool experts_bf16_supported(const dmoe_layer& L);
bool router_bf16_supported(const dmoe_layer& L);

}  // namespace dmoe
