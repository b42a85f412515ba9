// bf16 down-projection and merge for sparse selections: as down_bf16.hip (accumulators of 128 tokens for the
// whole kernel, a walk over all experts, every y element written once), on the structured-sparse matrix
// instruction.
//
// v_smfmac_f32_32x32x32_bf16 multiplies a 32 x 32 operand of which every row keeps two of each four
// neighbouring k, with a 2-bit position each, by a full 32 x 32 operand in the time that the dense
// instruction takes for half of that k.  Here the four neighbours are one neuron of four consecutive
// experts (a "quad"), and the two that a token keeps are two experts it selected: a token that selected
// at most two of a quad is served by one instruction, whichever two they are.  Its third and fourth go
// into a second image of the tile (level 2), which is multiplied only for the (quad, 32-token tile)
// pairs that have such a token.  With a share p of the experts selected, a token has three or four of a
// quad with probability 4 p^3 (1 - p) + p^4: at p = 0.07 one tile in 25 needs level 2, at p = 0.15 three in ten.
//
// Work split: workgroup = 128 tokens x 256 columns, eight wavefronts of 32 columns, one workgroup per CU.
// What bounds it is the vector memory path: the weights of a k-step are 16 KB per workgroup for 256 cycles of
// its matrix instructions, all of the 60 to 64 bytes per clock that a CU's path delivers.  (4096
// tokens x 256 gated experts of 64, d = 2048, 2 % density, 122 us: the matrix instructions alone 75, with the
// weights 91, with the tiles from LDS 99, with the level-2 test 105; the rest is the gather of the H rows.)
// With four wavefronts of 64 columns, half the LDS reads, it took 133 us: with one wavefront per
// SIMD nothing hides what is not a matrix instruction.  Measured against the dense kernel, us: the shape above at
// 7 % 144 against 172; 4096 tokens x 2048 gated experts of 8, 7 % density 168 against 198; 50432 tokens x 24 experts
// of 128, d = 768, 5 % 138 against 143.  Experts of 9 to 32 neurons stay with the dense kernel: 50432 tokens x 128
// experts of 24, d = 768, 6 %: 168 against 166.
//
// A stage is QS quads x PS pieces (of 8 neurons) = KS k-steps.  Stage n is multiplied while the tiles of
// stage n + 2 are written to LDS (requested two stages before) and the H rows of stage n + 4 are requested;
// one barrier per stage; four LDS buffers.
#include <algorithm>

#include "down_rmw.h"
#include "pack.h"

namespace dmoe {

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x16 __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) char LdsChar;
typedef __attribute__((address_space(3))) u32x4 LdsU32x4;
typedef __attribute__((address_space(3))) uint32_t LdsU32;
typedef __attribute__((address_space(3))) bf16x8 LdsBf16x8;

constexpr int kDqTokens = 128, kDqTiles = 4;  // 4 tiles of 32 tokens = 2 select groups of 64
constexpr int kDqWaves = 8, kDqCols = 32 * kDqWaves;
// A tile of the pair walk in units of one of its rows (fits the walk's times over 24 to 699 experts, 0.4 to 4 %)
constexpr int kTileCost64 = 9, kTileCost128 = 200;
constexpr int kDqTrip = 4;                    // stages per loop trip = LDS buffers
constexpr int kRawBuffer = 0x00020000;        // offsets from num_records on read as zero and move no data

// How experts of PG pieces are walked; SPQ stages per group of QS quads.
struct QuadShape {
    int PG, QS, PS, KS, SPQ;
};
constexpr QuadShape quad_shape(int PG) {
    const int qs = PG == 1 ? 4 : 1, ps = PG == 1 ? 1 : PG % 3 == 0 ? 3 : 4;
    return QuadShape{PG, qs, ps, qs * ps, PG / ps};
}
// The supported numbers of pieces (0: none): one, or H rows of 64 or 128 neurons.
int quad_pieces(int m) {
    const int pg = div_up(m, 8);
    return pg == 1 ? 1 : pg <= 4 ? 0 : pg <= 6 ? 6 : pg <= 8 ? 8 : 16;
}

// w2s[stage][d/32][KS][2][64][8]: lane (H, n) of part f of a k-step holds, for output column 32 tile + n, the
// positions p = 8 f + s of the B operand's 16: expert p & 3 of the quad, neuron
// 4 (p >> 3) + 2 H + ((p >> 2) & 1) of the piece -- so that A lane (h, .) meets the neurons 4h .. 4h + 3
// (lane half h of A covers positions 8h .. 8h + 7 of both lane halves of B).
struct QuadMap {
    static constexpr int kCols = 32;
    QuadShape q;
    int blocks;  // stages * KS * 2
    __device__ void row(int b, int H, int s, int& e, int& neuron) const {
        const int f = b & 1, ks = (b >> 1) % q.KS, st = (b >> 1) / q.KS;
        e = 4 * ((st / q.SPQ) * q.QS + ks / q.PS) + (s & 3);
        neuron = 8 * ((st % q.SPQ) * q.PS + ks % q.PS) + 4 * f + 2 * H + (s >> 2);
    }
    static __device__ int lane(int col) { return col; }
    __device__ size_t block(int b, int ct, int n_ct) const {
        return ((size_t)(b / (2 * q.KS)) * n_ct + ct) * (2 * q.KS) + b % (2 * q.KS);
    }
};

// Whether the walk over the pairs of a chunk (down_rmw.h) is the shorter one (uniform).  It costs tile_cost for each tile of up to 32
// rows of an expert and 1 for each row; limit: of four chunks, below 0: none.  If every pair were a tile of its own and that is still within
// the limit, nothing is counted; else four chunks spread over the batch are, by every workgroup alike: where chunks decided for
// themselves and some took the pairs, others the quads, both lost the weights that they share (50432 tokens x 100
// experts of 128, d = 768, 0.8 %: all pairs 399 us, all quads 427, mixed 500).
__device__ __forceinline__ bool pairs_are_less(int pairs, const int32_t* group_off, int T, int E, int NG, int tile_cost, int limit) {
    __shared__ int s_cost[kDqWaves];
    const int tid = threadIdx.x, n_chunks = (T + kChunk - 1) / kChunk;
    if (limit < 0 || 4ll * pairs * (tile_cost + 1) <= (long long)limit * n_chunks) return true;
    int cost = 0;
    for (int e = tid; e < E; e += 64 * kDqWaves) {
        int n[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int g = (n_chunks * (2 * i + 1) >> 3) * kChunkGroups;
            n[i] = group_off[(size_t)min(g + kChunkGroups, NG) * E + e] - group_off[(size_t)g * E + e];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) cost += ((n[i] + 31) >> 5) * tile_cost + n[i];
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) cost += __shfl_xor(cost, off, 64);
    if ((tid & 63) == 0) s_cost[tid >> 6] = cost;
    __syncthreads();
    int all = 0;
#pragma unroll
    for (int w = 0; w < kDqWaves; ++w) all += s_cost[w];
    return all <= limit;
}

// R: sets of weights (a k-step each) in flight.
template <int PG, int R>
__global__ __launch_bounds__(64 * kDqWaves, 2) void down_quad_kernel(
    const __bf16* __restrict__ w2s, const __bf16* __restrict__ w2f, const __bf16* __restrict__ b_down,
    const int32_t* __restrict__ item_start, const int32_t* __restrict__ group_off, const int32_t* __restrict__ alist,
    const uint64_t* __restrict__ mask, const int32_t* __restrict__ offsets, const __bf16* __restrict__ H,
    __bf16* __restrict__ y, int T, int d, int E, int NG, int W, int rows_per_item, int row_shift, uint32_t w_bytes,
    uint32_t h_bytes, long long max_pairs, long long max_rmw, int walk_limit, int parts, int xs, float* __restrict__ partial) {
    constexpr QuadShape Q = quad_shape(PG);
    constexpr int QS = Q.QS, PS = Q.PS, KS = Q.KS, SPQ = Q.SPQ;
    constexpr int TPB = kDqTrip * SPQ / QS;             // loop trips per batch of 64 experts
    constexpr int kImage = KS * kDqTiles * 1024;        // one level of a stage's tiles
    constexpr int kBuf = 2 * kImage + QS * 512;         // both levels and the position codes
    static_assert((kDqTrip * KS) % R == 0 && (SPQ == 1 || SPQ == 2 || SPQ == 4), "loop trip");
    static_assert((kDqTrip * KS / PS) % 2 == 0, "register sets of the codes");
    extern __shared__ __attribute__((aligned(16))) char img[];  // [kDqTrip][kBuf]
    if (offsets[E] > max_pairs) return;  // dense enough for down_bf16_kernel
    const int NS = d / kDqCols;
    const DownTile tile = down_tile(blockIdx.x, NS, (T + kDqTokens - 1) / kDqTokens, parts, xs);
    const int t_base = tile.chunk * kDqTokens;
    if (t_base >= T || tile.part >= parts) return;
    if constexpr (PG > 4) {
        const int pairs = offsets[E];
        if (pairs <= max_rmw && pairs_are_less(pairs, group_off, T, E, NG, PG == 16 ? kTileCost128 : kTileCost64, walk_limit)) {
            static_assert(kChunk == kDqTokens && kDownCols == kDqCols && kDownWaves == kDqWaves, "the same tiles");
            constexpr int KS = PG == 16 ? 4 : 2, RN = 32 * KS;
            const int chunk = tile.chunk, slice = tile.slice;
            const __bf16* Hf = H;
            char* smem = img;
#include "down_rmw_walk.inc"
            return;
        }
    }
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int h = lane >> 5, c = lane & 31;
    const int col_w = tile.slice * kDqCols + wave * 32;
    // this workgroup's share of the walk (none where there are more parts than trips: it then writes zeros)
    const int n_stages = ((E + 4 * QS - 1) / (4 * QS)) * SPQ;
    const int all_trips = (n_stages + kDqTrip - 1) / kDqTrip, part_trips = (all_trips + parts - 1) / parts;
    const int trip0 = tile.part * part_trips, n_trips = min(all_trips, trip0 + part_trips);

    // ---- building: select group bg of the chunk (lane = token), k-step bk of every stage
    const int bg = wave & 1, bk = wave >> 1;
    const bool builds = KS == 4 || bk < KS;
    const int g = tile.chunk * 2 + bg, tok_b = g * kGroup + lane;
    const bool tok_ok = tok_b < T;
    const uint64_t* mrow = mask + (size_t)min(tok_b, T - 1) * W;
    const int32_t* grow = group_off + (size_t)min(g, NG) * E;
    // Per batch of 64 experts: this token's mask word, and in lane i the first H row of (expert 64 b + i, group g).
    uint64_t mw, mw_next;
    int rowv, is_next, go_next;
    auto load_batch = [&](int b, uint64_t& m_out, int& is_out, int& go_out) {
        m_out = mrow[min(b, W - 1)];
        const int ec = min(64 * b + lane, E - 1);
        is_out = item_start[ec];
        go_out = grow[ec];
    };
    const __amdgpu_buffer_rsrc_t h_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)H, 0, (int)h_bytes, kRawBuffer);
    u32x4 hreg[2][4];  // H pieces on their way: [stage parity][rank of the expert]
    uint32_t off[4];   // row offsets of the 1st .. 4th selected expert of the quad; 2^31: none
    uint32_t code[2];  // position codes: low half level 1, high half level 2
    constexpr uint32_t kNone = 0x80000000u;
    // Quad at position qb of the batch: its selected experts in ascending order, and for either level the code
    // first | second << 2 of their positions, repeated for the instruction's four groups (an unused
    // second place repeats the first; a level-2 code is never 0, since a third is 2 or 3).
    auto prepare = [&](int qb, uint32_t& code_out) {
        const uint32_t nib = (uint32_t)(mw >> (4 * qb)) & 15u;
        uint32_t o[4] = {kNone, kNone, kNone, kNone};
#pragma unroll
        for (int i = 3; i >= 0; --i) {
            const bool sel = (nib >> i) & 1u;
            const uint64_t bal = __ballot(sel);
            const uint32_t row0 = (uint32_t)__builtin_amdgcn_readlane(rowv, 4 * qb + i);
            const uint32_t row = __builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, row0)) << row_shift;
            if (i == 0) o[3] = sel ? o[2] : o[3];
            if (i <= 1) o[2] = sel ? o[1] : o[2];
            if (i <= 2) o[1] = sel ? o[0] : o[1];
            o[0] = sel ? row : o[0];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) off[i] = builds ? o[i] : kNone;
        const uint32_t l1 = (uint32_t)(0x498e4dcf498a4500ull >> (4 * nib)) & 15u;  // digit `nib` of the tables
        const uint32_t l2 = (uint32_t)(0xeff0f000a0000000ull >> (4 * nib)) & 15u;
        code_out = __umul24(l1, 0x1111u) | (__umul24(l2, 0x1111u) << 16);
    };
    // stage i of a trip (qbase: quad position of the trip's first); the stages of one quad share its offsets
    int qbase = 0;
    auto prepare_stage = [&](int i, uint32_t& cd) {
        if (i % SPQ != 0) cd = code[(i + 1) & 1];
        else prepare(qbase + QS * (i / SPQ) + (PG == 1 ? bk : 0), cd);
    };
    auto fetch = [&](int r, int i, u32x4 (&hr)[4]) {
        hr[r] = __builtin_amdgcn_raw_buffer_load_b128(h_rsrc, off[r], 16u * (uint32_t)(PG == 1 ? 0 : PS * (i % SPQ) + bk % PS), 0);
    };
    auto fetch_rest = [&](int i, u32x4 (&hr)[4], uint32_t cd) {  // the third and fourth, if any token has them
        if (__ballot(cd > 0xffffu) != 0) {
            fetch(2, i, hr);
            fetch(3, i, hr);
        }
    };
    // One base per buffer, so that every LDS offset fits its instruction.
    LdsChar* wdst[kDqTrip];  // lane = token 32 h + c of the group: tile 2 bg + h of the chunk
    const LdsChar *rd[kDqTrip], *cdp[kDqTrip];
#pragma unroll
    for (int b = 0; b < kDqTrip; ++b) {
        wdst[b] = (LdsChar*)img + b * kBuf + (((2 * bg + h) * KS + bk) * 64 + c) * 16;
        rd[b] = (LdsChar*)img + b * kBuf + lane * 16;
        cdp[b] = (LdsChar*)img + b * kBuf + 2 * kImage + c * 16;
        asm volatile("" : "+v"(rd[b]), "+v"(cdp[b]));
    }
    // Values (first, second) of the neurons 4 hh .. 4 hh + 3 of the piece, in the order of A lane half hh.
    auto write_tile = [&](int buf, int level, const u32x4 (&hr)[4]) {
        const u32x4 a = hr[2 * level], b = hr[2 * level + 1];
#pragma unroll
        for (int hh = 0; hh < 2; ++hh) {
            u32x4 o;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                o[2 * i] = __builtin_amdgcn_perm(b[2 * hh + i], a[2 * hh + i], 0x05040100u);
                o[2 * i + 1] = __builtin_amdgcn_perm(b[2 * hh + i], a[2 * hh + i], 0x07060302u);
            }
            *(LdsU32x4*)(wdst[buf] + level * kImage + 32 * hh * 16) = o;
        }
    };
    auto write_level1 = [&](int buf, const u32x4 (&hr)[4]) {
        if (builds) write_tile(buf, 0, hr);
    };
    auto write_rest = [&](int buf, const u32x4 (&hr)[4], uint32_t cd) {
        if (PG == 1 || bk == 0)  // of a quad's wavefronts one writes the codes: [quad][token % 32][tile]
            *(LdsU32*)((LdsChar*)img + buf * kBuf + 2 * kImage + (PG == 1 ? bk : 0) * 512 + (c * 4 + 2 * bg + h) * 4) = cd;
        if (builds && __ballot(cd > 0xffffu) != 0) write_tile(buf, 1, hr);
    };

    // ---- multiplying: 128 tokens x columns col_w .. col_w + 31
    const __amdgpu_buffer_rsrc_t w_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)w2s, 0, (int)w_bytes, kRawBuffer);
    const uint32_t a_voff = (uint32_t)((col_w / 32) * KS * 2048 + lane * 16);
    const uint32_t w_stage_bytes = (uint32_t)(d / 32) * KS * 2048;
    uint32_t a_stage = (uint32_t)(trip0 * kDqTrip) * w_stage_bytes;
    u32x4 aw[R][2];
    auto load_w = [&](int ks, int f, u32x4 (&w)[2]) {
        w[f] = __builtin_amdgcn_raw_buffer_load_b128(w_rsrc, a_voff + (uint32_t)((ks & 1) * 2048 + f * 1024),
                                                     a_stage + (uint32_t)(ks >> 1) * 4096u, 0);
        if (f == 1 && ks == KS - 1) a_stage += w_stage_bytes;
    };
    auto weights = [&](const u32x4 (&w)[2]) {
        return __builtin_shufflevector(__builtin_bit_cast(bf16x8, w[0]), __builtin_bit_cast(bf16x8, w[1]), 0, 1, 2, 3, 4, 5,
                                       6, 7, 8, 9, 10, 11, 12, 13, 14, 15);
    };
    auto read_tile = [&](int buf, int ks, int j, int level) {
        return *(const LdsBf16x8*)(rd[buf] + level * kImage + (j * KS + ks) * 1024);
    };
    auto read_code = [&](int buf, int quad) { return *(const LdsU32x4*)(cdp[buf] + quad * 512); };

    // ---- start-up: stages 0 .. 3 of the part requested, 0 and 1 written
    {
        int is0, go0;
        load_batch(trip0 / TPB, mw, is0, go0);
        load_batch(trip0 / TPB + 1, mw_next, is_next, go_next);
        rowv = is0 * rows_per_item + go0;
        if (!tok_ok || trip0 / TPB >= W) mw = 0;
    }
    qbase = QS * ((trip0 % TPB) * kDqTrip / SPQ);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        prepare_stage(i, code[i & 1]);
        fetch(0, i, hreg[i & 1]);
        fetch(1, i, hreg[i & 1]);
        fetch_rest(i, hreg[i & 1], code[i & 1]);
    }
#pragma unroll
    for (int q = 0; q < R - 1; ++q) {
        load_w(q % KS, 0, aw[q]);
        load_w(q % KS, 1, aw[q]);
    }
    f32x16 acc[kDqTiles];
    {
        const float bias = b_down && tile.part == 0 ? (float)b_down[col_w + c] : 0.0f;
#pragma unroll
        for (int j = 0; j < kDqTiles; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[j][r] = bias;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        write_level1(i, hreg[i & 1]);
        write_rest(i, hreg[i & 1], code[i & 1]);
        prepare_stage(i + 2, code[i & 1]);
        fetch(0, i + 2, hreg[i & 1]);
        fetch(1, i + 2, hreg[i & 1]);
        fetch_rest(i + 2, hreg[i & 1], code[i & 1]);
    }
    lds_barrier();
    bf16x8 bb[2][kDqTiles];  // A operands of the current k-step and of the next one
    u32x4 cdv[2];            // codes of the four tiles
#pragma unroll
    for (int j = 0; j < kDqTiles; ++j) bb[0][j] = read_tile(0, 0, j, 0);
    cdv[0] = read_code(0, 0);

    // Stage i of a trip multiplies buffer i, writes the tiles of the stage two ahead (requested two stages
    // ago) and requests those of the stage four ahead, whose offsets it works out.  The barrier of a stage
    // stands before its last k-step, which reads the first tiles of the next: every wavefront has then written
    // its part of that stage (a stage ago), and all have left the stage whose buffer is written next.
    int trip = trip0;
    for (;;) {
        // the stages prepared in trip t are those of trip t + 1: a new batch?
        if ((trip + 1) % TPB == 0) {
            const int b = (trip + 1) / TPB;
            mw = tok_ok && b < W ? mw_next : 0ull;
            rowv = is_next * rows_per_item + go_next;
            load_batch(b + 1, mw_next, is_next, go_next);
        }
        const int run_end = min(n_trips, ((trip + 1) / TPB + 1) * TPB - 1);
        qbase = QS * (((trip + 1) % TPB) * kDqTrip / SPQ);
        do {
#pragma unroll
            for (int q = 0; q < kDqTrip * KS; ++q) {
                const int i = q / KS, ks = q % KS;
                const int nb = ks < KS - 1 ? i : (i + 1) % kDqTrip, nks = ks < KS - 1 ? ks + 1 : 0;
                const u32x4 cd = cdv[q / PS % 2];
                const bool level2 = __ballot((cd[0] | cd[1] | cd[2] | cd[3]) > 0xffffu) != 0;
                bool flag[kDqTiles];
                bf16x8 b2[kDqTiles];
                __builtin_amdgcn_sched_barrier(0);
                // (at most one global load and two LDS operations between two matrix instructions)
#pragma unroll
                for (int n = 0; n < kDqTiles; ++n) {
                    acc[n] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(bb[q & 1][n], weights(aw[q % R]), acc[n], (int)cd[n], 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    if (n == 0 && level2) {
#pragma unroll
                        for (int j = 0; j < kDqTiles; ++j) {
                            flag[j] = __ballot(cd[j] > 0xffffu) != 0;
                            if (flag[j]) b2[j] = read_tile(i, ks, j, 1);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    if (ks == 0 && n == 1) write_level1((i + 2) % kDqTrip, hreg[i & 1]);
                    if (ks == 0 && n == 3) write_rest((i + 2) % kDqTrip, hreg[i & 1], code[i & 1]);
                    if (ks == 1 && n == 0) prepare_stage(i, code[i & 1]);
                    if (ks == 1 && n < 2) fetch(n, i, hreg[i & 1]);
                    if (ks == 1 && n == 3) fetch_rest(i, hreg[i & 1], code[i & 1]);
                    if (n == 1 || n == 2) load_w((q + R - 1) % KS, n - 1, aw[(q + R - 1) % R]);
                    if (n == 0 && nks % PS == 0) cdv[(q + 1) / PS % 2] = read_code(nb, nks / PS);
                    bb[(q + 1) & 1][n] = read_tile(nb, nks, n, 0);
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (level2) {
#pragma unroll
                    for (int j = 0; j < kDqTiles; ++j)
                        if (flag[j])
                            acc[j] = __builtin_amdgcn_smfmac_f32_32x32x32_bf16(b2[j], weights(aw[q % R]), acc[j], (int)cd[j], 0, 1);
                }
                if (ks == KS - 2) lds_barrier();
            }
            qbase += QS * kDqTrip / SPQ;
        } while (++trip < run_end);
        if (trip >= n_trips) break;
    }

    // lane (h, c) of tile j: column col_w + c of the tokens t_base + 32 j + 8 (r / 4) + 4 h + r % 4
#pragma unroll
    for (int j = 0; j < kDqTiles; ++j) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int t = t_base + 32 * j + 8 * (r / 4) + 4 * h + r % 4;
            if (t < T) {
                if (parts > 1) partial[((size_t)tile.part * T + t) * d + col_w + c] = acc[j][r];
                else y[(size_t)t * d + col_w + c] = (__bf16)acc[j][r];
            }
        }
    }
}

template <int PG, int R>
void launch_quad_t(const dmoe_layer& L, int T, const int32_t* item_start, const int32_t* group_off,
                   const int32_t* alist, const uint64_t* mask, const int32_t* offsets, const void* H, void* y,
                   long long max_pairs, long long max_rmw, int walk_limit, float* partial, hipStream_t s) {
    constexpr QuadShape Q = quad_shape(PG);
    constexpr size_t lds = std::max((size_t)kDqTrip * (2 * Q.KS * kDqTiles * 1024 + Q.QS * 512), PG > 4 ? kDownLds : 0);
    static std::once_flag attr_once;  // kernel attributes: once per process, thread-safe
    std::call_once(attr_once, [&] {
        (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&down_quad_kernel<PG, R>),
                                  hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    });
    const PackedLayout P = packed_layout(L);
    const char* pk = static_cast<const char*>(L.packed);
    const int NS = L.d_model / kDqCols, parts = down_parts(L, T);
    // An XCD takes two slices of the columns and half of the chunks where there are eight slices: what the XCDs
    // read of the weights and of H together is the least then (4096 tokens x 2048 experts of 8: 172 -> 166 us).
    const int xs = NS % 4 == 0 ? 4 : 1;
    const int row_bytes = 2 * h_row_neurons(L);
    int row_shift = 0;
    while ((1 << row_shift) < row_bytes) ++row_shift;
    launch_kernel(down_quad_kernel<PG, R>, down_grid(div_up(T, kDqTokens), NS, parts), 64 * kDqWaves, lds, s,
                  (const __bf16*)(pk + P.w2s), (const __bf16*)(pk + P.w2f), (const __bf16*)L.b_down, item_start, group_off,
                  alist, mask, offsets, (const __bf16*)H, (__bf16*)y, T, L.d_model, L.n_experts, div_up(T, kGroup),
                  div_up(L.n_experts, 64), up_rows_bf16(L), row_shift, (uint32_t)down_quad_w_bytes(L),
                  (uint32_t)(h_fragments(L, T) * 16 * row_bytes), max_pairs, max_rmw, walk_limit, parts, xs, partial);
}

// Density up to which the quads are taken against the dense kernel: a - b / E, where b stands for what a workgroup does
// before and after its walk.  The dense kernel has two workgroups per CU, which hide that behind each other's walks once there
// is more than one workgroup per CU; here there is one of twice the wavefronts.  Quads / dense, us, at 3.5, 8 and 10.5 %: rows of
// 64, 24298 tokens, d = 1280 (950 workgroups) 12 experts 60 / 44, 63 / 44, 66 / 43; 40 102 / 102, 114 / 105, 122 / 107; 80 174 / 189,
// 194 / 199, 214 / 201; 256 483 / 588, 565 / 608, 626 / 629; 4096 tokens, d = 2048 (256) 12 experts 21 / 20, 23 / 21, 24 / 20; 40
// 32 / 36, 37 / 36, 40 / 36; 256 131 / 158, 147 / 164, 161 / 168.  Of 48 neurons, 50432 tokens, d = 768, 80 experts 176 / 178, 196 / 184,
// 220 / 187.  Rows of 128 at 3, 5, 7 %, 24298 tokens, d = 1280, 12 experts 73 / 66, 76 / 67, 80 / 68; 24 114 / 149, 120 / 124,
// 124 / 122.  Of 8 neurons at 5, 10, 13.5 %: 9000 tokens, d = 1024, 650 experts 98 / 99, 111 / 101, 124 / 101, 2500 317 / 364,
// 366 / 379, 414 / 413; 4096 tokens, d = 2048, 650 56 / 63, 63 / 65, 71 / 67.
double quad_density(const dmoe_layer& L, int T) {
    struct Line {
        int pieces;
        double most, a, b, a_more, b_more;  // up to one workgroup per CU, and more of them
    };
    constexpr Line lines[] = {{1, 0.14, 0.165, 33.0, 0.165, 75.0}, {6, 0.11, 0.105, 1.8, 0.1, 5.0},
                              {8, 0.11, 0.125, 1.6, 0.125, 3.4}, {16, 0.075, 0.105, 0.45, 0.105, 1.1}};
    const int PG = quad_pieces(L.expert_size), wgs = div_up(T, kDqTokens) * (L.d_model / kDqCols);
    for (const Line& l : lines)
        if (l.pieces == PG) return std::min(l.most, wgs > 256 ? l.a_more - l.b_more / L.n_experts : l.a - l.b / L.n_experts);
    return 0.0;
}

// Density up to which the walk over the pairs (down_rmw.h) is a choice, where the walk over the experts is not divided.  Against
// the dense kernel alone (384 columns) pairs decide: 3 %.  Against the quads the tiles that they make decide, on the device
// (pair_walk_limit): how many there are depends on how evenly the pairs fall on the experts.  Experts of 64, uniform
// selections of 1.8 and 2.4 %, pairs / quads: 4096 tokens x 256, d = 2048 142 / 121 and 152 / 123 us; a router's selection of
// 2.7 %, 4254 tokens x 699, d = 1280: 215 / 354; of 1.3 %, 4137 tokens x 1030 experts of 96: 397 / 1100.
// With few experts, for which the dense kernel is ahead of the quads, pairs are taken as far as they are ahead of it when even: 50432
// tokens x 24, d = 768, rows of 64 at 0.4 / 0.8 % 69 / 83 us against 79, of 128 96 / 130 against 141.
constexpr double kPairDensity = 0.03;
bool pairs_alone(const dmoe_layer& L, int T) {
    return down_bf16_wide(L, T) || (L.n_experts < 32 && quad_density(L, T) < kPairDensity);
}
double rmw_density(const dmoe_layer& L, int T) {
    const int PG = quad_pieces(L.expert_size);
    if (PG == 1 || down_parts(L, T) > 1) return 0.0;
    if (pairs_alone(L, T) && !down_bf16_wide(L, T)) return PG == 16 ? 0.01 : 0.007;
    return kPairDensity;
}

// Cost of four chunks (pairs_are_less) up to which the pairs are taken, -1: whatever it is.  The quads take a time that is nearly proportional to
// the experts, the longer for each the more their weights exceed the L2s.  Uniform selections, density of equal times: rows of 64
// 9000 tokens x 500, d = 512 (33 MB of weights) 0.85 %, 4096 x 256, d = 2048 (67 MB) 1.2 %, 4254 x 699, d = 1280 (114 MB)
// 1.8 %, of 48 neurons 0.72 % at 256 workgroups, 0.8 to 0.95 % at 516 to 1032; rows of 128 50432 x 24, d = 768 (5 MB) 0.8 %, 4096 x 256, d = 2048 (134 MB) 1.3 %, 4254 x 699, d = 1280 (179 MB) 1.8 %.
int pair_walk_limit(const dmoe_layer& L, int T) {
    if (pairs_alone(L, T)) return -1;
    const int PG = quad_pieces(L.expert_size);
    const double mb = 2e-6 * L.n_experts * m_pad_of(L.expert_size) * L.d_model;
    const double per_expert = PG == 16 ? kTileCost128 * std::min(0.9, 0.62 + mb / 640.0)
                                       : std::min(10.4, 7.2 + mb / 36.0) * (PG == 6 ? 0.82 : 1.0);  // (6 pieces: fewer products)
    return (int)(4.0 * per_expert * L.n_experts);
}

}  // namespace

// Walks of the dense kernel from which this one is worth a launch that may be for nothing (us, estimated): 256 gated experts
// of 64 at 1200 tokens, a walk of 55, 7 % density: 59 against 70 us; 600 tokens, 30: 36 against 48.
constexpr double kQuadMinWalk = 50.0;

size_t down_quad_w_bytes(const dmoe_layer& L) {
    const int PG = quad_pieces(L.expert_size);
    if (L.dtype != DMOE_BF16 || down_x8_shape(L) || PG == 0) return 0;
    if (PG == 1 && down_walk_us(L) < kQuadMinWalk) return 0;  // never launched (down_quad_max_pairs)
    const QuadShape q = quad_shape(PG);
    return (size_t)div_up(div_up(L.n_experts, 4), q.QS) * q.SPQ * (L.d_model / 32) * q.KS * 2048;
}

void launch_pack_down_quad(const dmoe_layer& L, void* packed, hipStream_t s) {
    const PackedLayout P = packed_layout(L);
    char* pk = static_cast<char*>(packed);
    const float* scales = weights_fp8(L) ? (const float*)(pk + P.scales) : nullptr;
    const QuadShape q = quad_shape(quad_pieces(L.expert_size));
    const int stages = div_up(div_up(L.n_experts, 4), q.QS) * q.SPQ;
    launch_pack_columns(L, scales, (__bf16*)(pk + P.w2s), QuadMap{q, stages * q.KS * 2}, s);
}

// Pairs up to which this kernel is taken; 0: not launched.  A launch that finds nothing to do costs 4 us.
long long down_quad_max_pairs(const dmoe_layer& L, int T) {
    const int PG = quad_pieces(L.expert_size);
    if (!down_quad_w_bytes(L)) return 0;
    double density = 0.0;
    if (down_bf16_wide(L, T)) {
        // the dense kernel has a shape that fills the chip once, this one does not (16384 tokens x 512 experts
        // of 6, d = 768, 11 %: 88 us against 72)
        density = rmw_density(L, T);
    } else if ((PG != 1 && down_parts(L, T) <= 1) || down_walk_us(L, T) >= kQuadMinWalk) {
        density = std::max(quad_density(L, T), rmw_density(L, T));
    }
    return density > 0.0 ? (long long)(density * (double)T * (double)L.n_experts) : 0;
}

void launch_down_quad(const dmoe_layer& L, int T, const int32_t* item_start, const int32_t* group_off,
                      const int32_t* alist, const uint64_t* mask, const int32_t* offsets, const void* H, void* y,
                      float* partial, long long max_pairs, hipStream_t s) {
    LaunchTimer tm(kSlotDownRmw, s);
    const double rmw = rmw_density(L, T);
    const int walk_limit = rmw > 0.0 ? pair_walk_limit(L, T) : -1;
    const long long max_rmw = rmw > 0.0 ? (long long)(rmw * (double)T * (double)L.n_experts) : -1;
#define DMOE_QUAD(PG_, R_) \
    launch_quad_t<PG_, R_>(L, T, item_start, group_off, alist, mask, offsets, H, y, max_pairs, max_rmw, walk_limit, partial, s)
    switch (quad_pieces(L.expert_size)) {
    case 1: DMOE_QUAD(1, 8); break;
    case 6: DMOE_QUAD(6, 6); break;
    case 8: DMOE_QUAD(8, 8); break;
    default: DMOE_QUAD(16, 8); break;
    }
#undef DMOE_QUAD
}

}  // namespace dmoe
