// bf16 down-projection and merge for SPARSE selections: work proportional to the executed
// (token, expert) pairs (Sec. 3.2; the merge the paper's kernel does with global atomics).
//
// down_bf16.hip and down_quad_bf16.hip sum over experts inside the matrix cores at a cost that hardly depends
// on how many experts a token selected; for H rows of 64 or 128 neurons it is cheaper, below a density
// of a per cent or two, to touch only the executed rows (down_quad_bf16.hip has the rule), and this form has
// no limit on the sizes it can address (down_rmw_bf16.hip).  The statements are in down_rmw_walk.inc.
//
// One workgroup per (128-token chunk, 256-column slice); KS = m_pad / 32 MFMA k-steps.
// The fp32 output tile Y[128][256] lives in LDS.  The eight wavefronts own 32 columns each, so
// no two wavefronts ever touch the same element and the merge is a plain read-add-write (LDS
// float atomics proved far slower).  All wavefronts walk the same list of tiles -- up to 32
// consecutive rows of one expert's part of H, all belonging to this chunk -- built once per
// batch of experts from the group offsets.
// Per tile and wavefront: D[32 cols][32 rows] = W2 slice * H_tile^T as 2 x 2 MFMA 16x16x32
// tiles with the tokens on the MFMA column axis, so a lane ends up with four consecutive output
// columns of ONE token: one 16-byte LDS read and write per MFMA tile, one row address per
// token.  The row stride of 260 floats spreads consecutive-token rows over the banks.
// Operands of the next kDepth tiles are kept in flight while the current one is merged.
// Weights: the 16x16x32 fragments w2f (also used by the small-token path); H rows as written by
// the up kernel (16-byte piece 4ks + q of a row = neurons 8(4ks + q) .. +7 = the k values of lane
// group q in k-step ks).  RN: neurons per H row (h_row_neurons).  Rows of one or two pieces have nothing for the
// other lane groups: those read, at every tile, the zeros that the packed weights of the first expert are there.
// (Rows of a size known only at run time and a zero chosen where the row is loaded, which waits for the load
// and ends the ring, against this, 1 % density, d = 768: 20000 tokens x 2048 experts of 24 1075 / 962 us; 50432
// tokens x 2048 experts of 8 2678 / 2368, x 1024 experts of 16 1341 / 1228.  All of those lanes at one address, or
// zeros chosen where they are used, 2539 and 2560 for the experts of 8.)
#pragma once

#include "dmoe_internal.h"
#include "mfma.h"

namespace dmoe {

constexpr int kDownWaves = 8;
constexpr int kDownCols = kDownWaves * 32;     // output columns per workgroup
constexpr int kDownBatch = 128;                // experts per tile-list batch
constexpr int kDownTilesPerExpert = (kChunk + 31) / 32;       // 32-row tiles per (chunk, expert)
constexpr int kDownStride = kDownCols + 4;     // LDS row stride in floats
constexpr size_t kDownLds = sizeof(float) * kChunk * kDownStride +
                            sizeof(int2) * kDownBatch * kDownTilesPerExpert;

}  // namespace dmoe
