// One-time weight packing: device code shared by the kernels that lay the expert matrices out as operands.
//
// Every operand keeps eight values of one output position together.  A thread fills whole positions, so the index
// arithmetic is paid once for 8 or 64 values, and it reads 16 bytes (8 of one-byte weights) at a time
// from the caller's matrices, which need no particular alignment.  (One value per thread, read and written 2 bytes
// at a time, all operands of 256 gated experts of 64, d = 2048, took 488 us against 185 now, fully 8-bit 892 against 243;
// 2048 gated experts of 8: 1239 against 424.)
#pragma once

#include "dmoe_internal.h"
#include "mfma.h"

namespace dmoe {

typedef __bf16 bf16x8_any __attribute__((ext_vector_type(8), aligned(2)));
typedef uint8_t u8x8 __attribute__((ext_vector_type(8)));
typedef uint8_t u8x8_any __attribute__((ext_vector_type(8), aligned(1)));

// Eight consecutive elements from `flat` on of expert e's matrix `which` (0 up, 1 gate, 2 down): as bf16 numbers (8-bit
// weights as scale * e4m3(byte), exact: the scales are powers of two), or the raw bytes of 8-bit weights.
template <typename OUT>
struct Packed8;
template <>
struct Packed8<__bf16> {
    typedef bf16x8 type;
    static __device__ __forceinline__ type load(const void* w, const float* scales, int fp8, int which, int e, size_t flat) {
        if (!fp8) return *reinterpret_cast<const bf16x8_any*>(static_cast<const __bf16*>(w) + flat);
        const u8x8 b = *reinterpret_cast<const u8x8_any*>(static_cast<const uint8_t*>(w) + flat);
        const float s = scales[3 * e + which];
        type v;
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = (__bf16)(s * e4m3_value(b[i]));
        return v;
    }
};
template <>
struct Packed8<uint8_t> {
    typedef u8x8 type;
    static __device__ __forceinline__ type load(const void* w, const float*, int, int, int, size_t flat) {
        return *reinterpret_cast<const u8x8_any*>(static_cast<const uint8_t*>(w) + flat);
    }
};

// Operands of the down-projections: blocks [lane 0..63][8] over d / MAP::kCols column tiles, whose eight values are
// eight rows (expert, neuron) of w_down[E][m][d] in one output column.  A thread takes eight columns of a
// block's lane group: eight loads of eight columns each, turned in registers.  Neighbouring threads take
// neighbouring columns.  MAP (any block without its column tile has an index b < map.blocks):
//   row(b, group, s, e, neuron): value s of lane group `group`;  lane(col): lane of column col of a tile within a
//   group;  block(b, ct, n_ct): the block's place in the output.
template <typename OUT, class MAP>
__global__ void pack_columns_kernel(const void* __restrict__ w_down, const float* __restrict__ scales, int fp8,
                                    OUT* __restrict__ out, int E, int m, int d, MAP map, size_t n_units) {
    typedef typename Packed8<OUT>::type Vec;
    constexpr int kGroups = 64 / MAP::kCols;
    const int n8 = d / 8, n_ct = d / MAP::kCols;
    size_t u = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (; u < n_units; u += stride) {
        const int c8 = (int)(u % n8), group = (int)(u / n8 % kGroups), b = (int)(u / n8 / kGroups);
        const int ct = 8 * c8 / MAP::kCols, col = 8 * c8 % MAP::kCols;
        Vec v[8];
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            int e, neuron;
            map.row(b, group, s, e, neuron);
            const bool valid = e < E && neuron < m;
            v[s] = valid ? Packed8<OUT>::load(w_down, scales, fp8, 2, e, ((size_t)e * m + neuron) * d + 8 * c8) : Vec{};
        }
        OUT* dst = out + (map.block(b, ct, n_ct) * 64 + group * MAP::kCols) * 8;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            Vec o;
#pragma unroll
            for (int s = 0; s < 8; ++s) o[s] = v[s][j];
            *reinterpret_cast<Vec*>(dst + MAP::lane(col + j) * 8) = o;
        }
    }
}
template <typename OUT, class MAP>
inline void launch_pack_columns(const dmoe_layer& L, const float* scales, OUT* out, const MAP& map, hipStream_t s) {
    const size_t n_units = (size_t)map.blocks * (64 / MAP::kCols) * (L.d_model / 8);
    launch_kernel(pack_columns_kernel<OUT, MAP>, (int)std::min<size_t>((n_units + 255) / 256, 8192), 256, 0, s, L.w_down,
                  scales, weights_fp8(L), out, L.n_experts, L.expert_size, L.d_model, map, n_units);
}

}  // namespace dmoe
