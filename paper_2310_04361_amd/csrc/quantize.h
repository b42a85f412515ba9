// Row-wise quantisation to E4M3 with a power-of-two scale (the first paragraph of ffn_x8.hip).
#pragma once

#include "mfma.h"

namespace dmoe {

// E4M3 code of v (|v| <= 448): round to nearest, ties to even.  The grid step at magnitude a is
// 2^(e - 3) with e = max(floor(log2 a), -6) (-6: the subnormal range), a / step is exact, rintf
// rounds it to nearest-even, and a result of 16 steps is the next power of two.
__device__ __forceinline__ uint32_t e4m3_code(float v, float* value) {
    const float a = fabsf(v);
    int e = (int)((__float_as_uint(a) >> 23) & 0xffu) - 127;
    e = max(e, -6);
    float r = rintf(ldexpf(a, 3 - e));   // 0 .. 16
    *value = copysignf(ldexpf(r, e - 3), v);
    uint32_t code;
    if (r < 8.0f) {
        code = (uint32_t)r;              // zero or subnormal (only at e == -6)
    } else {
        if (r == 16.0f) {
            e += 1;
            r = 8.0f;
        }
        code = ((uint32_t)(e + 7) << 3) | ((uint32_t)r - 8u);
    }
    return code | (v < 0.0f ? 0x80u : 0u);
}

// Codes of eight values by the hardware converter.  For every bf16 number of magnitude up to
// 448 (the only inputs here: bf16 values times a power of two) v_cvt_pk_fp8_f32 returns the code
// of e4m3_code above -- checked exhaustively on the device, all 34754 inputs -- at a tenth of the
// instructions, so the kernels that need only the codes use it.
__device__ __forceinline__ uint2 e4m3_codes8(const float (&v)[8]) {
    int lo = __builtin_amdgcn_cvt_pk_fp8_f32(v[0], v[1], 0, false);
    lo = __builtin_amdgcn_cvt_pk_fp8_f32(v[2], v[3], lo, true);
    int hi = __builtin_amdgcn_cvt_pk_fp8_f32(v[4], v[5], 0, false);
    hi = __builtin_amdgcn_cvt_pk_fp8_f32(v[6], v[7], hi, true);
    return make_uint2((uint32_t)lo, (uint32_t)hi);
}

// Row t by one wavefront: codes, scale and, if wanted, the quantised values.
__device__ __forceinline__ void quantize_row(const __bf16* __restrict__ x, int t, int d, uint8_t* __restrict__ x8,
                                             float* __restrict__ xscale, __bf16* __restrict__ xhat) {
    const int lane = threadIdx.x & 63;
    const __bf16* row = x + (size_t)t * d;
    float amax = 0.0f;
    for (int k = 8 * lane; k < d; k += 512) {
        const bf16x8 v = load8(row + k);
#pragma unroll
        for (int i = 0; i < 8; ++i) amax = fmaxf(amax, fabsf((float)v[i]));
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off, 64));
    // smallest power of two s with amax / s <= 448 = 0.875 * 2^9: amax = f * 2^ex, f in [0.5, 1)
    int s_exp = 0;
    if (amax > 0.0f && amax < INFINITY) {
        int ex;
        const float f = frexpf(amax, &ex);
        s_exp = f <= 0.875f ? ex - 9 : ex - 8;
        s_exp = min(max(s_exp, -100), 100);
    }
    if (lane == 0) xscale[t] = ldexpf(1.0f, s_exp);
    for (int k = 8 * lane; k < d; k += 512) {
        const bf16x8 v = load8(row + k);
        if (!xhat) {  // uniform: codes only
            float sv[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) sv[i] = ldexpf((float)v[i], -s_exp);
            *reinterpret_cast<uint2*>(x8 + (size_t)t * d + k) = e4m3_codes8(sv);
            continue;
        }
        uint32_t lo = 0, hi = 0;
        bf16x8 q;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            float val;
            const uint32_t code = e4m3_code(ldexpf((float)v[i], -s_exp), &val);
            if (i < 4) lo |= code << (8 * i); else hi |= code << (8 * (i - 4));
            q[i] = (__bf16)ldexpf(val, s_exp);   // exact: four significant bits
        }
        *reinterpret_cast<uint2*>(x8 + (size_t)t * d + k) = make_uint2(lo, hi);
        *reinterpret_cast<bf16x8*>(xhat + (size_t)t * d + k) = q;
    }
}

}  // namespace dmoe
