// float32 products on the bf16 matrix instruction: every float32 operand is taken apart into three bf16 numbers,
//     x = b1 + b2 + b3      b1 = bf16(x), b2 = bf16(x - b1), b3 = x - b1 - b2     (round to nearest even)
// exactly: 24 significant bits are 3 x 8, and the two differences are exact in float32.  Of the nine products the six
// down to 2^-18 of the largest are kept (b1 b1', b1 b2', b2 b1', b2 b2', b1 b3', b3 b1'); the three that are dropped
// are together below 2^-26 of |x x'|, a quarter of the rounding of one float32 product.  Six v_mfma_f32_32x32x16_bf16
// take 192 cycles of a SIMD for 16 values of k, eight v_mfma_f32_32x32x2_f32 take 512.
//
// Two things the three numbers cannot carry: infinities, NaN and |x| >= 2^128 - 2^119 (b1 is not finite, the
// differences are NaN), and numbers so small that b3 falls below the smallest bf16 subnormal.  Both show in the
// finished sums: the first makes them NaN or infinite, the second matters only where a sum itself is tiny.  The
// kernels therefore look at their sums once (SplitCheck) and form them again with the float32 instruction.
#pragma once
#include "dp_common.h"

namespace dpk {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// two values: their b1, b2 and b3, packed in pairs (x0 in bits 15:0)
__device__ __forceinline__ void split2(float x0, float x1, uint32_t& p1, uint32_t& p2, uint32_t& p3) {
#pragma clang fp contract(off)        // x may come from a product: the differences are to be taken from its rounded value
    p1 = pack_bf16(x0, x1);
    const float r0 = x0 - bf16_lo(p1), r1 = x1 - bf16_hi(p1);
    p2 = pack_bf16(r0, r1);
    p3 = pack_bf16(r0 - bf16_lo(p2), r1 - bf16_hi(p2));
}

// The sum over 16 k of x y.  The matrix instruction does not round its sum to nearest (on sums of one sign it loses about
// 2^-25 of the accumulator each time), so it starts from zero, takes the smallest products first, and only its last
// step is as large as the result; the callers keep their running sums with float32 additions.
__device__ __forceinline__ f32x16 split_mfma(const bf16x8 (&x)[3], const bf16x8 (&y)[3]) {
    f32x16 t = {};
    t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[2], y[0], t, 0, 0, 0);
    t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[0], y[2], t, 0, 0, 0);
    t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[1], y[1], t, 0, 0, 0);
    t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[1], y[0], t, 0, 0, 0);
    t = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[0], y[1], t, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[0], y[0], t, 0, 0, 0);
}

// Whether one of the sums has to be formed again in float32: not finite, or not zero but below 2^-96.
struct SplitCheck {
    uint32_t top = 0u, low = 0xffffffffu;
    __device__ __forceinline__ void add(float v) {
        const uint32_t u = __float_as_uint(v) & 0x7fffffffu;
        top = max(top, u); low = min(low, u - 1u);           // zero wraps to the top of the range
    }
    __device__ __forceinline__ bool suspect() const { return top >= 0x7f800000u || low < (uint32_t)((127 - 96) << 23) - 1u; }
};

}  // namespace dpk
