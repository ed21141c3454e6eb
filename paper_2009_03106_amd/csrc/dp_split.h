// float32 products on the bf16 matrix instruction: every float32 operand is taken apart into three bf16 numbers,
//     x = b1 + b2 + b3      b1 = bf16(x), b2 = bf16(x - b1), b3 = x - b1 - b2     (round to nearest even)
// exactly: 24 significant bits are 3 x 8, and the two differences are exact in float32.  Of the nine products the six
// largest are kept (b1 b1', b1 b2', b2 b1', b2 b2', b1 b3', b3 b1').  b2 reaches 2^-8 of x and b3 2^-17, so the three
// that are dropped are together at most 2^-24 of |x x'|, the rounding of one float32 product, and below 2^-26 for 97 of
// 100 pairs.  Six v_mfma_f32_32x32x16_bf16 take 192 cycles of a SIMD for 16 values of k, eight
// v_mfma_f32_32x32x2_f32 take 512.
//
// b3 of an operand below 2^-110 would lie under the smallest bf16, of a float32 subnormal b1 as well.  So the operands
// are multiplied by 2^24 (kSplitScale) before they are split and the sums by 2^-48 (kSplitUnscale): every part is then zero or
// at least 2^-125, and the split is exact down to the smallest float32 subnormal.  The price is the top of the range:
// operands from 2^104 on and sums from 2^80 on are infinite or NaN here, as infinities and NaN are themselves.  The
// kernels look for that in their finished sums (SplitCheck) and form them again with the float32 instruction, straight from
// memory: with every sum of a launch formed again 32 examples of 512 x (768, 768) take 0.43 ms for the Gram norms instead of
// 0.12 and 1.5 ms for the clipped sum instead of 0.12.
#pragma once
#include "dp_common.h"

namespace dpk {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr float kSplitScale = 0x1p24f, kSplitUnscale = 0x1p-48f;

// two values, scaled: their b1, b2 and b3, packed in pairs (x0 in bits 15:0)
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

// Whether one of the sums has to be formed again in float32: infinite or NaN.
struct SplitCheck {
    uint32_t top = 0u;
    __device__ __forceinline__ void add(float v) { top = max(top, __float_as_uint(v) & 0x7fffffffu); }
    __device__ __forceinline__ bool suspect() const { return top >= 0x7f800000u; }
};

}  // namespace dpk
