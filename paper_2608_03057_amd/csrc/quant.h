// Code decisions shared by the activation and the weight quantizer.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tasq {

// Correctly rounded x / d for many x and one d: Markstein's iteration
// (P. Markstein, "Computation of elementary functions on the IBM RISC
// System/6000 processor", 1990).  r = RN(1/d); q = x r is within two ulp of
// the quotient; a residual x - q d in one FMA and q + residual r in another
// give a faithful q, and the same step on a faithful q gives RN(x/d), d and
// the quotient being far from overflow and underflow.  Five instructions
// against eleven of a general division: the code pass of 4096x2240
// activations 9.8 -> 9.3 us, the quantizer of a 4608x1152 weight 11.1 -> 10.2
// (with its row kept in registers); large tensors stay bound by memory.
//
// Out of range, exact is false and the caller divides.  Where x itself is so
// small (about 2^-103) that the residual loses bits, the quotient is below
// 2^-42 and may be off in its last bits, which decide no code: beside a z of
// 2^-18 and more it vanishes in the sum, and with a smaller z the sum, next to
// zero, rounds to 0 and floors to 0 or -1, all of them code 0.
struct Divider {
    float d, r;
    bool exact;

    __device__ __forceinline__ explicit Divider(float divisor) : d(divisor)
    {
        exact = d >= 0x1p-60f && d <= 0x1p60f;
        r = __fdiv_rn(1.0f, d);
    }

    __device__ __forceinline__ float operator()(float x) const
    {
        float q = __fmul_rn(x, r);
        q = __fmaf_rn(__fmaf_rn(-q, d, x), r, q);
        return __fmaf_rn(__fmaf_rn(-q, d, x), r, q);
    }
};

// Four whole numbers clamped to [0, 255] (NaN: 0) and stored as Q - 128,
// first in the low byte: v_cvt_pk_u8_f32 clamps, converts and inserts.
__device__ __forceinline__ uint32_t pack_codes(float a, float b, float c, float d)
{
    uint32_t u = __builtin_amdgcn_cvt_pk_u8_f32(a, 0, 0u);
    u = __builtin_amdgcn_cvt_pk_u8_f32(b, 1, u);
    u = __builtin_amdgcn_cvt_pk_u8_f32(c, 2, u);
    u = __builtin_amdgcn_cvt_pk_u8_f32(d, 3, u);
    return u ^ 0x80808080u;
}

}  // namespace tasq
