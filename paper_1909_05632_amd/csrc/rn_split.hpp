// Float32 operands on the bf16 matrix cores: each float32 value x is split into
// three bf16 values h + m + l (round to nearest each, 8 significand bits each:
// the sum is x to 24 bits, at every exponent a float32 product can carry), and
// a product of two split operands keeps the six terms down to 2^-16 of the
// leading one, hh + (hm + mh) + (mm + hl + lh); the dropped terms are below a
// float32 rounding.  The leading term and the five small ones are summed in
// accumulators of their own, so the large accumulator is rounded once per
// matrix op and not six times.  Six bf16 matrix ops do the work of 16 (32x32x16)
// float32 ones in 6/16 of their time.
//
// Values that are not finite, or that round up to infinity in bf16, turn the
// sums they enter into NaN (inf - inf in the split).  The kernels detect any
// result that is not finite and recompute that one output in plain float32, so
// infinities and NaN come out as from float32 arithmetic.
#pragma once

#include "rn_device.hpp"

namespace rn {
namespace dev {

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

// The three bf16 planes of four values.
__device__ inline void split4(const floatx4 v, bf16x4 &h, bf16x4 &m, bf16x4 &l) {
    h = __builtin_convertvector(v, bf16x4);
    const floatx4 r = v - __builtin_convertvector(h, floatx4);
    m = __builtin_convertvector(r, bf16x4);
    l = __builtin_convertvector(r - __builtin_convertvector(m, floatx4), bf16x4);
}

// 0 while every value seen was finite, NaN after one that was not.
__device__ inline float nonfinite(float v, float seen) { return fmaf(v, 0.0f, seen); }

__device__ inline bool is_finite(float v) { return (__float_as_uint(v) & 0x7f800000u) != 0x7f800000u; }

}  // namespace dev
}  // namespace rn
