// Float32 operands on the bf16 matrix cores: each float32 value x is split into
// three bf16 values h + m + l (round to nearest each, 8 significand bits each:
// the sum is x to 24 bits for |x| >= 2^-109), and a product of two split
// operands keeps the six terms down to 2^-16 of the leading one,
// hh + (hm + mh) + (mm + hl + lh); the dropped terms are below a float32
// rounding.  Six bf16 matrix ops do the work of 16 (32x32x16) float32 ones in
// 6/16 of their time.  k_conv_mfma_split sums the leading term and the five
// small ones in accumulators of their own, so the large accumulator is rounded
// once per matrix op and not six times; k_conv_mfma_res and k_bwd_dw_split,
// whose registers hold no second set, keep one and add the small terms first.
//
// Operands below 2^-109 (1.5e-33) keep fewer bits, since the last planes leave
// bf16's range: a layer whose input is of size 2^-110 came out 3.5e-7 from
// float64, 2^-112 1.3e-6, 2^-120 3.4e-4 (normal sizes 1.0e-7 to 1.2e-7; the
// float32 instruction 2.3e-7 to 3.0e-7 down to 2^-120).
//
// Values that are not finite, or that round up to infinity in bf16, turn the
// sums they enter into NaN (inf - inf in the split).  Each kernel says how such
// results get the value that float32 arithmetic gives.
#pragma once

#include "rn_device.hpp"

namespace rn {
namespace dev {

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

// bf16 pairs rounded to nearest even, and the float32 values of a pair (a shift
// and a mask; converting element by element back would round each again).
__device__ inline uint32_t round_pair(float x, float y) {
    typedef float floatx2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{x, y}, bf16x2));
}
__device__ inline float pair_lo(uint32_t p) { return __uint_as_float(p << 16); }
__device__ inline float pair_hi(uint32_t p) { return __uint_as_float(p & 0xffff0000u); }

// The three bf16 planes of four values.  `rest`: the largest magnitude of what
// the leading planes leave; infinite once a finite value's rounded up to
// infinity (an infinity leaves NaN, which the maximum passes over).
__device__ inline void split4(const floatx4 v, bf16x4 &h, bf16x4 &m, bf16x4 &l, float &rest) {
    uint32_t p[3][2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        float x = v[2 * i], y = v[2 * i + 1];
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) {
            p[pl][i] = round_pair(x, y);
            x -= pair_lo(p[pl][i]);
            y -= pair_hi(p[pl][i]);
            if (pl == 0) rest = fmaxf(fmaxf(fabsf(x), fabsf(y)), rest);
        }
    }
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    h = __builtin_bit_cast(bf16x4, u32x2{p[0][0], p[0][1]});
    m = __builtin_bit_cast(bf16x4, u32x2{p[1][0], p[1][1]});
    l = __builtin_bit_cast(bf16x4, u32x2{p[2][0], p[2][1]});
}

__device__ inline void split4(const floatx4 v, bf16x4 &h, bf16x4 &m, bf16x4 &l) {
    float rest = 0.f;
    split4(v, h, m, l, rest);
}

// The same for every float32: the leading plane of a finite value is finite
// (clamped to the largest bf16), so its planes add up to it; an infinity is
// infinite in its leading plane and NaN in the others, NaN is NaN in all.
__device__ inline bool is_finite(float v) { return (__float_as_uint(v) & 0x7f800000u) != 0x7f800000u; }

__device__ inline void split4_any(const floatx4 v, bf16x4 &h, bf16x4 &m, bf16x4 &l) {
    constexpr float kMost = 0x1.fep127f;              // largest finite bf16
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    uint32_t p[3][2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        float x = v[2 * i], y = v[2 * i + 1];
        p[0][i] = round_pair(is_finite(x) ? __builtin_amdgcn_fmed3f(x, -kMost, kMost) : x,
                             is_finite(y) ? __builtin_amdgcn_fmed3f(y, -kMost, kMost) : y);
#pragma unroll
        for (int pl = 1; pl < 3; ++pl) {
            x -= pair_lo(p[pl - 1][i]);
            y -= pair_hi(p[pl - 1][i]);
            p[pl][i] = round_pair(x, y);
        }
    }
    h = __builtin_bit_cast(bf16x4, u32x2{p[0][0], p[0][1]});
    m = __builtin_bit_cast(bf16x4, u32x2{p[1][0], p[1][1]});
    l = __builtin_bit_cast(bf16x4, u32x2{p[2][0], p[2][1]});
}
constexpr float kWide = 0x1.ffp127f;                  // the smallest float32 that rounds to infinity

// 0 while every value seen was finite, NaN after one that was not.
__device__ inline float nonfinite(float v, float seen) { return fmaf(v, 0.0f, seen); }

}  // namespace dev
}  // namespace rn
