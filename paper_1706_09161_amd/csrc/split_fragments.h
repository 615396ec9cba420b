// split_fragments.h -- device pieces shared by the kernels that run FP32
// contractions on the BF16 matrix cores (fractional_far.hip).  Not part of the public ABI.
//
// An FP32 value is the exact sum of three BF16 values, x = h + m + l with
// h = bf16(x), m = bf16(x - h), l = x - h - m (round to nearest even; the two
// differences are exact and the last one fits 8 bits), so
//   K C = K_h C_h + (K_h C_m + K_m C_h) + (K_h C_l + K_m C_m + K_l C_h) + ...
// where the three products left out are at most 2^-26 of the first.  Weights
// are split from their FP64 values (27 bits).  The first product goes into
// "main" accumulators, the five others, at most 2^-8 of it, into a
// "correction" accumulator of their own: a main accumulator is then rounded
// once per 16 products instead of six times.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "lbm_internal.h"

namespace lbm {
namespace split {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
// 4 floats at any 4-byte aligned address (global loads need no more)
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// Two values split into their three BF16 planes, packed pairwise.
__device__ __forceinline__ void split3_pair(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l)
{
    h = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
    const float ra = a - __uint_as_float(h << 16), rb = b - __uint_as_float(h & 0xffff0000u);
    m = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{ra, rb}, bf16x2));
    const float sa = ra - __uint_as_float(m << 16), sb = rb - __uint_as_float(m & 0xffff0000u);
    l = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{sa, sb}, bf16x2));
}

// The three planes of 8 consecutive values, as one MFMA operand each.
struct Frag3 {
    bf16x8 h, m, l;
};

__device__ __forceinline__ void split3_8(const float (&v)[8], u32x4& h, u32x4& m, u32x4& l)
{
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        uint32_t hp, mp, lp;
        split3_pair(v[2 * p], v[2 * p + 1], hp, mp, lp);
        h[p] = hp;
        m[p] = mp;
        l[p] = lp;
    }
}

// s + e = a + b exactly
__device__ __forceinline__ void two_sum(float a, float b, float& s, float& e)
{
#pragma clang fp contract(off)
    s = a + b;
    const float t = s - a;
    e = (a - (s - t)) + (b - t);
}

// The same splits of a value given as an unevaluated sum a + ea: the third
// plane takes the part that FP32 rounding would drop.
__device__ __forceinline__ void split3_pair(float a, float ea, float b, float eb, uint32_t& h, uint32_t& m, uint32_t& l)
{
    h = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{a, b}, bf16x2));
    const float ra = a - __uint_as_float(h << 16), rb = b - __uint_as_float(h & 0xffff0000u);
    m = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{ra, rb}, bf16x2));
    const float sa = (ra - __uint_as_float(m << 16)) + ea, sb = (rb - __uint_as_float(m & 0xffff0000u)) + eb;
    l = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{sa, sb}, bf16x2));
}

__device__ __forceinline__ bf16x8 as_bf16(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

template <bool CFIRST>
__device__ __forceinline__ f32x16 mfma32(bf16x8 c, bf16x8 t, f32x16 acc)
{
    if constexpr (CFIRST) return __builtin_amdgcn_mfma_f32_32x32x16_bf16(c, t, acc, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_32x32x16_bf16(t, c, acc, 0, 0, 0);
}

// The fractional sum of one output from its definition, in FP32 (boundary
// columns not included): the value of an output whose split sum is not
// finite.  The split of an infinite (or larger than the largest BF16) value
// is not finite in every plane and would turn infinities into NaN.  A NaN
// ends the sum.
__device__ __forceinline__ float plain_sum(const float* gen0, int k_lo, int k_hi, const float* c, int64_t stride, int j)
{
    float acc = 0.f;
#pragma unroll 1
    for (int k = k_lo; k < k_hi; ++k) {
        acc = fmaf(gen0[j - k], c[(int64_t)k * stride], acc);
        if (acc != acc) break;
    }
    return acc;
}

__device__ __forceinline__ bool not_finite(float v) { return (__float_as_uint(v) & 0x7f800000u) == 0x7f800000u; }

}  // namespace split
}  // namespace lbm
