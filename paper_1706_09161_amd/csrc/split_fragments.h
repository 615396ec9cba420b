// split_fragments.h -- device pieces shared by the kernels that run FP32
// contractions on the BF16 matrix cores (fractional_split.hip, fractional_far.hip).
// Not part of the public ABI.
//
// An FP32 value is the exact sum of three BF16 values, x = h + m + l with
// h = bf16(x), m = bf16(x - h), l = x - h - m (round to nearest even; the two
// differences are exact and the last one fits 8 bits) as long as l is no finer
// than BF16's smallest subnormal, 2^-133: for |x| from 2^-110 (8e-34) up.  Below,
// x is kept to 2^-134 absolute (a field scaled by 2^-114: relative L2 of the sum
// 1.3e-7 instead of 4.6e-8, by 2^-120 8e-6; the FP32 register kernels keep
// 4.6e-8).  Scaling C by 2^16 before the split keeps every bit down there, at two
// more instructions a pair: 1 to 3 % of every launch, 7 % at 2048^2.  So
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

__device__ __forceinline__ bf16x8 ld16(const uint16_t* p) { return as_bf16(*reinterpret_cast<const u32x4*>(p)); }

__device__ __forceinline__ Frag3 planes(const float (&v)[8])
{
    u32x4 h, m, l;
    split3_8(v, h, m, l);
    return {as_bf16(h), as_bf16(m), as_bf16(l)};
}

// C of a line block through a buffer descriptor: a load past its end (or at
// a negative k) returns zero or a neighbouring line's value and never faults,
// so ragged ends need no separate code, only a mask on k.
typedef __amdgpu_buffer_rsrc_t Rsrc;

__device__ __forceinline__ float ldf(Rsrc r, uint32_t boff)
{
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, boff, 0, 0));
}

// 8 consecutive k of a line from byte offset boff (ks4: bytes between k)
template <bool CONTIG>
__device__ __forceinline__ void load8(Rsrc r, uint32_t boff, uint32_t ks4, float (&v)[8])
{
    if constexpr (CONTIG) {
        const u32x4 a = __builtin_amdgcn_raw_buffer_load_b128(r, boff, 0, 0);
        const u32x4 b = __builtin_amdgcn_raw_buffer_load_b128(r, boff + 16, 0, 0);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[e] = __uint_as_float(a[e]);
            v[4 + e] = __uint_as_float(b[e]);
        }
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = ldf(r, boff + (uint32_t)e * ks4);
    }
}

// v[e] = 0 unless k_lo <= k + e < k_hi
__device__ __forceinline__ void mask8(float (&v)[8], int k, int k_lo, int k_hi)
{
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = (unsigned)(k + e - k_lo) < (unsigned)(k_hi - k_lo) ? v[e] : 0.f;
}

// Toeplitz operand of a lane: T(d0), T(d0 - 1), ..., T(d0 - 7) are the pair
// words W(d0), W(d0 - 2), W(d0 - 4), W(d0 - 6) of every plane; w points at
// W(d0) of the first plane, `plane` words lie between planes.
template <int NT>
__device__ __forceinline__ Frag3 toeplitz(const uint32_t* w, int plane)
{
    u32x4 h, m, l = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        h[p] = w[2 * p];
        m[p] = w[plane + 2 * p];
        if constexpr (NT == 6) l[p] = w[2 * plane + 2 * p];
    }
    return {as_bf16(h), as_bf16(m), as_bf16(l)};
}

// Sums of one wavefront: 32 lines x 64 outputs (two blocks c of 32), two main
// sets and the correction.  Along the contiguous axis rows are lines and
// columns outputs, along the others the reverse.
template <bool CONTIG, int NT>
struct Accumulators {
    f32x16 main_[2][2], corr[2];

    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int r = 0; r < 16; ++r) main_[0][c][r] = main_[1][c][r] = corr[c][r] = 0.f;
    }
    static __device__ __forceinline__ f32x16 mfma(bf16x8 c, bf16x8 t, f32x16 a)
    {
        if constexpr (CONTIG) return __builtin_amdgcn_mfma_f32_32x32x16_bf16(c, t, a, 0, 0, 0);
        else return __builtin_amdgcn_mfma_f32_32x32x16_bf16(t, c, a, 0, 0, 0);
    }
    // one step of 16 k: x the C operand, y0 and y1 the Toeplitz operands of the two blocks
    __device__ __forceinline__ void add(const Frag3& x, const Frag3& y0, const Frag3& y1, int set)
    {
        if constexpr (NT == 6) {
            corr[0] = mfma(x.l, y0.h, corr[0]);
            corr[1] = mfma(x.l, y1.h, corr[1]);
        }
        main_[set][0] = mfma(x.h, y0.h, main_[set][0]);
        if constexpr (NT == 6) {
            corr[0] = mfma(x.h, y0.l, corr[0]);
            corr[1] = mfma(x.h, y1.l, corr[1]);
        }
        main_[set][1] = mfma(x.h, y1.h, main_[set][1]);
        if constexpr (NT == 6) {
            corr[0] = mfma(x.m, y0.m, corr[0]);
            corr[1] = mfma(x.m, y1.m, corr[1]);
        }
        corr[0] = mfma(x.m, y0.h, corr[0]);
        corr[1] = mfma(x.m, y1.h, corr[1]);
        corr[0] = mfma(x.h, y0.m, corr[0]);
        corr[1] = mfma(x.h, y1.m, corr[1]);
    }
    // BOTH: set 1 of the main accumulators was used
    template <bool BOTH = true>
    __device__ __forceinline__ void total(f32x16 (&sum)[2]) const
    {
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int r = 0; r < 16; ++r) sum[c][r] = (BOTH ? main_[0][c][r] + main_[1][c][r] : main_[0][c][r]) + corr[c][r];
    }
};

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

// Boundary operands of a wavefront's tile: cols[0..63], cols[64..127] the two
// boundary columns at its outputs (LDS); C at the walls of its lines, in LDS
// (contiguous axis) or this lane's (other axes).
struct Boundary {
    const float *cols, *w0s, *wNs;
    float b0, bN;
};

// Adds the boundary columns (a rank-2 correction) and stores row groups
// [u_lo, u_hi) of the tile (u = 4 c + r / 4) that lie in the box: nl lines,
// outputs jw .. n - 1.  ls4, ks4: byte strides of lines and nodes.  REDO:
// values whose sum is not finite are formed again from the definition.
template <bool CONTIG, bool REDO>
__device__ __forceinline__ void store_tile(const SplitOp& op, const f32x16 (&sum)[2], int u_lo, int u_hi,
                                           const Boundary& bd, const float* Cb, float* Pb, int nl, int jw, int k_lo,
                                           int k_hi, uint32_t ls4, uint32_t ks4)
{
    const int n = op.n, N = n - 1;
    const int lane = threadIdx.x & 63, li = lane & 31, lh = lane >> 5;
    bool odd = false;
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        if (u < u_lo || u >= u_hi) continue;
        const int c = u >> 2, r4 = u & 3;
        const int row = 8 * r4 + 4 * lh;  // first of 4 accumulator rows; columns are li
        f32x4 x0, xN, y0, yN;             // boundary weights, wall values
        if constexpr (CONTIG) {
            x0 = bd.cols[32 * c + li];
            xN = bd.cols[64 + 32 * c + li];
            y0 = *reinterpret_cast<const f32x4*>(bd.w0s + row);
            yN = *reinterpret_cast<const f32x4*>(bd.wNs + row);
        } else {
            x0 = *reinterpret_cast<const f32x4*>(bd.cols + 32 * c + row);
            xN = *reinterpret_cast<const f32x4*>(bd.cols + 64 + 32 * c + row);
            y0 = bd.b0;
            yN = bd.bN;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int line = CONTIG ? row + e : li;
            const int j = jw + 32 * c + (CONTIG ? li : row + e);
            float v = sum[c][4 * r4 + e];
            odd = odd || not_finite(v);
            if (line < nl && j < n) {
                v = fmaf(x0[e], y0[e], v);
                v = fmaf(xN[e], yN[e], v);
                *reinterpret_cast<float*>(reinterpret_cast<char*>(Pb) + (uint32_t)line * ls4 + (uint32_t)j * ks4) = v;
            }
        }
    }
    if (!REDO || !__any(odd)) return;
#pragma unroll 1
    for (int o = 4 * u_lo; o < 4 * u_hi; ++o) {
        const int row = 8 * ((o >> 2) & 3) + 4 * lh + (o & 3), col = 32 * (o >> 4);
        const int line = CONTIG ? row : li, jl = col + (CONTIG ? li : row), j = jw + jl;
        if (line >= nl || j >= n) continue;
        float* out = reinterpret_cast<float*>(reinterpret_cast<char*>(Pb) + (uint32_t)line * ls4 + (uint32_t)j * ks4);
        if (!not_finite(*out)) continue;
        const float* c = reinterpret_cast<const float*>(reinterpret_cast<const char*>(Cb) + (uint32_t)line * ls4);
        const int64_t ks = ks4 / 4;
        float v = plain_sum(op.gen + N, op.upper_only ? max(k_lo, j) : k_lo, op.lower_only ? min(k_hi, j + 1) : k_hi, c,
                            ks, j);
        v = fmaf(bd.cols[jl], c[0], v);
        *out = fmaf(bd.cols[64 + jl], c[(int64_t)N * ks], v);
    }
}

}  // namespace split
}  // namespace lbm
