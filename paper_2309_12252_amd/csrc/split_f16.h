// fp32 products on the fp16 matrix cores: every factor as the sum of two fp16 numbers (Ootomo and Yokota, "Recovering single precision accuracy from
// Tensor Cores while surpassing the FP32 theoretical peak performance", 2022).
//
// x = hi + lo + e with hi = fp16(x), lo = fp16(x - hi), |e| <= 2^-23 |x| while lo is a normal number, i.e. for |x| from 2^-2 to 65504: factors
// are scaled there by powers of two first, by their largest entry (one 2^-k of that is known to 2^-38 of it at best).  J, the left factor of the reductions, is
// not scaled: 2^-25 absolute.  A product is lo*hi + hi*lo + hi*hi, added in this order into one fp32
// accumulator (lo*lo is below 2^-22 of the product).  Measured against 64 bits, 400 products 16 x K by K x 16 of normal and of
// positive entries (2-norm): K = 32 8.0e-8 to 9.0e-8, K = 64 8.8e-8 to 9.6e-8; the fp32 matrix instructions give 1.03e-7 and
// 1.43e-7 there (they round the sum after every four terms).  Without the scaling 1.2e-7 to 1.7e-6.
// Time: a 16 x 16 x 32 product takes three instructions of 18 cycles and two vector instructions for each element that is
// split, in the place of eight instructions of 32 cycles.  Vector and matrix instructions of a SIMD do not overlap, of either
// kind (12 + 48 of them: 430 and 227 cycles apart, 657 together).
#pragma once
#include "deer_common.h"

namespace deer {
namespace {

using Half8 = _Float16 __attribute__((ext_vector_type(8)));
using Half4 = _Float16 __attribute__((ext_vector_type(4)));
using Half2 = _Float16 __attribute__((ext_vector_type(2)));
using F32x4 = float __attribute__((ext_vector_type(4)));
using F32x8 = float __attribute__((ext_vector_type(8)));

// hi and lo parts of the eight entries a lane supplies to a contraction of 32
struct Split8 {
    Half8 hi, lo;
};

__device__ __forceinline__ unsigned split_hi(float a, float b) { return __builtin_bit_cast(unsigned, Half2{(_Float16)a, (_Float16)b}); }

// x - hi, x mixed with the fp16 number in one instruction (the multiplier is one the compiler cannot see, or it would convert and subtract)
__device__ __forceinline__ float split_diff(float x, _Float16 hi) {
    float one = 1.0f;
    asm("" : "+s"(one));
    return __builtin_fmaf(x, one, -(float)hi);
}

__device__ __forceinline__ unsigned split_lo(float a, float b, unsigned hi) {
    const Half2 h = __builtin_bit_cast(Half2, hi);
    return split_hi(split_diff(a, h[0]), split_diff(b, h[1]));
}

// what the two parts leave out (exact: 0 or the last bit)
__device__ __forceinline__ unsigned split_rest(float a, float b, unsigned hi, unsigned lo) {
    const Half2 h = __builtin_bit_cast(Half2, hi), l = __builtin_bit_cast(Half2, lo);
    return split_hi((a - (float)h[0]) - (float)l[0], (b - (float)h[1]) - (float)l[1]);
}

// Two accumulators of 16 rows (rows 4g .. 4g + 3 of each in lane group g) as operand B of a contraction over those 32 rows: entry j
// < 4 of lane group g is row 4g + j of the first, j >= 4 row 4g + j - 4 of the second.  Operand A takes its columns in the same order.
__device__ __forceinline__ Split8 split8(F32x4 a, F32x4 b) {
    const F32x8 x = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
    Split8 s;
    s.hi = __builtin_convertvector(x, Half8);
    F32x8 r;
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = split_diff(x[i], s.hi[i]);
    s.lo = __builtin_convertvector(r, Half8);
    return s;
}

// Weights that stay in registers, scaled so that the largest is below 2^8, in three parts.  One that is much smaller keeps its digits all the same: lo and rest are
// 2^11 times what they stand for (|e| <= 2^-36 for the three, 2^-25 for two unscaled ones) and go with split_small() of the other factor.
struct Split8Weights {
    Half8 hi, lo, rest;
};
__device__ __forceinline__ Split8Weights split8_weights(F32x4 a, F32x4 b) {
    const F32x8 x = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
    Split8Weights s;
    s.hi = __builtin_convertvector(x, Half8);
    F32x8 r;
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = (x[i] - (float)s.hi[i]) * 2048.f;
    s.lo = __builtin_convertvector(r, Half8);
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] -= (float)s.lo[i];
    s.rest = __builtin_convertvector(r, Half8);
    return s;
}
__device__ __forceinline__ Half8 split_small(Half8 hi) { return hi * (_Float16)(1.f / 2048.f); }

__device__ __forceinline__ F32x4 mfma16(Half8 a, Half8 b, F32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }

// Factors whose hi*hi sums are exact (Ozaki, Ogita, Oishi and Rump, "Error-free transformations of matrix multiplication", 2012).  A matrix instruction drops what lies 24 bits or so below its largest product, and fp16 numbers that change slowly leave out
// the same there at many points in a row: small (4e-8 of the sum) but the same error again and again, where rounded fp32 sums scatter.  So hi lies on a grid: weights
// below 2^8 on multiples of 2^-6 (their eleven bits from 2^5 on), the other factor below 2^13 on multiples of 2^5; products are multiples of 1/2, and a sum below 2^23 is exact.
// What hi leaves out comes in lo and rest: lo*lo and hi*rest count here.
__device__ __forceinline__ float split_grid_weight(float x) { return (x + 1.5f * (1 << 17)) - 1.5f * (1 << 17); }
struct Split8Grid {
    Half8 hi, lo, rest;
};
__device__ __forceinline__ Split8Grid split8_grid(F32x4 a, F32x4 b) {
    F32x8 x = __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7), h;
    Split8Grid s;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        h[i] = (x[i] + 1.5f * (1 << 28)) - 1.5f * (1 << 28);
        x[i] -= h[i];
    }
    s.hi = __builtin_convertvector(h, Half8);
    s.lo = __builtin_convertvector(x, Half8);
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = split_diff(x[i], s.lo[i]);
    s.rest = __builtin_convertvector(x, Half8);
    return s;
}

// The same for a contraction of 16, i.e. one accumulator, with instructions for 16.  (Two of those for 32 that take (lo | hi) and (hi | lo) of A and (hi | lo) of B cost
// four moves a factor more.  Never one for 16 after one for 32 on the same accumulator: the compiler puts no wait between two lengths, and
// what it adds to is not there yet.)
struct Split4 {
    Half4 hi, lo;
};
__device__ __forceinline__ Split4 split4(F32x4 x) {
    Split4 s;
    s.hi = __builtin_convertvector(x, Half4);
    F32x4 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = split_diff(x[i], s.hi[i]);
    s.lo = __builtin_convertvector(r, Half4);
    return s;
}
__device__ __forceinline__ F32x4 mfma16(Half4 a, Half4 b, F32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x16f16(a, b, c, 0, 0, 0); }
// c + A B
__device__ __forceinline__ F32x4 split_product(const Split4& a, const Split4& b, F32x4 c) { return mfma16(a.hi, b.hi, mfma16(a.hi, b.lo, mfma16(a.lo, b.hi, c))); }

// where entry (row, 32 s + c) of a matrix goes as operand A: lane, and the place among the lane's eight
__device__ __forceinline__ int split_lane(int row, int c) { return 16 * ((c % 16) / 4) + row % 16; }
__device__ __forceinline__ int split_place(int c) { return 4 * (c / 16) + c % 4; }

// exponent e with |x| < 2^e (0 for 0, infinities and NaN)
__device__ __forceinline__ int exponent(float x) { return __builtin_amdgcn_frexp_expf(x); }

// A running product of split factors, Q <- A Q, whose columns are scaled by powers of two of their own: a column is 2^e times what it stands for.
// Columns decay and grow along a chunk; below 2^-2 the lo parts of a split lose digits, above 65504 the hi parts overflow.
struct ColumnScale {
    static constexpr int kStart = 4;   // the product starts from 2^kStart I
    int e;
    float down;
    __device__ __forceinline__ void reset(bool split) {
        e = split ? kStart : 0;
        down = split ? 1.f / (1 << kStart) : 1.f;
    }
    // does this lane's column, whose largest entry is m, want another scale (nothing to do for 0, infinities and NaN)
    __device__ __forceinline__ bool off(float m) const { return (m < 8.f || m > 2048.f) && m > 0.f && m < __builtin_huge_valf(); }
    // ... and the factor that goes to the column
    __device__ __forceinline__ float next(float m) {
        const int k = off(m) ? 7 - __builtin_amdgcn_frexp_expf(m) : 0;
        e += k;
        down = __builtin_amdgcn_ldexpf(1.f, -e);
        return __builtin_amdgcn_ldexpf(1.f, k);
    }
};

// largest of the four lane groups' values, in every lane
__device__ __forceinline__ float max_groups(float x) {
    unsigned u = __float_as_uint(x);
    const auto q = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    const float s = fmaxf(__uint_as_float(q[0]), __uint_as_float(q[1]));
    u = __float_as_uint(s);
    const auto w = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    return fmaxf(__uint_as_float(w[0]), __uint_as_float(w[1]));
}

}  // namespace
}  // namespace deer
