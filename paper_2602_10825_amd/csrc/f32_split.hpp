// fp32 products on the f16 matrix cores.  A float that a power of two has brought to at most 2^15 is
// the sum x = h + l of two f16 numbers, each rounded to nearest: 22 bits and two signs, an error of at
// most 2^-23 |x|.  Of the four products of two such sums the three larger are formed,
//   x y ~= l h' + h l' + h h',
// with float accumulation; the one left out is below 2^-24 |x y|.  The scale is taken per row of an
// operand (or follows the largest entry seen, see the callers): entries below 2^-16 of their row's largest
// are held to 2^-40 of that one instead.  Three v_mfma_f32_32x32x16_f16 take 96 cycles where eight
// v_mfma_f32_32x32x2_f32 take 512, and an accumulator is rounded 3 times per 16 terms instead of 8 times
// or more.  (Three bf16 parts and six products need no scales but twice the matrix and twice the vector
// work: attention of 12 heads x 128, 2 x 1021 rows on 4083 clean keys 456 us against 357.)
#pragma once

#include "fc_common.hpp"

typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// eight scaled floats in two parts, each an operand of a 32x32x16 product
struct Split8 { u32x4_native h, l; };

// elements 2 p and 2 p + 1: x0 * scale, x1 * scale
__device__ __forceinline__ void split_pair(Split8& s, int p, float x0, float x1, float scale) {
    const f16x2_t hv = {(_Float16)(x0 * scale), (_Float16)(x1 * scale)};
    uint32_t h = __builtin_bit_cast(uint32_t, hv);
    asm volatile("" : "+v"(h));                  // (or each half is converted once more for the difference)
    const f16x2_t g = __builtin_bit_cast(f16x2_t, h);
    const f16x2_t lv = {(_Float16)__builtin_fmaf(x0, scale, -(float)g[0]), (_Float16)__builtin_fmaf(x1, scale, -(float)g[1])};
    s.h[p] = h;
    s.l[p] = __builtin_bit_cast(uint32_t, lv);
}

// The power of two that brings numbers of magnitude `most` to [2^14, 2^15) / 2^room, and its inverse.
__device__ __forceinline__ float split_scale(float most, float& inverse, int room = 0) {
    int e = __builtin_amdgcn_frexp_expf(most) + room;   // most = f 2^e, 1/2 <= f < 1; 0 for 0
    e = e < -100 ? -100 : e;
    inverse = __builtin_amdgcn_ldexpf(1.0f, e - 15);
    return __builtin_amdgcn_ldexpf(1.0f, 15 - e);
}
__device__ __forceinline__ float max_abs4(float m, const f32x4_t& x) {
    return fmaxf(fmaxf(fmaxf(m, fabsf(x[0])), fabsf(x[1])), fmaxf(fabsf(x[2]), fabsf(x[3])));
}

// |x| if that is finite and above m, else m
__device__ __forceinline__ float max_finite(float m, float x) {
    return fabsf(x) > m && fabsf(x) < __builtin_inff() ? fabsf(x) : m;
}

__device__ __forceinline__ void split_mfma(const u32x4_native& a, const u32x4_native& b, f32x16_t& c) {
    c = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
}
