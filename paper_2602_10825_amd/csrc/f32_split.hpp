// fp32 products on the bf16 matrix cores.  A float is the sum x = h + m + l of three bf16 numbers, each what
// the ones before it leave, rounded to nearest: all 24 bits for |x| above 2^-110, whatever the other entries of its row or
// column are.  Of the nine products of two such sums six are formed,
//   x y ~= l h' + h l' + m m' + m h' + h m' + h h',
// with float accumulation; those left out are below 2^-24 |x y|, the rounding of one fp32 product.  Six
// v_mfma_f32_32x32x16_bf16 take 192 cycles where eight v_mfma_f32_32x32x2_f32 take 512, and an accumulator is rounded 6
// times per 16 terms instead of 8 times or more.  (Two f16 parts and three products take half of that, but a part has 5 bits of
// exponent: with operands scaled by powers of two, what is 2^17 below the largest of its row or tensor loses bits.)
// Where an entry is infinite, or above 3.389e38 and rounds to infinity, its other parts are not numbers, and neither is
// what they are multiplied into: the callers look for that in their sums, and for magnitudes at which parts are lost,
// and form those sums again with fp32 products.
#pragma once

#include "fc_common.hpp"

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// eight floats in three parts, each an operand of a 32x32x16 product
struct Split8 { u32x4_native h, m, l; };

// two floats -> their bf16 roundings, and what those leave
__device__ __forceinline__ uint32_t split_off(float& x0, float& x1) {
    const bf16x2_t v = {(__bf16)x0, (__bf16)x1};
    uint32_t u = __builtin_bit_cast(uint32_t, v);
    asm volatile("" : "+v"(u));                  // (or each half is converted once more for the difference)
    x0 -= __uint_as_float(u << 16);
    x1 -= __uint_as_float(u & 0xffff0000u);
    return u;
}
// elements 2 p and 2 p + 1
__device__ __forceinline__ void split_pair(Split8& s, int p, float x0, float x1) {
    s.h[p] = split_off(x0, x1);
    s.m[p] = split_off(x0, x1);
    const bf16x2_t v = {(__bf16)x0, (__bf16)x1};
    s.l[p] = __builtin_bit_cast(uint32_t, v);
}

__device__ __forceinline__ void split_mfma(const u32x4_native& a, const u32x4_native& b, f32x16_t& c) {
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

// Outside of 0 and 2^-100 <= |x| < 2^100.  Where one operand of a product has no such entry, what the smallest parts of the
// other one lose (below 2^-133) does not show in the scores.
__device__ __forceinline__ bool odd_magnitude(float x) {
    const uint32_t u = __float_as_uint(x) << 1;
    return u != 0u && u - (27u << 24) >= (200u << 24);
}
// Lanes where x is infinite, not a number (also where the compiler may assume that there are none) or 0 < |x| < 2^-90, of
// which parts are lost.
__device__ __forceinline__ uint64_t odd_sum(float x) {
    uint64_t lanes;
    asm("v_cmp_class_f32 %0, %1, %2" : "=s"(lanes) : "v"(x * 0x1p-36f), "v"(0x297));   // NaN, infinite, subnormal
    return lanes;
}
