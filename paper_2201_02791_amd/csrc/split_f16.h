// fp32 products on the fp16 matrix cores: two fp16 parts per number, three products per term.  The other split
// (split_bf16.h: three bf16 parts, six products) holds for any operands; this one for operands that a power of two brings
// into fp16's range, at half the matrix-core work and less of everything around it.
//
// A number is scaled so that the largest of its operand lies in 2^14 .. 2^15, rounded to fp16, and what is left (at most
// 2^-11 of the number, of either sign) is rounded to fp16 again: of the 24 bits of the number at most the last is lost.  The
// product of the two second parts, below 2^-22 of a product and 2^-25 of it in the mean, is left out.  Scaled numbers below
// 2^-2 lose more: the second part, and below 2^-14 the first, reach fp16's smallest numbers, which leave an error of up to
// 2^-25, 2^-39 of the largest number, whatever the number's own size.  A sum that rests on such numbers is the caller's to
// find and to form in another way.
// What the three products save is rounding: a sum is rounded 3 times per 16 terms instead of 6.  Relative error (2-norm) of
// dot products of K normally distributed terms against 64 bits, in 10^-7, three products / six / the fp32 instruction:
// K = 16: 0.85 / 0.36 / 0.75;  64: 1.15 / 1.12 / 1.44;  128: 1.44 / 1.66 / 2.03;  256: 1.90 / 2.40 / 2.86;  1024: 3.6 /
// 4.9 / 5.7.  So three products serve sums of 80 terms and more.  (With the fourth, and the products of second parts in sums of
// their own, 16 terms come to 0.76, which is what two parts of 11 bits leave: row_products.hip.)
//
// Infinities and NaN do not survive the split either, and numbers near fp32's limits cannot be scaled: operands that hold
// such are the caller's to send to the other split.  Conversion and matrix cores keep subnormal fp16 numbers.
#pragma once
#include "split_bf16.h"

typedef _Float16 split_halfx8 __attribute__((ext_vector_type(8)));
typedef _Float16 split_halfx2 __attribute__((ext_vector_type(2)));

struct Split2 { uint32_t w[2]; };      // leading and second parts of two numbers, packed

__device__ __forceinline__ Split2 split_pair_f16(float x, float y)
{
    const split_floatx2 v = {x, y};
    const split_halfx2 a = __builtin_convertvector(v, split_halfx2);
    // x - a in one instruction each (v_fma_mix_f32 reads the halves as they are packed)
    const split_floatx2 left = {__builtin_fmaf((float)a.x, -1.f, x), __builtin_fmaf((float)a.y, -1.f, y)};
    Split2 s;
    s.w[0] = __builtin_bit_cast(uint32_t, a);
    s.w[1] = __builtin_bit_cast(uint32_t, __builtin_convertvector(left, split_halfx2));
    return s;
}

// either split by its number of parts
template <int NP> __device__ __forceinline__ auto split_parts(float x, float y)
{
    if constexpr (NP == 2) return split_pair_f16(x, y);
    else return split_pair(x, y);
}
template <int NP> __host__ __device__ constexpr int split_terms() { return NP == 2 ? 3 : SPLIT_TERMS; }
// parts of A and B in term p: three parts smallest first, two parts in the order that frees A's second part first
template <int NP> __host__ __device__ constexpr int split_a(int p) { return NP == 2 ? (p == 0 ? 1 : 0) : (p == 0 ? 2 : p == 2 || p == 3 ? 1 : 0); }
template <int NP> __host__ __device__ constexpr int split_b(int p) { return NP == 2 ? (p == 2 ? 1 : 0) : (p == 1 ? 2 : p == 2 || p == 4 ? 1 : 0); }
template <int NP> __device__ __forceinline__ split_floatx16 split_product(uint4 a, uint4 b, split_floatx16 c)
{
    if constexpr (NP == 2)
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(split_halfx8, a), __builtin_bit_cast(split_halfx8, b), c, 0, 0, 0);
    else return split_mfma(a, b, c);
}
