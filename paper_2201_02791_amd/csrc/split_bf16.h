// fp32 products on the bf16 matrix cores, for the kernels whose operands are fp32.
//
// An fp32 number is the exact sum of three bf16 numbers: it rounded to nearest, what is left rounded to nearest, and what
// is left then.  What is left has either sign and at most half a unit of the part before: 2^-8 of the number and, after
// the second part, 2^-17.  Of the nine products of two such sums the six largest are formed; the three left out are below
// 2^-24 of the product, less than the rounding of one fp32 addition, and of either sign.  (Parts that are cut off instead
// of rounded leave out up to 7.8 x 2^-24 of it, always towards zero.)  All six accumulate in fp32, 16 terms per
// v_mfma_f32_32x32x16_bf16, so a sum is rounded 6 times per 16 terms where the fp32 instruction (v_mfma_f32_32x32x2_f32)
// rounds after every term or two.
//
// Why: the fp32 instruction delivers 157 TFLOP/s on this chip and the bf16 one 2.5 PFLOP/s; a sixth of that is 417.
//
// What does not survive the split: infinities (inf - inf), numbers that round to one (from 3.39e38 on) and sums that leave
// the fp32 range on the way.  All show as a result that is not finite, and the kernels form such results again with the
// fp32 instruction.  Conversion and matrix cores keep subnormal bf16 numbers; of a number below 2^-110 the last part can
// fall under the smallest of them, and at most 2^-134 of it is lost.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

typedef float split_floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 split_bf16x8 __attribute__((ext_vector_type(8)));

typedef __bf16 split_bf16x2 __attribute__((ext_vector_type(2)));
typedef float split_floatx2 __attribute__((ext_vector_type(2)));

// two numbers rounded to nearest even as one word of two bf16 numbers (a first): v_cvt_pk_bf16_f32
__device__ __forceinline__ uint32_t split_round(float a, float b)
{
    const split_floatx2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, split_bf16x2));
}

struct Split3 { uint32_t w[3]; };      // leading, middle and last parts of two numbers, packed

__device__ __forceinline__ Split3 split_pair(float x, float y)
{
    Split3 s;
    s.w[0] = split_round(x, y);
    const float x1 = x - __uint_as_float(s.w[0] << 16), y1 = y - __uint_as_float(s.w[0] & 0xffff0000u);
    s.w[1] = split_round(x1, y1);
    const float x2 = x1 - __uint_as_float(s.w[1] << 16), y2 = y1 - __uint_as_float(s.w[1] & 0xffff0000u);
    s.w[2] = split_round(x2, y2);
    return s;
}

// the six products of one 16-deep step, smallest first; term p multiplies part split_pa(p) of A by part split_pb(p) of B
__device__ __forceinline__ constexpr int split_pa(int p) { return p == 0 ? 2 : p == 1 ? 0 : p == 2 ? 1 : p == 3 ? 1 : 0; }
__device__ __forceinline__ constexpr int split_pb(int p) { return p == 0 ? 0 : p == 1 ? 2 : p == 2 ? 1 : p == 3 ? 0 : p == 4 ? 1 : 0; }
constexpr int SPLIT_TERMS = 6;

__device__ __forceinline__ split_floatx16 split_mfma(uint4 a, uint4 b, split_floatx16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(split_bf16x8, a), __builtin_bit_cast(split_bf16x8, b), c, 0, 0, 0);
}

__device__ __forceinline__ bool split_not_finite(float x) { return !(__builtin_fabsf(x) <= 3.402823466e38f); }
