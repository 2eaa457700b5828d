// fp32 products on the bf16 matrix cores, for the kernels whose operands are fp32.
//
// An fp32 number is the exact sum of three bf16 numbers: its leading 8 significant bits, the next 8 and the last 8
// (each part is cut off, not rounded, so the subtractions are exact and all parts have the number's sign).  Of the nine
// products of two such sums the six largest are formed; the three left out are below 2^-24 of the product, less than
// the rounding of one fp32 addition.  All six accumulate in fp32, 16 terms per v_mfma_f32_32x32x16_bf16, so a sum
// is rounded 6 times per 16 terms where the fp32 instruction (v_mfma_f32_32x32x2_f32) rounds after every term or two.
//
// Why: the fp32 instruction delivers 157 TFLOP/s on this chip and the bf16 one 2.5 PFLOP/s; a sixth of that is 417.
//
// What does not survive the split: infinities (inf - inf) and sums that leave the fp32 range on the way.  Both show as a
// result that is not finite, and the kernels form such results again with the fp32 instruction.  Parts of numbers below
// 2^-102 can fall under the smallest normal bf16 number; what is lost there is below 2^-126 in magnitude.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

typedef float split_floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 split_bf16x8 __attribute__((ext_vector_type(8)));

// the upper halves of two fp32 words as one word of two bf16 numbers (a first)
__device__ __forceinline__ uint32_t split_pack(uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); }

struct Split3 { uint32_t w[3]; };      // leading, middle and last parts of two numbers, packed

__device__ __forceinline__ Split3 split_pair(float x, float y)
{
    const uint32_t xb = __float_as_uint(x), yb = __float_as_uint(y);
    const float x1 = x - __uint_as_float(xb & 0xffff0000u), y1 = y - __uint_as_float(yb & 0xffff0000u);
    const uint32_t x1b = __float_as_uint(x1), y1b = __float_as_uint(y1);
    const float x2 = x1 - __uint_as_float(x1b & 0xffff0000u), y2 = y1 - __uint_as_float(y1b & 0xffff0000u);
    Split3 s;
    s.w[0] = split_pack(xb, yb);
    s.w[1] = split_pack(x1b, y1b);
    s.w[2] = split_pack(__float_as_uint(x2), __float_as_uint(y2));
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
