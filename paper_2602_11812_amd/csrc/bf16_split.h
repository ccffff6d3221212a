// An fp32 value as the exact sum of three bf16 values: its top 8 significant bits, the top 8 of what is left, and the rest
// (at most 8 more bits, since fp32 has 24).  bf16 has fp32's exponent range, so every piece is representable (the last
// of a value below 2^-110 loses bits); products of two pieces are exact in fp32, which is what lets the bf16 matrix cores
// accumulate fp32-grade dot products.
//
// Of the nine products of two values' pieces the six largest are taken.  What the other three (middle x last, last x middle, last x last)
// amount to depends on how the pieces are cut.  Cut off (split3_bits), the lower pieces have the value's sign: at most 2^-21 of a product
// is lost, 2^-24.5 on average, always towards zero.  Rounded to nearest (split3_pair_nearest): at most 2^-24, of either
// sign.  Device-side header.
#pragma once
#include <hip/hip_runtime.h>

namespace egtp {
namespace {

// the three pieces as fp32 bit patterns with the low 16 bits clear (bf16 = the high half)
__device__ __forceinline__ void split3_bits(float f, unsigned &hi, unsigned &mid, unsigned &lo)
{
    hi = __float_as_uint(f) & 0xffff0000u;
    const float r1 = f - __uint_as_float(hi);
    mid = __float_as_uint(r1) & 0xffff0000u;
    const float r2 = r1 - __uint_as_float(mid);
    lo = __float_as_uint(r2) & 0xffff0000u;
}

typedef __attribute__((ext_vector_type(8))) __bf16 split_bf16x8;
typedef __attribute__((ext_vector_type(4))) unsigned split_u32x4;

// the upper halves of two neighbours in one register
__device__ __forceinline__ unsigned pack_halves(unsigned even, unsigned odd)
{
    return __builtin_amdgcn_perm(odd, even, 0x07060302u);
}

// two neighbours, packed piece by piece
__device__ __forceinline__ void split3_pair(float even, float odd, unsigned &hi, unsigned &mid, unsigned &lo)
{
    const float e1 = even - __uint_as_float(__float_as_uint(even) & 0xffff0000u);
    const float o1 = odd - __uint_as_float(__float_as_uint(odd) & 0xffff0000u);
    hi = pack_halves(__float_as_uint(even), __float_as_uint(odd));
    mid = pack_halves(__float_as_uint(e1), __float_as_uint(o1));
    lo = pack_halves(__float_as_uint(e1 - __uint_as_float(__float_as_uint(e1) & 0xffff0000u)),
                     __float_as_uint(o1 - __uint_as_float(__float_as_uint(o1) & 0xffff0000u)));
}

// the same, each piece what is left rounded to the nearest bf16 (values above the largest bf16 have an infinite one)
__device__ __forceinline__ void split3_pair_nearest(float even, float odd, unsigned &hi, unsigned &mid, unsigned &lo)
{
    typedef __attribute__((ext_vector_type(2))) float f32x2;
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
    auto round = [](float e, float o) { return __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{e, o}, bf16x2)); };
    hi = round(even, odd);
    const float e1 = even - __uint_as_float(hi << 16), o1 = odd - __uint_as_float(hi & 0xffff0000u);
    mid = round(e1, o1);
    // (at most eight bits are left)
    lo = pack_halves(__float_as_uint(e1 - __uint_as_float(mid << 16)), __float_as_uint(o1 - __uint_as_float(mid & 0xffff0000u)));
}

}  // namespace
}  // namespace egtp
