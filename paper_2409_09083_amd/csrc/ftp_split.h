// An fp32 number as the sum of three bfloats (device code).
#pragma once
#include "ftp_device.h"

namespace ftp {

// two fp32 numbers rounded to bfloats (nearest, ties to even), the first in the low half: v_cvt_pk_bf16_f32
__device__ __forceinline__ uint32_t pack_bf16(float a, float b)
{
    typedef float v2f __attribute__((ext_vector_type(2)));
    typedef __bf16 v2b __attribute__((ext_vector_type(2)));
    const v2f v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, v2b));
}

// Operands are split at 2^24 times their size, so that the lowest plane of the smallest fp32 numbers still is a normal bfloat
// (unscaled, numbers below 2^-110 lost low bits: at 2^-118 9e-6 of their size, at 2^-126 2e-3); sums of products come out at
// 2^48 times theirs.
constexpr float kSplitScale = 16777216.0f, kSplitUnscale = 1.0f / (kSplitScale * kSplitScale);

// Three bfloats whose sum is the number, for two numbers at once (one dword per plane, low half the first).  Not for
// numbers above the largest bfloat, infinities and NaN: their planes add up to NaN or infinity.
__device__ __forceinline__ void split3(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l)
{
    h = pack_bf16(a, b);
    a -= __uint_as_float(h << 16); b -= __uint_as_float(h & 0xFFFF0000u);       // exact
    m = pack_bf16(a, b);
    a -= __uint_as_float(m << 16); b -= __uint_as_float(m & 0xFFFF0000u);       // exact
    l = pack_bf16(a, b);
}

}  // namespace ftp
