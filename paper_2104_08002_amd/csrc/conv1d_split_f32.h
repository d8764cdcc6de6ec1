// FP32 operands of the bf16 matrix instructions: every float is cut into three bfloat16 numbers whose sum it is.
#pragma once

#include "conv1d_internal.h"

namespace conv1d {
namespace sp {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;

__device__ __forceinline__ unsigned pack_hi(float lo, float hi) {  // upper halves of two floats, lo in the low half
    return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
}

// v = h + m + l.  h: the upper 8 significant bits, cut off (no value overflows by it); m: the next 8, rounded to nearest
// even, so that the products left out later (m l, l m, l l: 2^-25 of h h) have no preferred sign; l: what is left, which
// fits 8 bits.  Exact while v is at least 2^-110 (below that l drops under bfloat16's smallest number).
struct Split8 {
    u32x4 h, m, l;
};
__device__ __forceinline__ Split8 split8(const float (&v)[8]) {
    Split8 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float a = v[2 * i], b = v[2 * i + 1];
        r.h[i] = pack_hi(a, b);
        const float ra = a - __uint_as_float(__float_as_uint(a) & 0xffff0000u);
        const float rb = b - __uint_as_float(__float_as_uint(b) & 0xffff0000u);
        const unsigned mm = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{ra, rb}, bf16x2));
        r.m[i] = mm;
        r.l[i] = pack_hi(ra - __uint_as_float(mm << 16), rb - __uint_as_float(mm & 0xffff0000u));
    }
    return r;
}

__device__ __forceinline__ f32x4 mfma(u32x4 a, u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// The six products of a step start from zero, smallest first, and their sum is added to the running one in an ordinary
// FP32 addition.  Chained through the running sums themselves the matrix instruction's additions lost more than the
// FP32 instruction's did: error of a weight gradient of 3.4 million terms against 64 bits 2.9e-5 so, 8.2e-6 with
// v_mfma_f32_16x16x4_f32.
constexpr int kPartA[6] = {2, 0, 1, 1, 0, 0}, kPartB[6] = {0, 2, 1, 0, 1, 0};

}  // namespace sp
}  // namespace conv1d
