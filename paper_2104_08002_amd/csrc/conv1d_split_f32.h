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
__device__ __forceinline__ unsigned pack_bf16(float lo, float hi) {  // two floats to nearest even
    return __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{lo, hi}, bf16x2));
}
// no float rounds past the largest bfloat16; NaN comes out as a number here and stays NaN in what is left
__device__ __forceinline__ float within_bf16(float v) { return __builtin_amdgcn_fmed3f(v, -0x1.fep127f, 0x1.fep127f); }

// v = h + m + l.  h and m: 8 significant bits each, rounded to nearest even; l: what is left, which fits 6 bits.
// |m| <= 2^-8 |v| and |l| <= 2^-17 |v|, so the products left out later (m l, l m, l l) are at most 2^-24 of the whole, one
// half unit in the last place of an FP32 product.  (With h cut off they reached 2^-22, all with the sign of the whole:
// 2.35e-7 in a layer of equal values, x = w = 1 + 2^-7 - 2^-16; now 2.3e-10.)  The sum of the parts is exact while |v| is
// at least 2^-110; below that the lowest bits fall under bfloat16's smallest number, 2^-133.
struct Split8 {
    u32x4 h, m, l;
};
__device__ __forceinline__ Split8 split8(const float (&v)[8]) {
    Split8 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float a = v[2 * i], b = v[2 * i + 1];
        r.h[i] = pack_bf16(within_bf16(a), within_bf16(b));
        const float ra = a - __uint_as_float(r.h[i] << 16);
        const float rb = b - __uint_as_float(r.h[i] & 0xffff0000u);
        r.m[i] = pack_bf16(ra, rb);
        r.l[i] = pack_hi(ra - __uint_as_float(r.m[i] << 16), rb - __uint_as_float(r.m[i] & 0xffff0000u));
    }
    return r;
}

__device__ __forceinline__ f32x4 mfma(u32x4 a, u32x4 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// transposing LDS read: 16 lanes hand in the addresses of 8 bytes each and get these 16 rows of four elements transposed
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;
__device__ __forceinline__ u32x2 read_tr(const u32x2* p) {
    return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4*)p));
}

// keeps the compiler from knowing how a running index came about (or it keeps one register per address that it could be)
__device__ __forceinline__ void opaque(int& v) {
#ifndef HOSTMODEL
    asm volatile("" : "+v"(v));
#endif
}

constexpr size_t kLdsAll = 160 * 1024;

// Shortest sum taken, and the only rule: what has more terms and fits in LDS runs here, for any number of channels,
// filters, columns and samples.  (A rule that asked how many samples there are would give a sample other bits in another
// batch.)
// Error: the instruction's additions cut off, once per step, where the FP32 instruction rounds to nearest, once per four
// products.  Norm of the error against 64 bits in 1e-8, FP32 instruction and three parts: normal values 2.5 and 3.6 (1
// product), 5.4 and 3.1 (8), 7.4 and 3.4 (16), 10 and 3.8 (31); tracks of 80 % zeros, whose sums have a fifth of the
// products, 2.5 and 3.6 (1), 3.3 and 3.4 (8), 4.0 and 3.4 (16), 5.1 and 3.5 (31).
// Time, forward with S = 51, d = 8 on FP32 instruction and three parts, at 1000, 60000 and 960000 columns: C = K = 15 22.9
// and 16.2, 24.0 and 22.1, 226 and 130 us; C = K = 12 18.9 and 16.1, 20.0 and 21.9, 177 and 123; C = K = 4 10.6 and 9.0,
// 10.9 and 12.1, 83 and 63 (four channels are multiplied as eight, twelve as sixteen: slower where one wave of workgroups
// just fills the chip, faster on either side).  Weight gradient, C = K = 15: 24.3 and 9.5, 31.7 and 21.1, 246 and
// 125 us.
constexpr long kMinTerms = 16;

// The six products of a step start from zero, smallest first, and their sum is added to the running one in an ordinary
// FP32 addition.  Chained through the running sums themselves the matrix instruction's additions lost more than the
// FP32 instruction's did: error of a weight gradient of 3.4 million terms against 64 bits 2.9e-5 so, 8.2e-6 with
// v_mfma_f32_16x16x4_f32.
constexpr int kPartA[6] = {2, 0, 1, 1, 0, 0}, kPartB[6] = {0, 2, 1, 0, 1, 0};

// What a chain of n additions of independent terms rounds off, in roundings of the whole sum: partial sums grow as the
// root of their number, so their squares add up to this many of the last one's.
inline double chain_roundings(long n) { return n > 1 ? 0.5 * static_cast<double>(n + 1) - 1.0 / static_cast<double>(n) : 0.0; }

}  // namespace sp
}  // namespace conv1d
