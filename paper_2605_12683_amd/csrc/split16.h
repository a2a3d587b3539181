// fp32 matrix products on the bf16 matrix cores by splitting (internal to libdeer, not part of the
// ABI).
//
// A float x is exactly hi + mid + lo, hi = bf16(x), mid = bf16(x - hi), lo = x - hi - mid (8 + 8 + 8
// significant bits, rounded to nearest, the differences exact), for every x down to 2^-109 (below, lo
// and then mid are subnormal): bf16 has float's exponent, so nothing is scaled and entries of any sizes
// meet in one product.  (Two fp16 parts take half the instructions but hold 22 bits, and one scale for
// a whole operand loses small entries, which then is seen where latents differ in scale.)
// A product of two such operands takes six matrix instructions, lo hi + mid mid + hi lo,
// mid hi + hi mid, hi hi in this order, with fp32 products and sums; the dropped mid lo, lo mid and
// lo lo are together below 2^-23 of the largest such product, 2^-25 as a rule and of either sign.
// Against 64 bits the sums are as near as those of the fp32 instruction or nearer (it rounds once per
// four terms), and a power of two on a row or column of an operand gives the same bits times it.  The
// time is 3/7 of its: 16 instructions of 16 x 16 x 32 in bf16 take 127 ns on a SIMD, 16 of
// 16 x 16 x 4 in fp32 222 ns.
// A float above bf16's largest (3.39e38) rounds to an infinite hi and so to NaN, as infinities do.
#pragma once

#include "common.h"

namespace deer {

typedef uint32_t v4u __attribute__((ext_vector_type(4)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v2f __attribute__((ext_vector_type(2)));

// D = A B + acc for one 16 x 16 x 32 tile; lane (g, c) supplies eight k slots of row c of A and
// of column c of B and holds acc[4 g + r][c].  Any assignment of k to slots is allowed if A and
// B agree on it.
__device__ __forceinline__ v4f mfma_b(v4u a, v4u b, v4f acc) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), acc, 0, 0, 0);
}

__device__ __forceinline__ uint32_t cvt_pair(float x0, float x1) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector((v2f){x0, x1}, v2bf));
}

// hi, mid and lo of two consecutive k slots, packed
__device__ __forceinline__ void split_pair(float x0, float x1, uint32_t (&part)[3]) {
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const uint32_t p = part[q] = cvt_pair(x0, x1);
        x0 -= __uint_as_float(p << 16);   // exact
        x1 -= __uint_as_float(p & 0xffff0000u);
    }
}

// the same of a value known to more than float's bits, rounded once, to 24 bits
__device__ __forceinline__ void split_pair_f64(double x0, double x1, uint32_t (&part)[3]) {
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        const uint32_t p = part[q] = cvt_pair((float)x0, (float)x1);
        x0 -= (double)__uint_as_float(p << 16);
        x1 -= (double)__uint_as_float(p & 0xffff0000u);
    }
}

// sum over the four lane groups (lanes c, c + 16, c + 32, c + 48)
__device__ __forceinline__ float group_sum(float v) {
    auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(p[0]) + __uint_as_float(p[1]);
    auto q = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(q[0]) + __uint_as_float(q[1]);
}

}  // namespace deer
