// fp32 matrix products on the fp16 matrix cores by splitting (internal to libdeer, not part of
// the ABI).
//
// A float x in fp16's range is held as hi + lo, hi = fp16(x), lo = fp16(x - hi), both rounded to
// nearest (the difference is exact): 22 significant bits and a sign for lo, |x - hi - lo| <=
// 2^-23 of x's binade while lo is a normal number.  A product of two split operands takes three
// matrix instructions, lo hi + hi lo + hi hi in that order, each with fp32 products and sums; the
// dropped lo lo is below 2^-22.  Against 64 bits such a product of 64 terms is as near as the
// fp32 matrix instruction (whose 16 partial sums round more often) and takes 3/8 of its matrix
// time: 16 instructions of 16 x 16 x 32 in fp16 or bf16 take 127 ns on a SIMD, 16 of 16 x 16 x 4
// in fp32 222 ns.
//
// fp16 has 5 exponent bits, so operands are scaled by powers of two (exact) before they are
// split: the largest entry near the top of the range, where an entry needs to be 2^-17 of it
// before lo becomes subnormal (its error is then 2^-25 absolute, 2^-38 of the largest entry).
#pragma once

#include "common.h"

namespace deer {

typedef _Float16 v2h __attribute__((ext_vector_type(2)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef uint32_t v4u __attribute__((ext_vector_type(4)));

// D = A B + acc for one 16 x 16 x 32 tile; lane (g, c) supplies eight k slots of row c of A and
// of column c of B and holds acc[4 g + r][c].  Any assignment of k to slots is allowed if A and
// B agree on it.
__device__ __forceinline__ v4f mfma_h(v4u a, v4u b, v4f acc) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h, a), __builtin_bit_cast(v8h, b), acc, 0, 0, 0);
}

// -1 the compiler cannot see: x - float(h) then stays one mixed-precision multiply-add instead
// of a conversion and a subtraction
__device__ __forceinline__ float opaque_m1() {
    float m1 = -1.f;
    asm volatile("" : "+s"(m1));
    return m1;
}

// hi and lo of two consecutive k slots, packed
__device__ __forceinline__ void split_pair(float x0, float x1, float m1, uint32_t &hi, uint32_t &lo) {
    hi = __builtin_bit_cast(uint32_t, v2h{(_Float16)x0, (_Float16)x1});
    asm("" : "+v"(hi));   // one packed conversion (else the halves are converted again for lo)
    const v2h h = __builtin_bit_cast(v2h, hi);
    const v2h l = {(_Float16)__builtin_fmaf((float)h[0], m1, x0), (_Float16)__builtin_fmaf((float)h[1], m1, x1)};
    lo = __builtin_bit_cast(uint32_t, l);
}

// ---- three parts in bfloat16 -------------------------------------------------------------------------
// A float x is exactly hi + mid + lo, hi = bf16(x), mid = bf16(x - hi), lo = x - hi - mid (8 + 8 + 8
// significant bits, rounded to nearest, the differences exact), for every x of normal size down to
// 2^-109 (below, lo and then mid are subnormal): bf16 has float's exponent, so nothing is scaled and
// entries of any sizes meet in one product.  A product of two such operands takes six matrix
// instructions, lo hi + mid mid + hi lo, mid hi + hi mid, hi hi in this order, with fp32 products and
// sums; the dropped mid lo, lo mid and lo lo are together below 2^-23 of the largest such product, 2^-25
// as a rule and of either sign.  Against 64 bits the sums are nearer than those of the fp32 instruction, which rounds once per
// four terms; the time is 3/7 of its (16 instructions of 16 x 16 x 32 in bf16 take 127 ns on a SIMD, 16
// of 16 x 16 x 4 in fp32 222 ns).
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef float v2f __attribute__((ext_vector_type(2)));

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

// exponent of a non-negative float (0 for zero and subnormals read as -127)
__device__ __forceinline__ int exp_of(float v) { return (int)(__float_as_uint(v) >> 23) - 127; }
// exponent of the power of two that brings a column with the sum of squares m2 to a 2-norm in
// [2^13, 2^14) (its largest entry then is below 2^14 and no less than 2^-3 of that at 64 rows); a
// column whose squares vanish takes 2^77
__device__ __forceinline__ int norm_shift(float m2) { return 13 - (exp_of(m2) >> 1); }
__device__ __forceinline__ float pow2i(int e) { return __uint_as_float((uint32_t)(e + 127) << 23); }   // -126 <= e <= 127

}  // namespace deer
