// float32 values as three bf16 terms, for float32 products on the bf16 matrix cores (device side).
//
// x = x0 + x1 + x2, 8 bits each, every term the rounded rest of those before: together they hold x exactly.  A product takes the six
// of nine term products that are not below 2^-26 of it.  Six bf16 instructions take 0.37 times the cycles of the fp32 ones.
// A value near the largest float32 rounds to an infinite first term; what is done about non-finite results is the caller's.
#pragma once
#include <hip/hip_runtime.h>

namespace s2terms {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr int kTerms = 3;            // bf16 terms of a float32 value

// two float32 values as bf16 (low half: a), rounded to nearest even, and what that leaves of them
__device__ __forceinline__ unsigned cut_off(float &a, float &b)
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    unsigned u = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{a, b}, bf16x2));
    asm("" : "+v"(u));       // else the compiler converts each of the two once more for what follows
    a -= __builtin_bit_cast(float, u << 16);
    b -= __builtin_bit_cast(float, u & 0xffff0000u);
    return u;
}
__device__ __forceinline__ void cut(const float (&x)[8], bf16x8 (&b)[kTerms])
{
    u32x4 u[kTerms];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float lo = x[2 * i], hi = x[2 * i + 1];
#pragma unroll
        for (int k = 0; k < kTerms; ++k) u[k][i] = cut_off(lo, hi);
    }
#pragma unroll
    for (int k = 0; k < kTerms; ++k) b[k] = __builtin_bit_cast(bf16x8, u[k]);
}

}  // namespace s2terms
