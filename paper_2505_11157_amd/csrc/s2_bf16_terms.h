// float32 values as three bf16 terms, for float32 products on the bf16 matrix cores (device side).
//
// x = x0 + x1 + x2, 8 bits each, every term the rounded rest of those before: together they hold x exactly down to 2^-110, and within
// 2^-134 below that, where the last term ends at bf16's smallest number, 2^-133 (the matrix cores take subnormal terms as they are).
// Attention on unit-variance tensors, rms error of the result: v or dout times 2^-110 1.1e-7 as ever, 2^-114 6e-7, 2^-118 9e-6,
// 2^-126 2e-3.  Cut from 2^16 times the value, all normal numbers would be held; the multiplication takes 1.1 to 1.4 % of every training
// step (129 x 256, 32 slices, d = 32 1.629 -> 1.652 ms, d = 64 3.261 -> 3.304) and brings the overflow of products that much closer: not done.
// A product takes the six of nine term products that are not below 2^-26 of it.  Six bf16 instructions take 0.37 times the cycles of
// the fp32 ones.
// A value of (1 - 2^-9) 2^128 or more rounds to an infinite first term; what is done about non-finite results is the caller's.
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
// The same with the rests as two-element dot products, x - (t_a, t_b) . (1, 0): exact too, subnormal numbers included, and one
// instruction where widening the term and subtracting it are two.  A value that is not finite spoils its neighbor's rest here.
// Faster in the neighborhood kernels' loops over key tiles (forward 129 x 256, 32 slices: float32 d = 16 295 -> 287, d = 32 446 -> 436,
// bf16 d = 16 200 -> 190, d = 32 243 -> 236 us), not where float32 tensors are staged (no change) nor in the channel products
// (gradients behind 129 x 256, 4 x 128 channels: 91 -> 96 us).
__device__ __forceinline__ unsigned held(unsigned x)
{
    asm("" : "+s"(x));       // in a scalar register: as an immediate operand the pair means another one
    return x;
}
__device__ __forceinline__ unsigned cut_off_dot(float &a, float &b)
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    const bf16x2 t = __builtin_convertvector(f32x2{a, b}, bf16x2);
    unsigned u = __builtin_bit_cast(unsigned, t);
    asm("" : "+v"(u));
    a = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, u), __builtin_bit_cast(bf16x2, held(0x0000bf80u)), a, false);
    b = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, u), __builtin_bit_cast(bf16x2, held(0xbf800000u)), b, false);
    return u;
}
template <bool DOT = false>
__device__ __forceinline__ void cut(const float (&x)[8], bf16x8 (&b)[kTerms])
{
    u32x4 u[kTerms];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float lo = x[2 * i], hi = x[2 * i + 1];
#pragma unroll
        for (int k = 0; k < kTerms; ++k) u[k][i] = DOT ? cut_off_dot(lo, hi) : cut_off(lo, hi);
    }
#pragma unroll
    for (int k = 0; k < kTerms; ++k) b[k] = __builtin_bit_cast(bf16x8, u[k]);
}

}  // namespace s2terms
