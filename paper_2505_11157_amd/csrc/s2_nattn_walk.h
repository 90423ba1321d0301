// What the patch kernels of the neighborhood attention (s2_nattn_patch_impl.h) and the evaluation of single points
// (s2_nattn_exact.h) share.
//
// Both directions and all grid ratios are one problem (S2BandSide): owners (the points a wavefront accumulates for) and
// walked points lie on grids of the same longitude count nU.  Equal grids are that already; where one grid has r times
// the longitudes of the other, its latitude is cut into r interleaved classes s (longitudes r u + s, u < nU), each of
// them a row of its own.  On walked row r the neighbors of owner u are the columns u + lo .. u + lo + cnt - 1 around the
// circle of nU.
#pragma once
#include <hip/hip_runtime.h>

#include "s2_internal.h"
#include "s2_nattn_band.h"

namespace s2walk {

constexpr int kMaxRows = kS2PatchRows;

typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kMinRef = -1e30f;    // start value of the reference maximum: finite, so that x - m needs no guard (exp2(-inf) = 0)

__device__ __forceinline__ float group_max(float x)     // over the four lanes (g = 0..3) of a point
{
    x = fmaxf(x, __shfl_xor(x, 16));
    return fmaxf(x, __shfl_xor(x, 32));
}
__device__ __forceinline__ float group_sum(float x)
{
    x += __shfl_xor(x, 16);
    return x + __shfl_xor(x, 32);
}
// Matrix results that a branch may lead to a reader of: the compiler pads the wait states of an instruction on one side of
// a branch only.  Ten wait states here, after the last instruction of the tile.
template <int N>
__device__ __forceinline__ void settle(f32x4 (&a)[N])
{
#pragma unroll
    for (int i = 0; i + 1 < N; ++i) asm volatile("" : "+v"(a[i]));
    asm volatile("s_nop 9" : "+v"(a[N - 1]));
}

__device__ __forceinline__ int imin(int a, int b) { return a < b ? a : b; }

// x mod n for 0 <= x < 2^22: the float32 quotient is off by at most one
__device__ __forceinline__ int wrap_col(int x, int n, float inv_n)
{
    const int r = x - int(float(x) * inv_n) * n;
    return r < 0 ? r + n : r >= n ? r - n : r;
}

// Kernel arguments
struct BandArgs {
    S2BandSide b;
    const float *omega_rel;
    float ln_omega_ref, omega_ref, scale;
    int nbh, d, e;
    // patch kernels (S2BandSide::Patches)
    const int4 *seg, *row_rec;
    const int2 *patch;
    int npatch;
};

template <class V>
__device__ __forceinline__ V load_at(const void *row, unsigned off)
{
    return *reinterpret_cast<const V *>(static_cast<const char *>(row) + off);
}

}  // namespace s2walk
