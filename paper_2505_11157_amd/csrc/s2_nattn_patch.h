// Launchers of the float32 patch kernels by staging mode (s2_nattn_patch_impl.h; one translation unit each, so that they
// compile in parallel).
#pragma once
#include "s2_internal.h"
#include "s2_nattn_band.h"

template <int MODE>
struct PatchSet {
    static int configure();
    static void fwd(const S2DeviceTables &t, int nbh, int d, int e, float scale, const float *q, const float *k, const float *v, float *out,
                    float *lse, hipStream_t st);
    static void dq(const S2DeviceTables &t, int nbh, int d, int e, float scale, const float *q, const float *k, const float *v, const float *o,
                   const float *lse, const float *go, float *dq, float *Dws, hipStream_t st);
    static void dkdv(const S2DeviceTables &t, int nbh, int d, int e, float scale, const float *q, const float *k, const float *v,
                     const float *lse, const float *go, const float *Dws, float *dk, float *dv, hipStream_t st);
};
