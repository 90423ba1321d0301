// Launchers of the patch kernels by element type and staging mode (s2_nattn_patch_impl.h; one translation unit each, so that they
// compile in parallel).
#pragma once
#include "s2_internal.h"
#include "s2_nattn_band.h"

template <class T, int MODE, bool SPLIT = false>
struct PatchKernels {
    static int configure();
    static void fwd(const S2DeviceTables &t, int nbh, int d, int e, float scale, const T *q, const T *k, const T *v, T *out, float *lse, hipStream_t st);
    static void dq(const S2DeviceTables &t, int nbh, int d, int e, float scale, const T *q, const T *k, const T *v, const T *o, const float *lse,
                   const T *go, T *dq, float *Dws, hipStream_t st);
    static void dkdv(const S2DeviceTables &t, int nbh, int d, int e, float scale, const T *q, const T *k, const T *v, const float *lse, const T *go,
                     const float *Dws, T *dk, T *dv, hipStream_t st);
};
template <int MODE>
using PatchSet = PatchKernels<float, MODE>;
template <int MODE>
using PatchSet16 = PatchKernels<unsigned short, MODE>;      // bf16 tensors

// The same on the lists where wavefronts share patches (S2BandSide::Patches::split)
template <int MODE>
using SplitSet = PatchKernels<float, MODE, true>;
template <int MODE>
using SplitSet16 = PatchKernels<unsigned short, MODE, true>;

// The forward by columns (S2ColumnRow), float32 d = e = 32
int s2_nattn_columns_configure();
void s2_nattn_fwd_columns(const S2DeviceTables &t, int nbh, float scale, const float *q, const float *k, const float *v, float *out, float *lse,
                          hipStream_t st);
