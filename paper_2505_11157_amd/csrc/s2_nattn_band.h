// Launchers of the fp32 band-tile kernels by storage type and staging mode (s2_nattn_band_impl.h; one translation unit
// each, so that they compile in parallel).
#pragma once
#include "s2_internal.h"

// Storage type of the tensors: float, or bf16 bits (arithmetic, staged tiles, logsumexp and D stay float32).
typedef unsigned short bf16raw;

enum { kWide, kNarrow, kRagged };

template <class T, int MODE>
struct BandSet {
    static int configure();
    static void fwd(const S2DeviceTables &t, int nbh, int d, int e, float scale, const T *q, const T *k, const T *v, T *out,
                    float *lse, hipStream_t st);
    static void dq(const S2DeviceTables &t, int nbh, int d, int e, float scale, const T *q, const T *k, const T *v, const T *o,
                   const float *lse, const T *go, T *dq, float *Dws, hipStream_t st);
    static void dkdv(const S2DeviceTables &t, int nbh, int d, int e, float scale, const T *q, const T *k, const T *v,
                     const float *lse, const T *go, const float *Dws, T *dk, T *dv, hipStream_t st);
};
