// Launchers of the bf16 matrix-core tile kernels by staging mode (s2_nattn_tile_impl.h; one translation unit each, so that they
// compile in parallel).
#pragma once
#include "s2_internal.h"
#include "s2_nattn_band.h"

typedef unsigned short bf16raw;        // storage of a bf16 tensor

template <int MODE>
struct TileSet {
    static int configure();
    static void fwd(const S2DeviceTables &t, int nbh, int d, int e, float scale, const bf16raw *q, const bf16raw *k, const bf16raw *v, bf16raw *out,
                    float *lse, hipStream_t st);
    static void dq(const S2DeviceTables &t, int nbh, int d, int e, float scale, const bf16raw *q, const bf16raw *k, const bf16raw *v, const bf16raw *o,
                   const float *lse, const bf16raw *go, bf16raw *dq, float *Dws, hipStream_t st);
    static void dkdv(const S2DeviceTables &t, int nbh, int d, int e, float scale, const bf16raw *q, const bf16raw *k, const bf16raw *v,
                     const float *lse, const bf16raw *go, const float *Dws, bf16raw *dk, bf16raw *dv, hipStream_t st);
};
