// Launchers of the neighborhood-attention kernels (internal).
#pragma once
#include "s2_internal.h"

// Shape-agnostic float32 path: 1 <= d, e <= 128.
int s2_nattn_fwd_generic(const S2DeviceTables &t, int nbh, int d, int e, float scale, const float *q,
                         const float *k, const float *v, float *out, float *lse, hipStream_t st);
int s2_nattn_bwd_generic(const S2DeviceTables &t, int nbh, int d, int e, float scale, const float *q,
                         const float *k, const float *v, const float *o, const float *lse, const float *go,
                         float *dq, float *dk, float *dv, float *Dws, hipStream_t st);

// dk, dv of an input latitude of weight zero are zero: x is [rows][nlat_in][nlon_in], rows = slices * channels,
// float32 or bf16 elements.
void s2_nattn_zero_latitude(const S2DeviceTables &t, int lat, int rows, void *x, bool bf16, hipStream_t st);

// Shape-agnostic path on bf16 tensors (float32 arithmetic, float32 lse and D).
int s2_nattn_fwd_generic_bf16(const S2DeviceTables &t, int nbh, int d, int e, float scale, const void *q, const void *k,
                              const void *v, void *out, float *lse, hipStream_t st);
int s2_nattn_bwd_dq_generic_bf16(const S2DeviceTables &t, int nbh, int d, int e, float scale, const void *q,
                                 const void *k, const void *v, const void *o, const float *lse, const void *go, void *dq,
                                 float *Dws, hipStream_t st);
int s2_nattn_bwd_dkdv_generic_bf16(const S2DeviceTables &t, int nbh, int d, int e, float scale, const void *q,
                                   const void *k, const void *v, const float *lse, const void *go, const float *Dws,
                                   void *dk, void *dv, hipStream_t st);

// Split vector float32 forward for d = e = 32, nlon_in / nlon_out in {1, 2} or upsampling, longitudes a multiple of 4.
bool s2_nattn_fwd_tiled_supported(const S2DeviceTables &t, int d, int e);
int s2_nattn_fwd_tiled(const S2DeviceTables &t, int nbh, int d, int e, float scale, const float *q, const float *k,
                       const float *v, float *out, float *lse, hipStream_t st);

// Split vector float32 backward for d = e = 32, the same shapes.
bool s2_nattn_bwd_tiled_supported(const S2DeviceTables &t, int d, int e);
int s2_nattn_bwd_tiled(const S2DeviceTables &t, int nbh, int d, int e, float scale, const float *q, const float *k,
                       const float *v, const float *o, const float *lse, const float *go, float *dq, float *dk,
                       float *dv, float *Dws, hipStream_t st);

// Streaming kernels for the light latitudes (last class) on equal grids: each input latitude is staged in LDS once
// per workgroup and shared by the wavefronts that walk down consecutive output latitudes.
bool s2_nattn_stream_supported(const S2DeviceTables &t, int d, int e);
int s2_nattn_fwd_stream(const S2DeviceTables &t, int nbh, float qscale, const float *q, const float *k,
                        const float *v, float *out, float *lse, hipStream_t st);
bool s2_nattn_stream_dq_supported(const S2DeviceTables &t, int d, int e);
bool s2_nattn_stream_dkdv_supported(const S2DeviceTables &t, int d, int e);
int s2_nattn_bwd_dq_stream(const S2DeviceTables &t, int nbh, float scale, const float *q, const float *k,
                           const float *v, const float *o, const float *lse, const float *go, float *dq, float *Dws,
                           hipStream_t st);
int s2_nattn_bwd_dkdv_stream(const S2DeviceTables &t, int nbh, float scale, const float *q, const float *k,
                             const float *v, const float *lse, const float *go, const float *Dws, float *dk, float *dv,
                             hipStream_t st);

// float32 tensors on the bf16 matrix cores (three bf16 terms per value, s2_nattn_patch_impl.h), any grid pair, d and e up to 64.
bool s2_nattn_patch_supported(const S2DeviceTables &t, int d, int e);
int s2_nattn_fwd_patch(const S2DeviceTables &t, int nbh, int d, int e, float scale, const float *q, const float *k,
                       const float *v, float *out, float *lse, hipStream_t st);
int s2_nattn_bwd_patch(const S2DeviceTables &t, int nbh, int d, int e, float scale, const float *q, const float *k,
                       const float *v, const float *o, const float *lse, const float *go, float *dq, float *dk, float *dv,
                       float *Dws, hipStream_t st);

// The same of bf16 tensors.
int s2_nattn_fwd_patch_bf16(const S2DeviceTables &t, int nbh, int d, int e, float scale, const void *q, const void *k,
                           const void *v, void *out, float *lse, hipStream_t st);
int s2_nattn_bwd_dq_patch_bf16(const S2DeviceTables &t, int nbh, int d, int e, float scale, const void *q, const void *k,
                              const void *v, const void *o, const float *lse, const void *go, void *dq, float *Dws,
                              hipStream_t st);
int s2_nattn_bwd_dkdv_patch_bf16(const S2DeviceTables &t, int nbh, int d, int e, float scale, const void *q, const void *k,
                                const void *v, const float *lse, const void *go, const float *Dws, void *dk, void *dv,
                                hipStream_t st);

// Backward with the scratch for D_i given as a device pointer (checks and dispatch behind both C entry points).
int s2_nattn_bwd_run(const s2_grid_t *g, int batch, int heads, int d_qk, int d_v, int dtype, float scale,
                     const void *q, const void *k, const void *v, const void *out, const float *lse, const void *dout,
                     void *dq, void *dk, void *dv, float *Dws, hipStream_t st);

// Per-device set-up of the static scratch array behind s2_nattn_bwd_static (the device must be current).
int s2_static_scratch_setup(int device);
