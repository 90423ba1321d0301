// Dispatch of the fp32 band-tile kernels (s2_nattn_band_impl.h) over storage type and staging mode.
#include "s2_nattn_band.h"
#include "s2_nattn_kernels.h"

namespace {

int mode_of(const S2BandSide &b, int d, int e)
{
    if (d != e || (d != 16 && d != 32 && d != 64)) return kRagged;
    return b.c_walk == 1 && b.nU % 4 == 0 ? kWide : kNarrow;
}
// f(set) with the launchers of a storage type and a staging mode
template <class T, class F>
void by_mode(int mode, F &&f)
{
    if (mode == kWide) f(BandSet<T, kWide>());
    else if (mode == kNarrow) f(BandSet<T, kNarrow>());
    else f(BandSet<T, kRagged>());
}

template <class T>
void fwd(const S2DeviceTables &t, int nbh, int d, int e, float scale, const void *q, const void *k, const void *v, void *out,
         float *lse, hipStream_t st)
{
    by_mode<T>(mode_of(t.side_out, d, e), [&](auto set) { set.fwd(t, nbh, d, e, scale, static_cast<const T *>(q), static_cast<const T *>(k), static_cast<const T *>(v),
      static_cast<T *>(out), lse, st); });
}
template <class T>
void dq(const S2DeviceTables &t, int nbh, int d, int e, float scale, const void *q, const void *k, const void *v,
        const void *o, const float *lse, const void *go, void *gq, float *Dws, hipStream_t st)
{
    by_mode<T>(mode_of(t.side_out, d, e), [&](auto set) { set.dq(t, nbh, d, e, scale, static_cast<const T *>(q), static_cast<const T *>(k), static_cast<const T *>(v),
      static_cast<const T *>(o), lse, static_cast<const T *>(go), static_cast<T *>(gq), Dws, st); });
}
template <class T>
void dkdv(const S2DeviceTables &t, int nbh, int d, int e, float scale, const void *q, const void *k, const void *v,
          const float *lse, const void *go, const float *Dws, void *gk, void *gv, hipStream_t st)
{
    by_mode<T>(mode_of(t.side_in, d, e), [&](auto set) { set.dkdv(t, nbh, d, e, scale, static_cast<const T *>(q), static_cast<const T *>(k), static_cast<const T *>(v), lse,
      static_cast<const T *>(go), Dws, static_cast<T *>(gk), static_cast<T *>(gv), st); });
}

}  // namespace

int s2_nattn_band_configure()
{
    return BandSet<float, kWide>::configure() || BandSet<float, kNarrow>::configure() || BandSet<float, kRagged>::configure() ||
           BandSet<bf16raw, kWide>::configure() || BandSet<bf16raw, kNarrow>::configure() || BandSet<bf16raw, kRagged>::configure();
}

bool s2_nattn_band_supported(const S2DeviceTables &t, int d, int e)
{
    return d <= 64 && e <= 64 && t.band_rows_ok && !s2_debug_flag(S2_DEBUG_NO_MFMA);
}

int s2_nattn_fwd_band(const S2DeviceTables &t, int nbh, int d, int e, float scale, const float *q, const float *k,
                      const float *v, float *out, float *lse, hipStream_t st)
{
    if (s2_debug_flag(S2_DEBUG_FAIL_LAUNCH)) return -1;
    fwd<float>(t, nbh, d, e, scale, q, k, v, out, lse, st);
    return 0;
}

int s2_nattn_bwd_band(const S2DeviceTables &t, int nbh, int d, int e, float scale, const float *q, const float *k,
                      const float *v, const float *o, const float *lse, const float *go, float *gq, float *gk, float *gv,
                      float *Dws, hipStream_t st)
{
    if (s2_debug_flag(S2_DEBUG_FAIL_LAUNCH)) return -1;
    dq<float>(t, nbh, d, e, scale, q, k, v, o, lse, go, gq, Dws, st);
    dkdv<float>(t, nbh, d, e, scale, q, k, v, lse, go, Dws, gk, gv, st);
    return 0;
}

// bf16 tensors on the same kernels (float32 arithmetic on the fp32 matrix cores, bf16 loads and stores)
int s2_nattn_fwd_band_bf16(const S2DeviceTables &t, int nbh, int d, int e, float scale, const void *q, const void *k,
                           const void *v, void *out, float *lse, hipStream_t st)
{
    if (s2_debug_flag(S2_DEBUG_FAIL_LAUNCH)) return -1;
    fwd<bf16raw>(t, nbh, d, e, scale, q, k, v, out, lse, st);
    return 0;
}
int s2_nattn_bwd_dq_band_bf16(const S2DeviceTables &t, int nbh, int d, int e, float scale, const void *q, const void *k,
                              const void *v, const void *o, const float *lse, const void *go, void *gq, float *Dws,
                              hipStream_t st)
{
    if (s2_debug_flag(S2_DEBUG_FAIL_LAUNCH)) return -1;
    dq<bf16raw>(t, nbh, d, e, scale, q, k, v, o, lse, go, gq, Dws, st);
    return 0;
}
int s2_nattn_bwd_dkdv_band_bf16(const S2DeviceTables &t, int nbh, int d, int e, float scale, const void *q, const void *k,
                                const void *v, const float *lse, const void *go, const float *Dws, void *gk, void *gv,
                                hipStream_t st)
{
    if (s2_debug_flag(S2_DEBUG_FAIL_LAUNCH)) return -1;
    dkdv<bf16raw>(t, nbh, d, e, scale, q, k, v, lse, go, Dws, gk, gv, st);
    return 0;
}
