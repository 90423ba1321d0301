// Dispatch of the fp32 band-tile kernels (s2_nattn_band_impl.h) over the staging mode.
#include "s2_nattn_band.h"
#include "s2_nattn_kernels.h"

unsigned s2_compute_units()
{
    static const unsigned ncu = [] {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1)
            n = 256;
        return unsigned(n);
    }();
    return ncu;
}

// the band-tile kernels of both element types
int s2_nattn_band_configure()
{
    return BandSet<kWide>::configure() || BandSet<kNarrow>::configure() || BandSet<kRagged>::configure() || s2_nattn_tile_configure();
}

bool s2_nattn_band_supported(const S2DeviceTables &t, int d, int e)
{
    return d <= 64 && e <= 64 && t.band_rows_ok && !s2_debug_flag(S2_DEBUG_NO_MFMA);
}

int s2_nattn_fwd_band(const S2DeviceTables &t, int nbh, int d, int e, float scale, const float *q, const float *k,
                      const float *v, float *out, float *lse, hipStream_t st)
{
    if (s2_debug_flag(S2_DEBUG_FAIL_LAUNCH)) return -1;
    s2_by_band_mode<BandSet>(s2_band_mode(t.side_out, d, e, sizeof(float)), [&](auto set) { set.fwd(t, nbh, d, e, scale, q, k, v, out, lse, st); });
    return 0;
}

int s2_nattn_bwd_band(const S2DeviceTables &t, int nbh, int d, int e, float scale, const float *q, const float *k,
                      const float *v, const float *o, const float *lse, const float *go, float *dq, float *dk, float *dv,
                      float *Dws, hipStream_t st)
{
    if (s2_debug_flag(S2_DEBUG_FAIL_LAUNCH)) return -1;
    s2_by_band_mode<BandSet>(s2_band_mode(t.side_out, d, e, sizeof(float)), [&](auto set) { set.dq(t, nbh, d, e, scale, q, k, v, o, lse, go, dq, Dws, st); });
    s2_by_band_mode<BandSet>(s2_band_mode(t.side_in, d, e, sizeof(float)), [&](auto set) { set.dkdv(t, nbh, d, e, scale, q, k, v, lse, go, Dws, dk, dv, st); });
    return 0;
}
