// Dispatch of the fp32 band-tile kernels (s2_nattn_band_impl.h) over the staging mode.
#include "s2_nattn_band.h"
#include "s2_nattn_kernels.h"

namespace {

int mode_of(const S2BandSide &b, int d, int e)
{
    if (d != e || (d != 16 && d != 32 && d != 64)) return kRagged;
    return b.c_walk == 1 && b.nU % 4 == 0 ? kWide : kNarrow;
}
// f(set) with the launchers of a staging mode
template <class F>
void by_mode(int mode, F &&f)
{
    if (mode == kWide) f(BandSet<kWide>());
    else if (mode == kNarrow) f(BandSet<kNarrow>());
    else f(BandSet<kRagged>());
}

}  // namespace

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
    by_mode(mode_of(t.side_out, d, e), [&](auto set) { set.fwd(t, nbh, d, e, scale, q, k, v, out, lse, st); });
    return 0;
}

int s2_nattn_bwd_band(const S2DeviceTables &t, int nbh, int d, int e, float scale, const float *q, const float *k,
                      const float *v, const float *o, const float *lse, const float *go, float *dq, float *dk, float *dv,
                      float *Dws, hipStream_t st)
{
    if (s2_debug_flag(S2_DEBUG_FAIL_LAUNCH)) return -1;
    by_mode(mode_of(t.side_out, d, e), [&](auto set) { set.dq(t, nbh, d, e, scale, q, k, v, o, lse, go, dq, Dws, st); });
    by_mode(mode_of(t.side_in, d, e), [&](auto set) { set.dkdv(t, nbh, d, e, scale, q, k, v, lse, go, Dws, dk, dv, st); });
    return 0;
}
