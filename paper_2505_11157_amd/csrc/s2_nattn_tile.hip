// Dispatch of the bf16 matrix-core tile kernels (s2_nattn_tile_impl.h) over the staging mode.
#include "s2_nattn_tile.h"
#include "s2_nattn_kernels.h"

int s2_nattn_tile_configure() { return TileSet<kWide>::configure() || TileSet<kNarrow>::configure() || TileSet<kRagged>::configure(); }

bool s2_nattn_tile_supported(const S2DeviceTables &t, int d, int e)
{
    return d <= 64 && e <= 64 && t.band_rows_ok && !s2_debug_flag(S2_DEBUG_NO_MFMA);
}

namespace {
const bf16raw *in(const void *p) { return static_cast<const bf16raw *>(p); }
bf16raw *res(void *p) { return static_cast<bf16raw *>(p); }
}  // namespace

int s2_nattn_fwd_tile_bf16(const S2DeviceTables &t, int nbh, int d, int e, float scale, const void *q, const void *k,
                           const void *v, void *out, float *lse, hipStream_t st)
{
    if (s2_debug_flag(S2_DEBUG_FAIL_LAUNCH)) return -1;
    s2_by_band_mode<TileSet>(s2_band_mode(t.side_out, d, e, sizeof(bf16raw)), [&](auto set) { set.fwd(t, nbh, d, e, scale, in(q), in(k), in(v), res(out), lse, st); });
    return 0;
}
int s2_nattn_bwd_dq_tile_bf16(const S2DeviceTables &t, int nbh, int d, int e, float scale, const void *q, const void *k,
                              const void *v, const void *o, const float *lse, const void *go, void *dq, float *Dws,
                              hipStream_t st)
{
    if (s2_debug_flag(S2_DEBUG_FAIL_LAUNCH)) return -1;
    s2_by_band_mode<TileSet>(s2_band_mode(t.side_out, d, e, sizeof(bf16raw)), [&](auto set) {
        set.dq(t, nbh, d, e, scale, in(q), in(k), in(v), in(o), lse, in(go), res(dq), Dws, st);
    });
    return 0;
}
int s2_nattn_bwd_dkdv_tile_bf16(const S2DeviceTables &t, int nbh, int d, int e, float scale, const void *q, const void *k,
                                const void *v, const float *lse, const void *go, const float *Dws, void *dk, void *dv,
                                hipStream_t st)
{
    if (s2_debug_flag(S2_DEBUG_FAIL_LAUNCH)) return -1;
    s2_by_band_mode<TileSet>(s2_band_mode(t.side_in, d, e, sizeof(bf16raw)), [&](auto set) {
        set.dkdv(t, nbh, d, e, scale, in(q), in(k), in(v), lse, in(go), Dws, res(dk), res(dv), st);
    });
    return 0;
}
