// Dispatch of the patch kernels (s2_nattn_patch_impl.h) over the staging mode.
#include "s2_nattn_kernels.h"
#include "s2_nattn_patch.h"

// the matrix-core kernels for any grid pair, of both element types
int s2_nattn_band_configure()
{
    return PatchSet<kWide>::configure() || PatchSet<kNarrow>::configure() || PatchSet<kRagged>::configure() || PatchSet<kPairs>::configure() || PatchSet<kHalves>::configure() ||
           PatchSet16<kWide>::configure() || PatchSet16<kNarrow>::configure() || PatchSet16<kRagged>::configure() || PatchSet16<kPairs>::configure() || PatchSet16<kHalves>::configure() ||
           SplitSet<kWide>::configure() || SplitSet<kNarrow>::configure() || SplitSet<kRagged>::configure() || SplitSet<kPairs>::configure() || SplitSet<kHalves>::configure() ||
           SplitSet16<kWide>::configure() || SplitSet16<kNarrow>::configure() || SplitSet16<kRagged>::configure() || SplitSet16<kPairs>::configure() || SplitSet16<kHalves>::configure() ||
           s2_nattn_columns_configure();
}

bool s2_nattn_patch_supported(const S2DeviceTables &t, int d, int e)
{
    return d <= 64 && e <= 64 && t.band_rows_ok && !s2_debug_flag(S2_DEBUG_NO_MFMA);
}

// f(set) with the launchers for owners of a side, of float32 or bf16 tensors
template <class F>
static void on_patches(const S2BandSide &b, int nbh, int d, int e, bool backward, bool no_halves, F &&f)
{
    int mode = s2_band_mode(b, d, e, sizeof(float));
    if (mode == kHalves && no_halves) mode = kNarrow;
    if (s2_split_list(b, nbh, d, e, sizeof(float), backward)) s2_by_band_mode<SplitSet>(mode, f);
    else s2_by_band_mode<PatchSet>(mode, f);
}
template <class F>
static void on_patches16(const S2BandSide &b, int nbh, int d, int e, bool backward, F &&f)
{
    const int mode = s2_band_mode(b, d, e, 2);
    if (s2_split_list(b, nbh, d, e, 2, backward)) s2_by_band_mode<SplitSet16>(mode, f);
    else s2_by_band_mode<PatchSet16>(mode, f);
}

static double pair_count(const double (&p)[4], int nbh) { return nbh * (p[0] + p[1] + p[2] + p[3]); }

int s2_nattn_fwd_patch(const S2DeviceTables &t, int nbh, int d, int e, float scale, const float *q, const float *k,
                       const float *v, float *out, float *lse, hipStream_t st)
{
    if (s2_debug_flag(S2_DEBUG_FAIL_LAUNCH)) return -1;
    S2TraceScope tr("nattn_fwd_patch", pair_count(t.fwd_pairs, nbh), st);
    if (d == 32 && e == 32 && t.columns.npatch > 0 && !s2_debug_flag(S2_DEBUG_FORCE_BAND)) {
        s2_nattn_fwd_columns(t, nbh, scale, q, k, v, out, lse, st);
        return 0;
    }
    on_patches(t.side_out, nbh, d, e, false, false, [&](auto set) { set.fwd(t, nbh, d, e, scale, q, k, v, out, lse, st); });
    return 0;
}

int s2_nattn_bwd_patch(const S2DeviceTables &t, int nbh, int d, int e, float scale, const float *q, const float *k,
                       const float *v, const float *o, const float *lse, const float *go, float *dq, float *dk, float *dv,
                       float *Dws, hipStream_t st)
{
    if (s2_debug_flag(S2_DEBUG_FAIL_LAUNCH)) return -1;
    {
        S2TraceScope tr("nattn_bwd_dq_patch", pair_count(t.fwd_pairs, nbh), st);
        // Classes of a finer grid meet few chunks, of which halves save less than the registers that dq spills for them cost: 119 x 238 -> 238 x
        // 476, 16 slices, d = 32, backward 614 us, by halves 670; of 160 such pairs 2 % in the mean.
        const bool no_halves = t.side_out.c_own > 1 && d == 32;
        on_patches(t.side_out, nbh, d, e, true, no_halves, [&](auto set) { set.dq(t, nbh, d, e, scale, q, k, v, o, lse, go, dq, Dws, st); });
    }
    S2TraceScope tr("nattn_bwd_dkdv_patch", pair_count(t.bwd_pairs, nbh), st);
    on_patches(t.side_in, nbh, d, e, true, false, [&](auto set) { set.dkdv(t, nbh, d, e, scale, q, k, v, lse, go, Dws, dk, dv, st); });
    return 0;
}

static const unsigned short *in16(const void *p) { return static_cast<const unsigned short *>(p); }

int s2_nattn_fwd_patch_bf16(const S2DeviceTables &t, int nbh, int d, int e, float scale, const void *q, const void *k, const void *v,
                            void *out, float *lse, hipStream_t st)
{
    if (s2_debug_flag(S2_DEBUG_FAIL_LAUNCH)) return -1;
    S2TraceScope tr("nattn_fwd_patch", pair_count(t.fwd_pairs, nbh), st);
    on_patches16(t.side_out, nbh, d, e, false, [&](auto set) {
        set.fwd(t, nbh, d, e, scale, in16(q), in16(k), in16(v), static_cast<unsigned short *>(out), lse, st);
    });
    return 0;
}
int s2_nattn_bwd_dq_patch_bf16(const S2DeviceTables &t, int nbh, int d, int e, float scale, const void *q, const void *k, const void *v,
                               const void *o, const float *lse, const void *go, void *dq, float *Dws, hipStream_t st)
{
    if (s2_debug_flag(S2_DEBUG_FAIL_LAUNCH)) return -1;
    S2TraceScope tr("nattn_bwd_dq_patch", pair_count(t.fwd_pairs, nbh), st);
    on_patches16(t.side_out, nbh, d, e, true, [&](auto set) {
        set.dq(t, nbh, d, e, scale, in16(q), in16(k), in16(v), in16(o), lse, in16(go), static_cast<unsigned short *>(dq), Dws, st);
    });
    return 0;
}
int s2_nattn_bwd_dkdv_patch_bf16(const S2DeviceTables &t, int nbh, int d, int e, float scale, const void *q, const void *k, const void *v,
                                 const float *lse, const void *go, const float *Dws, void *dk, void *dv, hipStream_t st)
{
    if (s2_debug_flag(S2_DEBUG_FAIL_LAUNCH)) return -1;
    S2TraceScope tr("nattn_bwd_dkdv_patch", pair_count(t.bwd_pairs, nbh), st);
    on_patches16(t.side_in, nbh, d, e, true, [&](auto set) {
        set.dkdv(t, nbh, d, e, scale, in16(q), in16(k), in16(v), lse, in16(go), Dws, static_cast<unsigned short *>(dk), static_cast<unsigned short *>(dv), st);
    });
    return 0;
}
