// C entry points of the neighborhood attention: argument checks and dispatch.
#include <algorithm>

#include "s2_nattn_kernels.h"

namespace {

int check_common(const s2_grid_t *g, int batch, int heads, int d_qk, int d_v, int dtype)
{
    if (!g) return s2_fail(S2_ERR_INVALID_ARG, "grid is NULL");
    if (batch < 1 || heads < 1 || d_qk < 1 || d_v < 1) return s2_fail(S2_ERR_INVALID_ARG, "batch, heads, d must be >= 1");
    if (dtype != S2_F32 && dtype != S2_BF16) return s2_fail(S2_ERR_UNSUPPORTED, "unknown dtype");
    if (d_qk > 128 || d_v > 128) return s2_fail(S2_ERR_UNSUPPORTED, "head dimensions above 128 are not supported");
    if (long(batch) * heads > (1l << 20)) return s2_fail(S2_ERR_INVALID_ARG, "batch*heads too large");
    if (!g->on_device) return s2_fail(S2_ERR_DEVICE, "grid handle has no device tables (no HIP device at init)");
    return S2_OK;
}

// Slices that the launches of one round take: a launch of 2^32 threads or more leaves the rest out without an error.  No kernel
// has more than 512 threads for 64 longitudes (of one class) of a latitude and slice, or 256 for a workgroup's patches.
int slices_at_once(const s2_grid_t *g)
{
    const long lat = std::max(g->nlat_in, g->nlat_out), lon = std::min(g->nlon_in, g->nlon_out), classes = std::max(g->pscale, g->upscale);
    const long threads = std::max(512 * lat * classes * ((lon + 63) / 64), 256l * std::max({g->dt.side_out.patches.npatch, g->dt.side_in.patches.npatch, g->dt.columns.npatch}));
    return int(std::clamp(((1l << 32) - 1) / threads, 1l, 1l << 20));
}
size_t points_out(const s2_grid_t *g) { return size_t(g->nlat_out) * g->nlon_out; }
size_t points_in(const s2_grid_t *g) { return size_t(g->nlat_in) * g->nlon_in; }
template <class T>
T *skip(T *p, size_t bytes) { return reinterpret_cast<T *>(reinterpret_cast<uintptr_t>(p) + bytes); }

// the tuned kernels move 16-byte pieces (vector loads and stores, LDS-direct copies)
bool misaligned(const void *p) { return reinterpret_cast<uintptr_t>(p) % 16 != 0; }

}  // namespace

extern "C" size_t s2_nattn_bwd_workspace_bytes(const s2_grid_t *g, int batch, int heads, int d_qk, int d_v, int dtype)
{
    (void)d_qk; (void)d_v; (void)dtype;
    if (!g || batch < 1 || heads < 1) return 0;
    // D_i = dout_i . out_i, one float per output point and (batch, head)
    return size_t(batch) * heads * g->nlat_out * g->nlon_out * sizeof(float);
}

// The patch kernels take everything up to 64 channels whose walked rows fit their tables.
static bool use_patch(const S2DeviceTables &t, int d, int e)
{
    return s2_nattn_patch_supported(t, d, e) && !s2_debug_flag(S2_DEBUG_NO_BAND);
}

extern "C" int s2_nattn_fwd(const s2_grid_t *g, int batch, int heads, int d_qk, int d_v, int dtype, float scale,
                            const void *q, const void *k, const void *v, void *out, float *lse, void *hip_stream)
{
    int rc = check_common(g, batch, heads, d_qk, d_v, dtype);
    if (rc) return rc;
    if (!q || !k || !v || !out || !lse) return s2_fail(S2_ERR_INVALID_ARG, "NULL tensor pointer");
    if (misaligned(q) || misaligned(k) || misaligned(v) || misaligned(out) || misaligned(lse))
        return s2_fail(S2_ERR_INVALID_ARG, "tensor pointers must be 16-byte aligned");
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const int nbh = batch * heads, most = slices_at_once(g);
    const size_t element = dtype == S2_BF16 ? 2 : 4, so = points_out(g) * element, si = points_in(g) * element;
    for (int b = 0; b < nbh; b += most) {
        const int n = std::min(most, nbh - b);
        const void *qb = skip(q, b * d_qk * so), *kb = skip(k, b * d_qk * si), *vb = skip(v, b * d_v * si);
        void *ob = skip(out, b * d_v * so);
        float *lb = lse + b * points_out(g);
        int failed;
        if (dtype == S2_BF16) {
            auto *fwd16 = use_patch(g->dt, d_qk, d_v) ? s2_nattn_fwd_patch_bf16 : s2_nattn_fwd_generic_bf16;
            failed = fwd16(g->dt, n, d_qk, d_v, scale, qb, kb, vb, ob, lb, st);
        } else {
            auto *fwd = use_patch(g->dt, d_qk, d_v)                      ? s2_nattn_fwd_patch
                        : s2_nattn_fwd_tiled_supported(g->dt, d_qk, d_v) ? s2_nattn_fwd_tiled
                                                                         : s2_nattn_fwd_generic;
            failed = fwd(g->dt, n, d_qk, d_v, scale, static_cast<const float *>(qb), static_cast<const float *>(kb),
                         static_cast<const float *>(vb), static_cast<float *>(ob), lb, st);
        }
        if (failed) return s2_fail(S2_ERR_DEVICE, "forward launch configuration failed");
    }
    S2_HIP_CHECK(hipGetLastError());
    return S2_OK;
}

// Argument checks and dispatch shared by s2_nattn_bwd and s2_nattn_bwd_static; Dws: device scratch for D_i.
int s2_nattn_bwd_run(const s2_grid_t *g, int batch, int heads, int d_qk, int d_v, int dtype, float scale,
                     const void *q, const void *k, const void *v, const void *out, const float *lse, const void *dout,
                     void *dq, void *dk, void *dv, float *Dws, hipStream_t st)
{
    int rc = check_common(g, batch, heads, d_qk, d_v, dtype);
    if (rc) return rc;
    if (!q || !k || !v || !out || !lse || !dout || !dq || !dk || !dv)
        return s2_fail(S2_ERR_INVALID_ARG, "NULL tensor pointer");
    if (misaligned(q) || misaligned(k) || misaligned(v) || misaligned(out) || misaligned(lse) || misaligned(dout) ||
        misaligned(dq) || misaligned(dk) || misaligned(dv))
        return s2_fail(S2_ERR_INVALID_ARG, "tensor pointers must be 16-byte aligned");
    const int nbh = batch * heads, most = slices_at_once(g);
    const size_t element = dtype == S2_BF16 ? 2 : 4, so = points_out(g) * element, si = points_in(g) * element;
    for (int b = 0; b < nbh; b += most) {
        const int n = std::min(most, nbh - b);
        const void *qb = skip(q, b * d_qk * so), *kb = skip(k, b * d_qk * si), *vb = skip(v, b * d_v * si), *ob = skip(out, b * d_v * so),
                   *gb = skip(dout, b * d_v * so);
        void *dqb = skip(dq, b * d_qk * so), *dkb = skip(dk, b * d_qk * si), *dvb = skip(dv, b * d_v * si);
        const float *lb = lse + b * points_out(g);
        float *Db = Dws + b * points_out(g);
        int failed;
        if (dtype == S2_BF16) {
            const bool patch = use_patch(g->dt, d_qk, d_v);
            auto *dq16 = patch ? s2_nattn_bwd_dq_patch_bf16 : s2_nattn_bwd_dq_generic_bf16;
            auto *kv16 = patch ? s2_nattn_bwd_dkdv_patch_bf16 : s2_nattn_bwd_dkdv_generic_bf16;
            failed = dq16(g->dt, n, d_qk, d_v, scale, qb, kb, vb, ob, lb, gb, dqb, Db, st) ||
                     kv16(g->dt, n, d_qk, d_v, scale, qb, kb, vb, lb, gb, Db, dkb, dvb, st);
        } else {
            auto *bwd = use_patch(g->dt, d_qk, d_v)                      ? s2_nattn_bwd_patch
                        : s2_nattn_bwd_tiled_supported(g->dt, d_qk, d_v) ? s2_nattn_bwd_tiled
                                                                         : s2_nattn_bwd_generic;
            failed = bwd(g->dt, n, d_qk, d_v, scale, static_cast<const float *>(qb), static_cast<const float *>(kb),
                         static_cast<const float *>(vb), static_cast<const float *>(ob), lb, static_cast<const float *>(gb),
                         static_cast<float *>(dqb), static_cast<float *>(dkb), static_cast<float *>(dvb), Db, st);
        }
        if (failed) return s2_fail(S2_ERR_DEVICE, "backward launch configuration failed");
    }
    // input latitudes of weight zero (the pole row of the grid of App. A.1): dk = dv = 0 exactly
    for (int lat : g->zero_lat) {
        s2_nattn_zero_latitude(g->dt, lat, batch * heads * d_qk, dk, dtype == S2_BF16, st);
        s2_nattn_zero_latitude(g->dt, lat, batch * heads * d_v, dv, dtype == S2_BF16, st);
    }
    S2_HIP_CHECK(hipGetLastError());
    return S2_OK;
}

extern "C" int s2_nattn_bwd(const s2_grid_t *g, int batch, int heads, int d_qk, int d_v, int dtype, float scale,
                            const void *q, const void *k, const void *v, const void *out, const float *lse,
                            const void *dout, void *dq, void *dk, void *dv, void *workspace, size_t workspace_bytes,
                            void *hip_stream)
{
    if (!g) return s2_fail(S2_ERR_INVALID_ARG, "grid is NULL");
    if (!workspace || workspace_bytes < s2_nattn_bwd_workspace_bytes(g, batch, heads, d_qk, d_v, dtype))
        return s2_fail(S2_ERR_WORKSPACE, "workspace missing or smaller than s2_nattn_bwd_workspace_bytes()");
    if (misaligned(workspace)) return s2_fail(S2_ERR_WORKSPACE, "workspace must be 16-byte aligned");
    return s2_nattn_bwd_run(g, batch, heads, d_qk, d_v, dtype, scale, q, k, v, out, lse, dout, dq, dk, dv,
                            static_cast<float *>(workspace), static_cast<hipStream_t>(hip_stream));
}
