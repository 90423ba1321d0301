// The forward of float32 tensors on upsampling grids with d = e = 32 by columns: rolled in longitude, its results are the same bit for bit.
#include "s2_nattn_patch_impl.h"

using ColumnGeo = Geo<float, 32, kS2ColumnStage, 4>;

int s2_nattn_columns_configure()
{
    return raise_lds(reinterpret_cast<const void *>(nattn_fwd_patch<ColumnGeo, kColumns>), sizeof(Shared<ColumnGeo, kColumns>));
}
void s2_nattn_fwd_columns(const S2DeviceTables &t, int nbh, float scale, const float *q, const float *k, const float *v, float *out, float *lse,
                          hipStream_t st)
{
    S2BandSide b = t.side_out;
    b.patches = t.columns;
    const PatchLaunch l = patch_launch(t, b, nbh, ColumnGeo::D, ColumnGeo::D, scale, nullptr);
    hipLaunchKernelGGL((nattn_fwd_patch<ColumnGeo, kColumns>), l.grid, dim3(ColumnGeo::NT), sizeof(Shared<ColumnGeo, kColumns>), st, l.a, q, k, v, out, lse);
}
