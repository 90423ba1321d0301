// Spherical multi-head attention sub-block (Sec. 3.4 "Spherical attention blocks": pre-norm, residual) around the
// neighborhood attention kernels, float32:
//     xhat = instance norm of x per (batch, channel) over the grid points (plain moments, biased variance)
//     xn   = gamma xhat + beta + pos
//     q, k, v = Wq xn + bq, Wk xn + bk, Wv xn + bv          (1x1 convolutions; head i owns channels i d .. (i+1) d - 1,
//                                                            which is the [batch][heads][d] layout of the kernels)
//     a    = s2_nattn_fwd(q, k, v), scale 1 / sqrt(d)
//     y    = x + Wo a + bo
// and its backward.  The channel products are those of s2_channel.hip: q, k and v in one launch, their three gradients
// to xn in one, the weight and bias gradients of the three projections in one.
#include <algorithm>
#include <initializer_list>
#include <type_traits>

#include "s2_nattn_kernels.h"

namespace {

// Sum over a workgroup of THREADS, the same in every thread, in a fixed order
template <int THREADS>
__device__ __forceinline__ float block_sum(float x, float *red)
{
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) x += __shfl_xor(x, s);
    const int tid = threadIdx.x;
    if ((tid & 63) == 0) red[tid >> 6] = x;
    __syncthreads();
    float r = red[0];
#pragma unroll
    for (int i = 1; i < THREADS / 64; ++i) r += red[i];
    __syncthreads();
    return r;
}

// Instance normalisation: one workgroup per (batch, channel): mean and 1 / sqrt(var + eps) over the N grid points
// (two passes: the moments are taken about the mean), then xn = gamma xhat + beta + pos.  N is a multiple of 4 and the
// rows are 16-byte aligned: 16-byte accesses, each lane with four running sums (one per component) that are added in a
// fixed order.  A row of up to 4 KEEP THREADS points is read once and kept in registers: short ones by 256 threads (28 x 48,
// 512 rows: 1024 threads 2 us more of 52), longer ones by 1024; KEEP = 0: what is longer still, read three times.  Bound: memory (129 x 256, 4 x 128 channels: 256 threads that read three times 51 us, 30 with the row
// kept; backward 59, 45).
constexpr int kNormKeep = 9;
template <class F>
void by_row(int N, F &&f)       // f(threads, KEEP)
{
    using std::integral_constant;
    if (N <= 4 * kNormKeep * 256) f(integral_constant<int, 256>(), integral_constant<int, kNormKeep>());
    else if (N <= 4 * kNormKeep * 1024) f(integral_constant<int, 1024>(), integral_constant<int, kNormKeep>());
    else f(integral_constant<int, 1024>(), integral_constant<int, 0>());
}
__device__ __forceinline__ float sum4(float4 a) { return (a.x + a.y) + (a.z + a.w); }

// f(r, i) for the pieces i of a row of n4 that are this thread's, r = 0, 1, ... (in registers where KEEP says so)
template <int THREADS, int KEEP, class F>
__device__ __forceinline__ void pieces(int n4, F &&f)
{
    if constexpr (KEEP > 0) {
#pragma unroll
        for (int r = 0; r < KEEP; ++r) {
            const int i = threadIdx.x + r * THREADS;
            if (i < n4) f(r, i);
        }
    } else {
#pragma unroll 4
        for (int i = threadIdx.x; i < n4; i += THREADS) f(0, i);
    }
}

template <int THREADS, int KEEP>
__global__ void __launch_bounds__(THREADS)
mha_instnorm_fwd(int C, int N, float eps, const float *__restrict__ x, const float *__restrict__ gamma,
                 const float *__restrict__ beta, const float *__restrict__ pos, float *__restrict__ mean,
                 float *__restrict__ rstd, float *__restrict__ xn)
{
    __shared__ float red[THREADS / 64];
    const int bc = blockIdx.x, c = bc % C, n4 = N >> 2;
    const float4 *xr = reinterpret_cast<const float4 *>(x + size_t(bc) * N);
    float4 kept[KEEP > 0 ? KEEP : 1];
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    if (KEEP > 0) pieces<THREADS, KEEP>(n4, [&](int r, int i) { kept[r] = xr[i]; });
    auto at = [&](int r, int i) { return KEEP > 0 ? kept[r] : xr[i]; };
    pieces<THREADS, KEEP>(n4, [&](int r, int i) {
        const float4 a = at(r, i);
        s.x += a.x; s.y += a.y; s.z += a.z; s.w += a.w;
    });
    const float mu = block_sum<THREADS>(sum4(s), red) / float(N);
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    pieces<THREADS, KEEP>(n4, [&](int r, int i) {
        const float4 a = at(r, i);
        const float dx = a.x - mu, dy = a.y - mu, dz = a.z - mu, dw = a.w - mu;
        v.x = fmaf(dx, dx, v.x); v.y = fmaf(dy, dy, v.y); v.z = fmaf(dz, dz, v.z); v.w = fmaf(dw, dw, v.w);
    });
    const float rs = 1.f / sqrtf(block_sum<THREADS>(sum4(v), red) / float(N) + eps);
    if (threadIdx.x == 0) { mean[bc] = mu; rstd[bc] = rs; }
    const float ga = gamma ? gamma[c] : 1.f, be = beta ? beta[c] : 0.f;
    const float4 *pr = pos ? reinterpret_cast<const float4 *>(pos + size_t(c) * N) : nullptr;
    float4 *o = reinterpret_cast<float4 *>(xn + size_t(bc) * N);
    pieces<THREADS, KEEP>(n4, [&](int r, int i) {
        const float4 a = at(r, i), p = pr ? pr[i] : make_float4(0.f, 0.f, 0.f, 0.f);
        o[i] = make_float4(fmaf(ga, (a.x - mu) * rs, be) + p.x, fmaf(ga, (a.y - mu) * rs, be) + p.y,
                           fmaf(ga, (a.z - mu) * rs, be) + p.z, fmaf(ga, (a.w - mu) * rs, be) + p.w);
    });
}

// dx = dy + rstd (dxhat - mean(dxhat) - xhat mean(dxhat xhat)), dxhat = gamma dxn; one workgroup per (batch, channel).
// The two sums over the row, of dxn and of dxn xhat, are kept for the gradients of beta and gamma.
template <int THREADS, int KEEP>
__global__ void __launch_bounds__(THREADS)
mha_instnorm_bwd(int C, int N, const float *__restrict__ x, const float *__restrict__ gamma, const float *__restrict__ mean,
                 const float *__restrict__ rstd, const float *__restrict__ dxn, const float *__restrict__ dy,
                 float *__restrict__ dx, float *__restrict__ sums)
{
    __shared__ float red[THREADS / 64];
    const int bc = blockIdx.x, c = bc % C, n4 = N >> 2;
    const float mu = mean[bc], rs = rstd[bc], ga = gamma ? gamma[c] : 1.f;
    const float4 *xr = reinterpret_cast<const float4 *>(x + size_t(bc) * N);
    const float4 *gr = reinterpret_cast<const float4 *>(dxn + size_t(bc) * N);
    const float4 *yr = reinterpret_cast<const float4 *>(dy + size_t(bc) * N);
    float4 kg[KEEP > 0 ? KEEP : 1], ka[KEEP > 0 ? KEEP : 1];
    if (KEEP > 0) pieces<THREADS, KEEP>(n4, [&](int r, int i) { kg[r] = gr[i]; ka[r] = xr[i]; });
    float4 s1 = make_float4(0.f, 0.f, 0.f, 0.f), s2 = s1;
    pieces<THREADS, KEEP>(n4, [&](int r, int i) {
        const float4 g = KEEP > 0 ? kg[r] : gr[i], a = KEEP > 0 ? ka[r] : xr[i];
        s1.x += g.x; s1.y += g.y; s1.z += g.z; s1.w += g.w;
        s2.x = fmaf(g.x, (a.x - mu) * rs, s2.x); s2.y = fmaf(g.y, (a.y - mu) * rs, s2.y);
        s2.z = fmaf(g.z, (a.z - mu) * rs, s2.z); s2.w = fmaf(g.w, (a.w - mu) * rs, s2.w);
    });
    const float t1 = block_sum<THREADS>(sum4(s1), red), t2 = block_sum<THREADS>(sum4(s2), red);
    const float m1 = ga * t1 / float(N), m2 = ga * t2 / float(N);
    if (threadIdx.x == 0) {
        sums[bc] = t1;
        sums[gridDim.x + bc] = t2;
    }
    float4 *o = reinterpret_cast<float4 *>(dx + size_t(bc) * N);
    pieces<THREADS, KEEP>(n4, [&](int r, int i) {
        const float4 g = KEEP > 0 ? kg[r] : gr[i], a = KEEP > 0 ? ka[r] : xr[i], y = yr[i];
        o[i] = make_float4(y.x + rs * (ga * g.x - m1 - (a.x - mu) * rs * m2), y.y + rs * (ga * g.y - m1 - (a.y - mu) * rs * m2),
                           y.z + rs * (ga * g.z - m1 - (a.z - mu) * rs * m2), y.w + rs * (ga * g.w - m1 - (a.w - mu) * rs * m2));
    });
}

// dbeta[c] = sum_b sum_n dxn, dgamma[c] = sum_b sum_n dxn xhat, from the row sums of mha_instnorm_bwd
__global__ void __launch_bounds__(256)
mha_affine_grads(int batch, int C, const float *__restrict__ sums, float *__restrict__ dgamma, float *__restrict__ dbeta)
{
    const int c = blockIdx.x * 256 + threadIdx.x;
    if (c >= C) return;
    float t1 = 0.f, t2 = 0.f;
    for (int b = 0; b < batch; ++b) {
        t1 += sums[b * C + c];
        t2 += sums[(batch + b) * C + c];
    }
    if (dbeta) dbeta[c] = t1;
    if (dgamma) dgamma[c] = t2;
}

// dpos[c][n] = sum_b dxn[b][c][n]
__global__ void __launch_bounds__(256)
mha_batch_sum(int batch, size_t CN4, const float4 *__restrict__ u, float *__restrict__ out)
{
    const size_t i = size_t(blockIdx.x) * 256 + threadIdx.x;
    if (i >= CN4) return;
    float4 s = u[i];
    for (int b = 1; b < batch; ++b) {
        const float4 v = u[size_t(b) * CN4 + i];
        s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
    }
    out[4 * i] = s.x; out[4 * i + 1] = s.y; out[4 * i + 2] = s.z; out[4 * i + 3] = s.w;      // (any alignment)
}

struct Layout {      // offsets (in floats) into the workspace
    size_t mean, rstd, xn, q, k, v, a, lse, da, dq, dk, dv, dxn, D, part, sums, total;
};
Layout layout(const s2_grid_t *g, int batch, int C, int heads)
{
    const size_t N = size_t(g->nlat_in) * g->nlon_in, T = size_t(batch) * C * N;
    auto up = [](size_t x) { return (x + 63) / 64 * 64; };      // 256-byte pieces
    Layout L{};
    size_t at = 0;
    L.mean = at; at += up(size_t(batch) * C);
    L.rstd = at; at += up(size_t(batch) * C);
    L.xn = at; at += up(T);
    L.q = at; at += up(T);
    L.k = at; at += up(T);
    L.v = at; at += up(T);
    L.a = at; at += up(T);
    L.lse = at; at += up(size_t(batch) * heads * N);
    L.da = at; at += up(T);
    L.dq = at; at += up(T);
    L.dk = at; at += up(T);
    L.dv = at; at += up(T);
    L.dxn = at; at += up(T);
    L.D = at; at += up(size_t(batch) * heads * N);
    L.part = at; at += up(std::max(s2_channel_grad_floats(C, C, 1), s2_channel_grad_floats(C, C, 3)));
    L.sums = at; at += up(size_t(2) * batch * C);
    L.total = at;
    return L;
}

// the kernels read tensors and weight matrices in 16-byte pieces (NULL = an optional tensor that is absent)
bool aligned16(std::initializer_list<const void *> ptrs)
{
    for (const void *q : ptrs)
        if (reinterpret_cast<uintptr_t>(q) % 16 != 0) return false;
    return true;
}

int check(const s2_grid_t *g, int batch, int C, int heads, const void *ws, size_t ws_bytes)
{
    if (!g) return s2_fail(S2_ERR_INVALID_ARG, "grid is NULL");
    if (batch < 1 || heads < 1 || C < 1 || C % heads != 0) return s2_fail(S2_ERR_INVALID_ARG, "channels must be a positive multiple of heads");
    if (!g->on_device) return s2_fail(S2_ERR_DEVICE, "grid handle has no device tables (no HIP device at init)");
    if (g->nlat_in != g->nlat_out || g->nlon_in != g->nlon_out)
        return s2_fail(S2_ERR_UNSUPPORTED, "the attention sub-block is self-attention: input and output grid must be equal");
    if (C % 16 != 0 || (size_t(g->nlat_in) * g->nlon_in) % 16 != 0)
        return s2_fail(S2_ERR_UNSUPPORTED, "channels and the number of grid points must be multiples of 16");
    if (C / heads > 128) return s2_fail(S2_ERR_UNSUPPORTED, "head dimensions above 128 are not supported");
    if (!ws || reinterpret_cast<uintptr_t>(ws) % 256 != 0 || ws_bytes < layout(g, batch, C, heads).total * sizeof(float))
        return s2_fail(S2_ERR_WORKSPACE, "workspace missing, not 256-byte aligned or smaller than s2_mha_workspace_bytes()");
    return S2_OK;
}

}  // namespace

extern "C" size_t s2_mha_workspace_bytes(const s2_grid_t *g, int batch, int channels, int heads)
{
    if (!g || batch < 1 || channels < 1 || heads < 1) return 0;
    return layout(g, batch, channels, heads).total * sizeof(float);
}

extern "C" int s2_mha_fwd(const s2_grid_t *g, int batch, int channels, int heads, float eps, const float *x,
                          const s2_mha_params_t *p, float *y, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    int rc = check(g, batch, channels, heads, workspace, workspace_bytes);
    if (rc) return rc;
    if (!x || !p || !y || !p->Wq || !p->Wk || !p->Wv || !p->Wo) return s2_fail(S2_ERR_INVALID_ARG, "NULL tensor or weight pointer");
    if (!aligned16({x, y, p->pos, p->Wq, p->Wk, p->Wv, p->Wo}))
        return s2_fail(S2_ERR_INVALID_ARG, "x, y, pos and the weight matrices must be 16-byte aligned");
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const int C = channels, N = g->nlat_in * g->nlon_in, d = C / heads;
    float *ws = static_cast<float *>(workspace);
    const Layout L = layout(g, batch, C, heads);
    {
        S2TraceScope tr("mha_instnorm_fwd", 0.0, st);
        by_row(N, [&](auto threads, auto keep) {
            hipLaunchKernelGGL((mha_instnorm_fwd<decltype(threads)::value, decltype(keep)::value>), dim3(batch * C), dim3(threads), 0, st, C, N, eps, x, p->gamma, p->beta, p->pos,
                           ws + L.mean, ws + L.rstd, ws + L.xn);
        });
    }
    {
        S2TraceScope tr("mha_gemm qkv", 0.0, st);
        const float *xn = ws + L.xn;
        s2_channel_product(false, {C, N, C, batch, 3, 1, {p->Wq, p->Wk, p->Wv}, {xn, xn, xn}, {p->bq, p->bk, p->bv}, nullptr,
                                   {ws + L.q, ws + L.k, ws + L.v}}, st);
    }
    rc = s2_nattn_fwd(g, batch, heads, d, d, S2_F32, 1.f / sqrtf(float(d)), ws + L.q, ws + L.k, ws + L.v, ws + L.a,
                      ws + L.lse, hip_stream);
    if (rc) return rc;
    {
        S2TraceScope tr("mha_gemm out", 0.0, st);
        s2_channel_product(false, {C, N, C, batch, 1, 1, {p->Wo}, {ws + L.a}, {p->bo}, x, {y}}, st);
    }
    S2_HIP_CHECK(hipGetLastError());
    return S2_OK;
}

extern "C" int s2_mha_bwd(const s2_grid_t *g, int batch, int channels, int heads, float eps, const float *x,
                          const s2_mha_params_t *p, const float *dy, float *dx, const s2_mha_grads_t *grads,
                          void *workspace, size_t workspace_bytes, void *hip_stream)
{
    (void)eps;      // the moments saved by the forward pass are reused
    int rc = check(g, batch, channels, heads, workspace, workspace_bytes);
    if (rc) return rc;
    if (!x || !p || !dy || !dx || !grads || !p->Wq || !p->Wk || !p->Wv || !p->Wo)
        return s2_fail(S2_ERR_INVALID_ARG, "NULL tensor or weight pointer");
    if (!aligned16({x, dy, dx, p->pos, p->Wq, p->Wk, p->Wv, p->Wo}))
        return s2_fail(S2_ERR_INVALID_ARG, "x, dy, dx, pos and the weight matrices must be 16-byte aligned");
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const int C = channels, N = g->nlat_in * g->nlon_in, d = C / heads;
    float *ws = static_cast<float *>(workspace);
    const Layout L = layout(g, batch, C, heads);
    {
        // y = x + Wo a + bo
        S2TraceScope tr("mha_bwd out-projection", 0.0, st);
        if (grads->Wo || grads->bo)
            s2_channel_grad({C, N, C, batch, 1, {dy}, {ws + L.a}, {grads->Wo}, {grads->bo}}, ws + L.part, st);
        s2_channel_product(true, {C, N, C, batch, 1, 1, {p->Wo}, {dy}, {nullptr}, nullptr, {ws + L.da}}, st);
    }
    rc = s2_nattn_bwd(g, batch, heads, d, d, S2_F32, 1.f / sqrtf(float(d)), ws + L.q, ws + L.k, ws + L.v, ws + L.a,
                      ws + L.lse, ws + L.da, ws + L.dq, ws + L.dk, ws + L.dv, ws + L.D,
                      s2_nattn_bwd_workspace_bytes(g, batch, heads, d, d, S2_F32), hip_stream);
    if (rc) return rc;
    {
        S2TraceScope tr("mha_bwd qkv-projections", 0.0, st);
        const float *xn = ws + L.xn, *dq = ws + L.dq, *dk = ws + L.dk, *dv = ws + L.dv;
        if (grads->Wq || grads->Wk || grads->Wv || grads->bq || grads->bk || grads->bv)
            s2_channel_grad({C, N, C, batch, 3, {dq, dk, dv}, {xn, xn, xn}, {grads->Wq, grads->Wk, grads->Wv},
                             {grads->bq, grads->bk, grads->bv}}, ws + L.part, st);
        s2_channel_product(true, {C, N, C, batch, 1, 3, {p->Wq, p->Wk, p->Wv}, {dq, dk, dv}, {nullptr}, nullptr, {ws + L.dxn}}, st);
    }
    {
        S2TraceScope tr("mha_bwd instnorm", 0.0, st);
        if (grads->pos)
            hipLaunchKernelGGL(mha_batch_sum, dim3(unsigned((size_t(C) * N / 4 + 255) / 256)), dim3(256), 0, st, batch,
                               size_t(C) * N / 4, reinterpret_cast<const float4 *>(ws + L.dxn), grads->pos);
        by_row(N, [&](auto threads, auto keep) {
            hipLaunchKernelGGL((mha_instnorm_bwd<decltype(threads)::value, decltype(keep)::value>), dim3(batch * C), dim3(threads), 0, st, C, N, x, p->gamma, ws + L.mean, ws + L.rstd,
                           ws + L.dxn, dy, dx, ws + L.sums);
        });
        if (grads->gamma || grads->beta)
            hipLaunchKernelGGL(mha_affine_grads, dim3((C + 255) / 256), dim3(256), 0, st, batch, C, ws + L.sums, grads->gamma,
                               grads->beta);
    }
    S2_HIP_CHECK(hipGetLastError());
    return S2_OK;
}
