// One point of the neighborhood attention over its true neighbors only (device side).
//
// The matrix-core tiles (s2_nattn_patch_impl.h) give a staged column outside an owner's disk the
// weight zero, and zero times a NaN or an infinity is a NaN: a non-finite value next to a disk would spoil the point.  A
// mask on the staged values cannot tell owners apart that share a tile.  So a wavefront looks at its finished sums, and
// owners with a sum that is not finite are evaluated again here, where no other point is touched.  With finite inputs
// that costs one multiply-add per sum; the evaluation itself is slow (one owner at a time, lanes over its neighbors) and
// only runs where the inputs hold non-finite values or the results overflow.
#pragma once
#include "s2_nattn_walk.h"

namespace s2walk {

// owners (bit n) of a 16-owner tile with a sum that is not finite; own: the lane's owner is a point of the grid
template <int N>
__device__ __forceinline__ unsigned not_finite(const f32x4 (&acc)[N], bool own)
{
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) t = fmaf(acc[i][rr], 0.f, t);
    unsigned long long b = __ballot(own && !(t == 0.f));
    b |= b >> 32;
    b |= b >> 16;
    return unsigned(b) & 0xffffu;
}

template <class T>
__device__ __forceinline__ float exact_load(const T *p)
{
    if constexpr (sizeof(T) == 2) return __builtin_bit_cast(float, unsigned(*p) << 16);
    else return *p;
}
template <class T>
__device__ __forceinline__ void exact_store(T *p, float x)
{
    if constexpr (sizeof(T) == 2) *p = __builtin_bit_cast(T, (__bf16)x);
    else *p = x;
}
// The lane's number, found out on the spot: taken from the thread index, the compiler would keep that index and the six
// lane addresses of a sum over the wavefront in registers from the kernel's start on.
__device__ __forceinline__ int lane_here()
{
    int lane;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=&v"(lane));
    return lane;
}
__device__ __forceinline__ float other_lane(float x, int lane)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(4 * lane, __builtin_bit_cast(int, x)));
}
__device__ __forceinline__ float wave_sum(float x, int lane)
{
#pragma unroll
    for (int s = 1; s < 64; s *= 2) x += other_lane(x, lane ^ s);
    return x;
}
__device__ __forceinline__ float wave_max(float x, int lane)
{
#pragma unroll
    for (int s = 1; s < 64; s *= 2) x = fmaxf(x, other_lane(x, lane ^ s));
    return x;
}

// f(row, at, in): up to 64 neighbors of owner u at a time, one per lane: walked row, the lane's place inside a plane of the
// walked tensors, and whether it is a neighbor (else `at` is the place of one)
template <class Where, class F>
__device__ __forceinline__ void exact_neighbors(const BandArgs &a, const Where &w, int u, F &&f)
{
    const int n = a.b.bn[w.own], first = a.b.blo[w.own];
#pragma unroll 1
    for (int i = 0; i < n; ++i) {
        const int2 arc = a.b.arc[w.own * a.b.bmax + i];
#pragma unroll 1
        for (int t0 = 0; t0 < arc.y; t0 += 64) {
            const int t = t0 + w.lane;
            const int col = (u + arc.x + imin(t, arc.y - 1)) % w.nU;
            f(first + i, w.walk_at(first + i) + size_t(w.c_walk) * (col < 0 ? col + w.nU : col), t < arc.y);
        }
    }
}
// sum over the channels of (owner's value, the same for all lanes) * (the lane's neighbor's value)
template <class T>
__device__ __forceinline__ float exact_dot(const T *own, size_t plane_own, const T *walked, size_t plane_walk, int nch)
{
    float s = 0.f;
#pragma unroll 1
    for (int c = 0; c < nch; ++c) s = fmaf(exact_load(own + c * plane_own), exact_load(walked + c * plane_walk), s);
    return s;
}
// lane c: x += sum over the neighbors of p * (channel c of the walked tensor)
template <class T>
__device__ __forceinline__ void exact_add(float &x, float p, bool in, const T *walked, size_t plane_walk, int nch, int lane)
{
#pragma unroll 1
    for (int c = 0; c < nch; ++c) {
        const float s = wave_sum(in ? p * exact_load(walked + c * plane_walk) : 0.f, lane);
        if (c == lane) x += s;
    }
}

// The kernel's parameters read again: P lists them in order (they lie one behind the other at their natural alignment).
// What the evaluation below needs is taken from here, so that nothing of it stays in registers during the tile loop (kept
// alive it cost the kernels 3 to 10 %: 30 more scalar registers spilled, and d = 64 dq 2.02 -> 2.23 ms on 129 x 256, 32 slices).
template <class P>
__device__ __forceinline__ P kernel_params()
{
    static_assert(sizeof(P) % 8 == 0, "whole words");
    typedef const __attribute__((address_space(4))) unsigned long long *Words;
    Words p = (Words)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    struct {
        unsigned long long v[sizeof(P) / 8];
    } raw;
#pragma unroll
    for (unsigned i = 0; i < sizeof(P) / 8; ++i) raw.v[i] = p[i];
    return __builtin_bit_cast(P, raw);
}
__device__ __forceinline__ bool any_owner(unsigned owners) { return __builtin_expect(owners != 0, 0); }
// The three kernels: their parameters, and the evaluation of owners (bit n of owners[o]).
template <class T>
struct FwdParams {
    BandArgs a;
    const T *q, *k, *v;
    T *out;
    float *lse;
};
template <class T, class Where>
__device__ __forceinline__ void exact_fwd(unsigned owners, int wave)
{
    if (!any_owner(owners)) return;
    const auto p = kernel_params<FwdParams<T>>();
    Where w;
    w.set(p.a, 64 * wave + lane_here());
    const BandArgs &a = p.a;
    const float c2 = a.scale * kLog2e;
    const T *ks = p.k + size_t(w.bh) * a.d * w.plane_walk, *vs = p.v + size_t(w.bh) * a.e * w.plane_walk;
    w.each(owners, [&](int u) {
        const size_t qs = size_t(w.bh) * a.d * w.plane_own + w.own_at, os = size_t(w.bh) * a.e * w.plane_own + w.own_at;
        const size_t at_own = size_t(w.c_own) * u;
        float m = kMinRef, l = 0.f, acc = 0.f;
        exact_neighbors(a, w, u, [&](int row, size_t at, bool in) {
            const float s = exact_dot(p.q + qs + at_own, w.plane_own, ks + at, w.plane_walk, a.d) * c2;
            const float m_new = fmaxf(m, wave_max(in ? s : -INFINITY, w.lane)), corr = __builtin_amdgcn_exp2f(m - m_new);
            const float x = in ? a.omega_rel[row / w.c_walk] * __builtin_amdgcn_exp2f(s - m_new) : 0.f;
            l = l * corr + wave_sum(x, w.lane);
            acc *= corr;
            exact_add(acc, x, in, vs + at, w.plane_walk, a.e, w.lane);
            m = m_new;
        });
        if (w.lane < a.e) exact_store(p.out + os + w.lane * w.plane_own + at_own, acc / l);
        if (w.lane == 0)
            p.lse[size_t(w.bh) * w.plane_own + w.own_at + at_own] = (m + log2f(l * a.omega_ref)) * 0.6931471805599453f;
    });
}

template <class T>
struct DqParams {
    BandArgs a;
    const T *q, *k, *v, *o;
    const float *lse;
    const T *go;
    T *dq;
    float *Dws;
};
template <class T, class Where>
__device__ __forceinline__ void exact_dq(unsigned owners, int wave)
{
    if (!any_owner(owners)) return;
    const auto p = kernel_params<DqParams<T>>();
    Where w;
    w.set(p.a, 64 * wave + lane_here());
    const BandArgs &a = p.a;
    const float c2 = a.scale * kLog2e;
    const T *ks = p.k + size_t(w.bh) * a.d * w.plane_walk, *vs = p.v + size_t(w.bh) * a.e * w.plane_walk;
    w.each(owners, [&](int u) {
        const size_t qs = size_t(w.bh) * a.d * w.plane_own + w.own_at, os = size_t(w.bh) * a.e * w.plane_own + w.own_at;
        const size_t at_own = size_t(w.c_own) * u, c = os + imin(w.lane, a.e - 1) * w.plane_own + at_own;
        const float D = wave_sum(w.lane < a.e ? exact_load(p.go + c) * exact_load(p.o + c) : 0.f, w.lane);
        const float L2 = (p.lse[size_t(w.bh) * w.plane_own + w.own_at + at_own] - a.ln_omega_ref) * kLog2e;
        float acc = 0.f;
        exact_neighbors(a, w, u, [&](int row, size_t at, bool in) {
            const float s = exact_dot(p.q + qs + at_own, w.plane_own, ks + at, w.plane_walk, a.d);
            const float dp = exact_dot(p.go + os + at_own, w.plane_own, vs + at, w.plane_walk, a.e) - D;
            const float x = a.omega_rel[row / w.c_walk] * __builtin_amdgcn_exp2f(fmaf(s, c2, -L2));
            exact_add(acc, x * dp, in, ks + at, w.plane_walk, a.d, w.lane);
        });
        if (w.lane < a.d) exact_store(p.dq + qs + w.lane * w.plane_own + at_own, acc * a.scale);
    });
}

template <class T>
struct DkdvParams {
    BandArgs a;
    const T *q, *k, *v;
    const float *lse;
    const T *go;
    const float *Dws;
    T *dk, *dv;
};
template <class T, class Where>
__device__ __forceinline__ void exact_dkdv(unsigned owners, int wave)
{
    if (!any_owner(owners)) return;
    const auto p = kernel_params<DkdvParams<T>>();
    Where w;
    w.set(p.a, 64 * wave + lane_here());
    const BandArgs &a = p.a;
    const float c2 = a.scale * kLog2e;
    const size_t kv = size_t(w.bh) * w.plane_own, stat = size_t(w.bh) * w.plane_walk;
    const T *qs = p.q + a.d * stat, *gs = p.go + a.e * stat;
    w.each(owners, [&](int u) {
        const float omega = a.omega_rel[w.own / w.c_own];
        const size_t at_own = w.own_at + size_t(w.c_own) * u, ko = a.d * kv + at_own, vo = a.e * kv + at_own;
        float adk = 0.f, adv = 0.f;
        exact_neighbors(a, w, u, [&](int, size_t at, bool in) {
            const float s = exact_dot(p.k + ko, w.plane_own, qs + at, w.plane_walk, a.d);
            const float dp = exact_dot(p.v + vo, w.plane_own, gs + at, w.plane_walk, a.e) - p.Dws[stat + at];
            const float x = __builtin_amdgcn_exp2f(fmaf(s, c2, (a.ln_omega_ref - p.lse[stat + at]) * kLog2e));
            exact_add(adk, x * dp, in, qs + at, w.plane_walk, a.d, w.lane);
            exact_add(adv, x, in, gs + at, w.plane_walk, a.e, w.lane);
        });
        if (w.lane < a.d) exact_store(p.dk + ko + w.lane * w.plane_own, adk * (omega * a.scale));
        if (w.lane < a.e) exact_store(p.dv + vo + w.lane * w.plane_own, adv * omega);
    });
}

}  // namespace s2walk
