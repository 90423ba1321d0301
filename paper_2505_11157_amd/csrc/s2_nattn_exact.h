// One point of the neighborhood attention over its true neighbors only (device side).
//
// The matrix-core tiles (s2_nattn_patch_impl.h) give a staged column outside an owner's disk the
// weight zero, and zero times a NaN or an infinity is a NaN: a non-finite value next to a disk would spoil the point.  A
// mask on the staged values cannot tell owners apart that share a tile.  So a wavefront looks at its finished sums, and
// sums that are not finite are evaluated again here, where no other point is touched, except where it is a NaN of the owner's that
// makes all its sums NaN.  With finite inputs that costs one multiply-add per sum; the evaluation itself is slow (one owner at a time,
// lanes over its neighbors, then over the channels) and only runs where the inputs hold non-finite values or the results overflow.
#pragma once
#include "s2_nattn_walk.h"

namespace s2walk {

// bit n: is b true for one of the four lanes of owner n
__device__ __forceinline__ unsigned owner_bits(bool one)
{
    unsigned long long b = __ballot(one);
    b |= b >> 32;
    b |= b >> 16;
    return unsigned(b) & 0xffffu;
}
// owners (bit n) of a 16-owner tile with a sum that is not finite; own: the lane's owner is a point of the grid
template <int N>
__device__ __forceinline__ unsigned not_finite(const f32x4 (&acc)[N], bool own)
{
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) t = fmaf(acc[i][rr], 0.f, t);
    return owner_bits(own && !(t == 0.f));
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

// Lane i's value, the same for all lanes (i uniform)
__device__ __forceinline__ float lane_value(float x, int i)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), i));
}

// f(row, at, n): up to 64 neighbors of owner u at a time, one per lane: walked row, the lane's place inside a plane of the walked
// tensors (lanes from n on: that of a neighbor too), how many.  Ends where f says false.
template <class Where, class F>
__device__ __forceinline__ void exact_neighbors(const BandArgs &a, const Where &w, int u, F &&f)
{
    const int n = a.b.bn[w.own], first = a.b.blo[w.own];
    bool more = true;
#pragma unroll 1
    for (int i = 0; i < n && more; ++i) {
        const int2 arc = a.b.arc[w.own * a.b.bmax + i];
#pragma unroll 1
        for (int t0 = 0; t0 < arc.y && more; t0 += 64) {
            const int col = (u + arc.x + imin(t0 + w.lane, arc.y - 1)) % w.nU;
            const int at = int(w.walk_at(first + i)) + w.c_walk * (col < 0 ? col + w.nU : col);
            more = f(first + i, at, __builtin_amdgcn_readfirstlane(imin(arc.y - t0, 64)));
        }
    }
}
// Channel c of the owner in lane c, zero in the lanes behind the last
template <class T>
__device__ __forceinline__ float exact_own(const T *p, size_t plane_own, int nch, int lane)
{
    const float x = exact_load(p + size_t(imin(lane, nch - 1)) * plane_own);
    return lane < nch ? x : 0.f;
}
// Eight loads at a time here and below: they wait together (one at a time, a wavefront's sums over 64 neighbors took some 60 us).
// sum over the channels of (owner's value) * (the lane's neighbor's value)
template <class T>
__device__ __forceinline__ float exact_dot(float own, const T *walked, size_t plane_walk, int nch)
{
    float s = 0.f;
#pragma unroll 1
    for (int c0 = 0; c0 < nch; c0 += 8) {
        float x[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            x[j] = exact_load(walked);
            if (c0 + j + 1 < nch) walked += plane_walk;
            asm volatile("" : "+v"(walked));         // one lane address moved on, not eight uniform distances kept in scalar registers
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) s = fmaf(lane_value(own, c0 + j), c0 + j < nch ? x[j] : 0.f, s);
    }
    return s;
}
// lane c: x + sum over the n neighbors of (lane j's p) * (channel c of the walked tensor)
template <class T>
__device__ __forceinline__ float exact_add(float x, float p, int at, int n, const T *walked, size_t plane_walk, int nch, int lane)
{
    const T *ch = walked + size_t(imin(lane, nch - 1)) * plane_walk;
    p = lane < n ? p : 0.f;
#pragma unroll 1
    for (int j0 = 0; j0 < n; j0 += 8) {
        float y[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) y[j] = exact_load(ch + unsigned(__builtin_amdgcn_ds_bpermute(4 * (j0 + j), at)));
#pragma unroll
        for (int j = 0; j < 8; ++j) x = fmaf(lane_value(p, j0 + j), j0 + j < n ? y[j] : 0.f, x);
    }
    return x;
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
// What is the same for all lanes kept in vector registers all the same: the scalar ones are all in use
template <class P>
__device__ __forceinline__ P held_v(P p)
{
    asm volatile("" : "+v"(p));
    return p;
}
struct Held {
    int x;
    __device__ __forceinline__ Held(bool b) : x(b ? 1 : 0) { asm volatile("" : "+v"(x)); }
    __device__ __forceinline__ operator bool() const { return x != 0; }
};
// The three kernels: their parameters, and the evaluation of owners (bit n of owners).  marked(w, n): is the lane's channel of owner n
// wanted; the others are stored already.  A sum that is NaN stays it: an owner is done when all that are wanted are.
// 129 x 256, 32 slices, d = 32, float32, forward and backward, 2.1 ms without: every channel to the end, load after load, and as it is: one
// NaN of k, at a pole, 18.6 and 2.0 ms, of v 18.7 and 2.1, of dout 10.0 and 2.1, one infinity of k 18.6 and 4.0; everything NaN 189 and
// 1.5; one percent of v at random 186 and 16.7 (most owners have one next to their disk, in a channel that stays finite).
template <class T>
struct FwdParams {
    BandArgs a;
    const T *q, *k, *v;
    T *out;
    float *lse;
};
template <class T, class Where, class M>
__device__ __forceinline__ void exact_fwd(unsigned owners, unsigned no_lse, int wave, M &&marked)
{
    if (!any_owner(owners)) return;
    const auto p = kernel_params<FwdParams<T>>();
    Where w;
    w.set(p.a, 64 * wave + lane_here());
    const BandArgs &a = p.a;
    const float c2 = a.scale * kLog2e;
    const T *ks = p.k + size_t(w.bh) * a.d * w.plane_walk, *vs = p.v + size_t(w.bh) * a.e * w.plane_walk;
    w.each(owners, [&](int i, int u) {
        const size_t qs = size_t(w.bh) * a.d * w.plane_own + w.own_at, os = size_t(w.bh) * a.e * w.plane_own + w.own_at;
        const size_t at_own = size_t(w.c_own) * u;
        const bool wants_lse = no_lse >> i & 1;
        const Held mine = marked(w, i) && w.lane < a.e;
        const float q = exact_own(p.q + qs + at_own, w.plane_own, a.d, w.lane);
        float m = kMinRef, l = 0.f, acc = 0.f;
        exact_neighbors(a, w, u, [&](int row, int at, int n) {
            const bool in = w.lane < n;
            const float s = exact_dot(q, ks + at, w.plane_walk, a.d) * c2;
            const float m_new = fmaxf(m, wave_max(in ? s : -INFINITY, w.lane)), corr = __builtin_amdgcn_exp2f(m - m_new);
            const float x = in ? a.omega_rel[row / w.c_walk] * __builtin_amdgcn_exp2f(s - m_new) : 0.f;
            l = l * corr + wave_sum(x, w.lane);
            m = m_new;
            if (l != l) return false;                // so are all results, and they stay it
            acc = exact_add(acc * corr, x, at, n, vs, w.plane_walk, a.e, w.lane);
            return wants_lse || !__all(!mine || acc != acc);
        });
        if (mine) exact_store(p.out + os + w.lane * w.plane_own + at_own, acc / l);
        if (wants_lse && w.lane == 0)
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
template <class T, class Where, class M>
__device__ __forceinline__ void exact_dq(unsigned owners, int wave, M &&marked)
{
    if (!any_owner(owners)) return;
    const auto p = kernel_params<DqParams<T>>();
    Where w;
    w.set(p.a, 64 * wave + lane_here());
    const BandArgs &a = p.a;
    const float c2 = a.scale * kLog2e;
    const T *ks = held_v(p.k + size_t(w.bh) * a.d * w.plane_walk), *vs = held_v(p.v + size_t(w.bh) * a.e * w.plane_walk);
    w.each(owners, [&](int i, int u) {
        const Held mine = marked(w, i) && w.lane < a.d;
        const size_t qs = size_t(w.bh) * a.d * w.plane_own + w.own_at, os = size_t(w.bh) * a.e * w.plane_own + w.own_at;
        const size_t at_own = size_t(w.c_own) * u;
        const float q = exact_own(p.q + qs + at_own, w.plane_own, a.d, w.lane), go = exact_own(p.go + os + at_own, w.plane_own, a.e, w.lane);
        const float D = wave_sum(go * exact_own(p.o + os + at_own, w.plane_own, a.e, w.lane), w.lane);
        const float L2 = (p.lse[size_t(w.bh) * w.plane_own + w.own_at + at_own] - a.ln_omega_ref) * kLog2e;
        float acc = 0.f;
        exact_neighbors(a, w, u, [&](int row, int at, int n) {
            const float s = exact_dot(q, ks + at, w.plane_walk, a.d);
            const float dp = exact_dot(go, vs + at, w.plane_walk, a.e) - D;
            const float x = a.omega_rel[row / w.c_walk] * __builtin_amdgcn_exp2f(fmaf(s, c2, -L2));
            acc = exact_add(acc, x * dp, at, n, ks, w.plane_walk, a.d, w.lane);
            return !__all(!mine || acc != acc);
        });
        if (mine) exact_store(p.dq + qs + w.lane * w.plane_own + at_own, acc * a.scale);
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
template <class T, class Where, class MK, class MV>
__device__ __forceinline__ void exact_dkdv(unsigned owners, int wave, MK &&marked_k, MV &&marked_v)
{
    if (!any_owner(owners)) return;
    const auto p = kernel_params<DkdvParams<T>>();
    Where w;
    w.set(p.a, 64 * wave + lane_here());
    const BandArgs &a = p.a;
    const float c2 = a.scale * kLog2e;
    const size_t kv = size_t(w.bh) * w.plane_own, stat = size_t(w.bh) * w.plane_walk;
    const T *qs = held_v(p.q + a.d * stat), *gs = held_v(p.go + a.e * stat);
    w.each(owners, [&](int i, int u) {
        const Held mine_k = marked_k(w, i) && w.lane < a.d, mine_v = marked_v(w, i) && w.lane < a.e;
        const float omega = a.omega_rel[w.own / w.c_own];
        const size_t at_own = w.own_at + size_t(w.c_own) * u, ko = a.d * kv + at_own, vo = a.e * kv + at_own;
        const float k = exact_own(p.k + ko, w.plane_own, a.d, w.lane), v = exact_own(p.v + vo, w.plane_own, a.e, w.lane);
        float adk = 0.f, adv = 0.f;
        exact_neighbors(a, w, u, [&](int, int at, int n) {
            const float s = exact_dot(k, qs + at, w.plane_walk, a.d);
            const float dp = exact_dot(v, gs + at, w.plane_walk, a.e) - p.Dws[stat + at];
            const float x = __builtin_amdgcn_exp2f(fmaf(s, c2, (a.ln_omega_ref - p.lse[stat + at]) * kLog2e));
            adk = exact_add(adk, x * dp, at, n, qs, w.plane_walk, a.d, w.lane);
            adv = exact_add(adv, x, at, n, gs, w.plane_walk, a.e, w.lane);
            return !__all((!mine_k || adk != adk) && (!mine_v || adv != adv));
        });
        if (mine_k) exact_store(p.dk + ko + w.lane * w.plane_own, adk * (omega * a.scale));
        if (mine_v) exact_store(p.dv + vo + w.lane * w.plane_own, adv * omega);
    });
}

}  // namespace s2walk
