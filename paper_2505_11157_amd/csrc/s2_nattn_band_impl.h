// Neighborhood attention (Sec. 3.3, eq. (9)-(10); gradients App. B.4) on the fp32 matrix cores: band tiles of 16 keys x
// 16 outputs on v_mfma_f32_16x16x4_f32, float32 throughout, for d, e <= 64 (rounded up to 16, 32 or 64 channels: the
// missing ones are zeros in LDS and registers) and any pair of grids.  s2_nattn_walk.h describes the walk; a staged row
// is channel-major, as it lies in memory, and serves every wavefront whose band holds it.
//
// Operands of v_mfma_f32_16x16x4_f32 (A: 16 x 4, one value per lane (row = lane & 15, k = lane >> 4); B: 4 x 16
// (k = lane >> 4, column = lane & 15); C/D: lane holds rows 4 (lane >> 4) + 0..3 of column lane & 15):
//   S^T = K Q^T      A = K[channel 4 kb + g][key column]  (one LDS word per lane), B = q of the lane's output,
//                    kb = 0 .. d/4 - 1: lane (n, g) ends with the logits of keys 4 g + 0..3 for output n;
//   O^T += V P^T     the contraction index of instruction j is key 4 g + j, so B is the lane's own probability j
//                    (no data movement between lanes) and A = V[channel 16 mt + (lane & 15)][keys 4 g + 0..3]:
//                    one 16-byte LDS read serves four instructions.
// Channel row c of a staged tile starts at c * pitch + 4 ((c >> 2) & 3) floats with a pitch of 16 mod 32 words: the four
// rows 4 kb + g of the first read pattern fall into four different groups of 16 banks, and the 16 rows 16 mt + n of
// the second into 16 different groups of four banks, so both are free of bank conflicts.
// Softmax: base 2, lazy reference maximum over the bare logits (moves when exceeded by 2^8; only then do the four lanes of
// an output exchange maxima).  The quadrature weight is a factor, not a bias of |log2 omega| ~ 10 that would cost every
// exponent a rounding at that magnitude: the forward stages omega V, dq stages omega V and starts dP from -omega D, dk/dv
// multiplies its finished sums.  Every matrix result is consumed in the block that issues it.
//
// Staging (MODE): kWide copies pieces of four columns (walked rows contiguous in memory, longitude count a multiple of four,
// so that no piece straddles the seam); kNarrow copies column by column, a wavefront on 64 columns of one channel at a
// time (odd counts, the classes of a finer grid); kRagged does the same for channel counts other than 16, 32 or 64.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "s2_internal.h"
#include "s2_nattn_band.h"
#include "s2_nattn_exact.h"
#include "s2_nattn_walk.h"

namespace {

using namespace s2walk;

template <int D, int NO>
struct Geo {
    static constexpr int OW = 16 * NO;           // longitudes per workgroup
    static constexpr int SW = OW + 64;           // staged columns
    static constexpr int COLS = SW + 32;         // + zeroed padding (a tile may reach past the window)
    static constexpr int PITCH = (COLS + 16) % 32 == 16 ? COLS + 16 : COLS + 32;      // floats per channel row (16 mod 32); row c starts 4 ((c >> 2) & 3) floats in
    static constexpr int TILE = D * PITCH;       // floats per staged tensor
    static_assert(PITCH % 32 == 16, "geometry");
};

__device__ __forceinline__ f32x4 mfma4(float a, float b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ float max4(float a, float b, float c, float d)
{
    float r;
    asm("v_max3_f32 %0, %1, %2, %3\n\tv_max_f32 %0, %0, %4" : "=&v"(r) : "v"(a), "v"(b), "v"(c), "v"(d));
    return r;
}

// The reads of a first product's operands up to AHEAD of the matrix instructions that use them (left alone, the compiler waits
// for every single one: 64 x 128, 8 slices, d = 32 forward 83.2 against 81.7 us).
template <int READS, int AHEAD = READS < 8 ? READS : 8>
__device__ __forceinline__ void read_ahead()
{
    constexpr int STEP = AHEAD < 4 ? AHEAD : 4;
    __builtin_amdgcn_sched_group_barrier(0x100, AHEAD, 0);
#pragma unroll
    for (int i = AHEAD; i < READS; i += STEP) {
        __builtin_amdgcn_sched_group_barrier(0x008, STEP, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, STEP, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, AHEAD, 0);
}


// One tensor's stage in registers, and its way to LDS.
template <int D, int NO, int MODE>
struct Stage {
    using G = Geo<D, NO>;
    using Idx = StageIdx<float, D, G::SW, MODE>;
    static constexpr bool WIDE = MODE == kWide;
    static constexpr int NC = Idx::NC, NJ = D / 4;
    std::conditional_t<WIDE, f32x4, float> r[WIDE ? Idx::NP : NJ * NC];
    __device__ __forceinline__ void load(const BandWhere &w, const Idx &at, const float *row, int nch)
    {
        if constexpr (WIDE) {
#pragma unroll
            for (int j = 0; j < Idx::NP; ++j) r[j] = load_at<f32x4>(row, at.at(j));
        } else {
            size_t step = w.plane_walk;
            asm volatile("" : "+s"(step));   // else the compiler keeps every channel's address in (spilled) scalar registers
            int c = MODE == kRagged ? imin(w.wave, nch - 1) : w.wave;
            const float *p = row + c * step;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
#pragma unroll
                for (int i = 0; i < NC; ++i) r[j * NC + i] = load_at<float>(p, at.at(i));
                // past the last channel: that channel again (not stored); a branch around a load would make the compiler
                // wait for all loads in flight where its sides meet
                const int up = MODE == kRagged ? imin(w.wave + 4 * j + 4, nch - 1) - c : 4;
                p += up * step;
                c += up;
            }
        }
    }
    __device__ __forceinline__ void store(const BandWhere &w, float *tile, int nch, float factor = 1.f) const
    {
        if constexpr (WIDE) {
#pragma unroll
            for (int j = 0; j < Idx::NP; ++j) {
                const int i = w.tid + 256 * j, c = i / Idx::P4, pc = i % Idx::P4;
                if (Idx::EVEN || i < D * Idx::P4)
                    *reinterpret_cast<f32x4 *>(tile + c * G::PITCH + 4 * ((c >> 2) & 3) + 4 * pc) = r[j] * factor;
            }
        } else {
            float *p = tile + w.wave * G::PITCH + w.lane;
#pragma unroll
            for (int i = 0; i < NC; ++i) {
                if (64 * i + 64 > G::SW && w.lane + 64 * i >= G::SW) break;
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                    if (MODE != kRagged || w.wave + 4 * j < nch)
                        p[4 * j * G::PITCH + 4 * (j & 3) + 64 * i] = r[j * NC + i] * factor;
            }
        }
    }
};

// ---------------------------------------------------------------------------------------------------------------
// Forward.  Up to 32 channels four wavefronts per SIMD, as many as the two tiles in LDS allow (91 x 181, 32 slices: 424 us; with 129
// registers, three wavefronts, 465 us).
template <int D, int NO, int MODE>
__global__ void __launch_bounds__(256, D <= 32 ? 4 : 2)
nattn_fwd_band(BandArgs a, const float *__restrict__ q, const float *__restrict__ k, const float *__restrict__ v, float *__restrict__ out,
               float *__restrict__ lse)
{
    using G = Geo<D, NO>;
    extern __shared__ __attribute__((aligned(16))) float lds[];
    float *Kc = lds, *Vc = lds + G::TILE;
    BandWhere w;
    w.set<G::OW>(a);
    const int nU = w.nU, n = w.n, g = w.g;
    const float c2 = a.scale * kLog2e;
    const float *qs = q + size_t(w.bh) * (MODE == kRagged ? a.d : D) * w.plane_own + w.own_at;
    const float *ks = k + size_t(w.bh) * (MODE == kRagged ? a.d : D) * w.plane_walk, *vs = v + size_t(w.bh) * (MODE == kRagged ? a.e : D) * w.plane_walk;

    float qreg[NO][D / 4];
    f32x4 acc[NO][D / 16];
    float m[NO], l[NO];
#pragma unroll
    for (int o = 0; o < NO; ++o) {
        const int u = w.W0 + 16 * o + n;
        const bool own = w.active && u < nU;
#pragma unroll
        for (int kb = 0; kb < D / 4; ++kb)
            qreg[o][kb] = own && has<MODE>(4 * kb + g, a.d) ? *(qs + size_t(4 * kb + g) * w.plane_own + w.c_own * u) : 0.f;
#pragma unroll
        for (int mt = 0; mt < D / 16; ++mt) acc[o][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
        m[o] = kMinRef;
        l[o] = 0.f;
    }
    Walker wk;
    typename Stage<D, NO, MODE>::Idx at;
    at.init(w);
    Stage<D, NO, MODE> rk, rv;
    bool more = wk.start<G::OW, G::SW>(a.b, w.first, w.own, a.omega_rel, w.lane, w.Wb);
    if (more) {
        const size_t row = w.walk_at(wk.r);
        at.set(w, wk.cur.Xs0);
        rk.load(w, at, ks + row, a.d);
        rv.load(w, at, vs + row, a.e);
    }
    for (int i = w.tid; i < 2 * G::TILE; i += 256) lds[i] = 0.f;
    while (more) {
        const float omega = wk.rows.weight(wk.r);
        __syncthreads();                    // everybody is done with the previous stage (first pass: with the zero fill)
        rk.store(w, Kc, a.d);
        rv.store(w, Vc, a.e, omega);
        __syncthreads();
        const RowPlan p = wk.cur;
        const int Xst = p.Xs0 + wk.s * G::SW;
        int lo, cnt;
        wk.rows.arc(wk.r, lo, cnt);
        more = wk.next<G::OW, G::SW>(nU, w.Wb);
        if (more) {
            const size_t row = w.walk_at(wk.r);
            at.set(w, wk.cur.Xs0 + wk.s * G::SW);
            rk.load(w, at, ks + row, a.d);
            rv.load(w, at, vs + row, a.e);
        }
        if (cnt <= 0) continue;
        // one copy of the tile loop for rows on the common grid, one for rows whose tiles follow their owners (backward: one
        // copy for both; two take the registers of a wavefront: d = 64 dk/dv on 129 x 256, 32 slices, 3.67 against 2.47 ms)
        auto tiles = [&](auto kind) {
            constexpr int KIND = decltype(kind)::value;
#pragma unroll
            for (int o = 0; o < NO; ++o) {
                if (w.W0 + 16 * o >= nU) break;
                const int Wo = w.Wb + 16 * o;
                const int T0 = on_grid<KIND>(p) ? Xst : (Wo + lo) & ~3;
                const int Tend = on_grid<KIND>(p) ? imin(Xst + G::SW, p.Xend) : Wo + 15 + lo + cnt;
                TileRow<KIND> tr;
                tr.start(p, T0, Wo, lo, cnt, nU);
                for (int Xt = T0; Xt < Tend; Xt += 16, tr.next()) {
                    if (!tr.touch()) continue;
                    const int col0 = Xt - Xst;
                    const float *kp = Kc + g * G::PITCH + col0 + n;
                    f32x4 sc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int kb = 0; kb < D / 4; ++kb) sc = mfma4(kp[kb * 4 * G::PITCH + 4 * (kb & 3)], qreg[o][kb], sc);
                    read_ahead<D / 4>();
                    float x[4];
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr) x[rr] = sc[rr] * c2;
                    if (tr.mask(Xt)) {
                        bool keep[4];
                        tr.keep(keep, Xt, 4 * g, n);
#pragma unroll
                        for (int rr = 0; rr < 4; ++rr) x[rr] = keep[rr] ? x[rr] : -INFINITY;
                    }
                    float mx = max4(x[0], x[1], x[2], x[3]);
                    if (__any(mx > m[o] + 8.f)) {
                        mx = group_max(mx);
                        const float m_new = mx > m[o] + 8.f ? mx : m[o];
                        const float corr = __builtin_amdgcn_exp2f(m[o] - m_new);
                        m[o] = m_new;
                        l[o] *= corr;
#pragma unroll
                        for (int mt = 0; mt < D / 16; ++mt)
#pragma unroll
                            for (int rr = 0; rr < 4; ++rr) acc[o][mt][rr] *= corr;
                    }
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr) {
                        x[rr] = __builtin_amdgcn_exp2f(x[rr] - m[o]);
                        l[o] = fmaf(omega, x[rr], l[o]);
                    }
                    const float *vp = Vc + n * G::PITCH + 4 * ((n >> 2) & 3) + col0 + 4 * g;
                    f32x4 va[D / 16];
#pragma unroll
                    for (int mt = 0; mt < D / 16; ++mt) va[mt] = *reinterpret_cast<const f32x4 *>(vp + mt * 16 * G::PITCH);
#pragma unroll
                    for (int j = 0; j < 4; ++j)          // consecutive instructions belong to different accumulators
#pragma unroll
                        for (int mt = 0; mt < D / 16; ++mt) acc[o][mt] = mfma4(va[mt][j], x[j], acc[o][mt]);
                    settle(acc[o]);
                }
            }
        };
        if (p.multi) tiles(std::integral_constant<int, kGridTiles>());
        else tiles(std::integral_constant<int, kOwnTiles>());
    }
    if (!w.active) return;
    unsigned again[NO];                  // owners whose sums took in a non-finite value (s2_nattn_exact.h)
#pragma unroll
    for (int o = 0; o < NO; ++o) {
        const float lt = group_sum(l[o]);
        const int u = w.W0 + 16 * o + n;
        again[o] = not_finite(acc[o], u < nU);
        if (u >= nU || (again[o] >> n & 1)) continue;
        const float inv = 1.f / lt;
        float *ob = out + size_t(w.bh) * (MODE == kRagged ? a.e : D) * w.plane_own + w.own_at + w.c_own * u;
#pragma unroll
        for (int mt = 0; mt < D / 16; ++mt)
#pragma unroll
            for (int rr = 0; rr < 4; ++rr)
                if (has<MODE>(16 * mt + 4 * g + rr, a.e)) *(ob + size_t(16 * mt + 4 * g + rr) * w.plane_own) = acc[o][mt][rr] * inv;
        if (g == 0)
            lse[size_t(w.bh) * w.plane_own + w.own_at + w.c_own * u] = (m[o] + log2f(lt * a.omega_ref)) * 0.6931471805599453f;
    }
    exact_fwd<float, G::OW>(again, w.wave);
}

// ---------------------------------------------------------------------------------------------------------------
// Backward, query side: dq and D_i = dout_i . out_i (written for the key-side launch).
template <int D, int NO, int MODE>
__global__ void __launch_bounds__(256, D <= 32 ? 4 : 2)
nattn_bwd_dq_band(BandArgs a, const float *__restrict__ q, const float *__restrict__ k, const float *__restrict__ v,
                  const float *__restrict__ o_, const float *__restrict__ lse, const float *__restrict__ go, float *__restrict__ dq,
                  float *__restrict__ Dws)
{
    using G = Geo<D, NO>;
    extern __shared__ __attribute__((aligned(16))) float lds[];
    float *Kc = lds, *Vc = lds + G::TILE;
    BandWhere w;
    w.set<G::OW>(a);
    const int nU = w.nU, n = w.n, g = w.g;
    const float c2 = a.scale * kLog2e;
    const size_t slice_q = size_t(w.bh) * (MODE == kRagged ? a.d : D) * w.plane_own + w.own_at, slice_o = size_t(w.bh) * (MODE == kRagged ? a.e : D) * w.plane_own + w.own_at;
    const float *ks = k + size_t(w.bh) * (MODE == kRagged ? a.d : D) * w.plane_walk, *vs = v + size_t(w.bh) * (MODE == kRagged ? a.e : D) * w.plane_walk;

    float qreg[NO][D / 4], greg[NO][D / 4];
    f32x4 acc[NO][D / 16];
    float L2[NO], Dn[NO];
#pragma unroll
    for (int o = 0; o < NO; ++o) {
#pragma unroll
        for (int mt = 0; mt < D / 16; ++mt) acc[o][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
        L2[o] = 0.f;
        Dn[o] = 0.f;
        float dsum = 0.f;
        const int u = w.W0 + 16 * o + n;
        const bool own = w.active && u < nU;
#pragma unroll
        for (int kb = 0; kb < D / 4; ++kb) {
            const int c = 4 * kb + g;
            const size_t at = size_t(c) * w.plane_own + w.c_own * u;
            qreg[o][kb] = own && has<MODE>(c, a.d) ? *(q + slice_q + at) : 0.f;
            greg[o][kb] = own && has<MODE>(c, a.e) ? *(go + slice_o + at) : 0.f;
            dsum = fmaf(greg[o][kb], own && has<MODE>(c, a.e) ? *(o_ + slice_o + at) : 0.f, dsum);
        }
        dsum = group_sum(dsum);
        if (own) {
            const size_t at = size_t(w.bh) * w.plane_own + w.own_at + w.c_own * u;
            if (g == 0) Dws[at] = dsum;
            Dn[o] = -dsum;
            L2[o] = (lse[at] - a.ln_omega_ref) * kLog2e;
        }
    }
    Walker wk;
    typename Stage<D, NO, MODE>::Idx at;
    at.init(w);
    Stage<D, NO, MODE> rk, rv;
    bool more = wk.start<G::OW, G::SW>(a.b, w.first, w.own, a.omega_rel, w.lane, w.Wb);
    if (more) {
        const size_t row = w.walk_at(wk.r);
        at.set(w, wk.cur.Xs0);
        rk.load(w, at, ks + row, a.d);
        rv.load(w, at, vs + row, a.e);
    }
    for (int i = w.tid; i < 2 * G::TILE; i += 256) lds[i] = 0.f;
    while (more) {
        const float omega = wk.rows.weight(wk.r);
        __syncthreads();
        rk.store(w, Kc, a.d);
        rv.store(w, Vc, a.e, omega);
        __syncthreads();
        const RowPlan p = wk.cur;
        const int Xst = p.Xs0 + wk.s * G::SW;
        int lo, cnt;
        wk.rows.arc(wk.r, lo, cnt);
        more = wk.next<G::OW, G::SW>(nU, w.Wb);
        if (more) {
            const size_t row = w.walk_at(wk.r);
            at.set(w, wk.cur.Xs0 + wk.s * G::SW);
            rk.load(w, at, ks + row, a.d);
            rv.load(w, at, vs + row, a.e);
        }
        if (cnt <= 0) continue;
        // one copy of the tile loop for rows on the common grid, one for rows whose tiles follow their owners (backward: one
        // copy for both; two take the registers of a wavefront: d = 64 dk/dv on 129 x 256, 32 slices, 3.67 against 2.47 ms)
        auto tiles = [&](auto kind) {
            constexpr int KIND = decltype(kind)::value;
#pragma unroll
            for (int o = 0; o < NO; ++o) {
                if (w.W0 + 16 * o >= nU) break;
                const int Wo = w.Wb + 16 * o;
                const int T0 = on_grid<KIND>(p) ? Xst : (Wo + lo) & ~3;
                const int Tend = on_grid<KIND>(p) ? imin(Xst + G::SW, p.Xend) : Wo + 15 + lo + cnt;
                const float Dw = Dn[o] * omega;
                TileRow<KIND> tr;
                tr.start(p, T0, Wo, lo, cnt, nU);
                for (int Xt = T0; Xt < Tend; Xt += 16, tr.next()) {
                    if (!tr.touch()) continue;
                    const int col0 = Xt - Xst;
                    const float *kp = Kc + g * G::PITCH + col0 + n, *vp = Vc + g * G::PITCH + col0 + n;
                    f32x4 sc = {0.f, 0.f, 0.f, 0.f}, dp = {Dw, Dw, Dw, Dw};
#pragma unroll
                    for (int kb = 0; kb < D / 4; ++kb) {
                        sc = mfma4(kp[kb * 4 * G::PITCH + 4 * (kb & 3)], qreg[o][kb], sc);
                        dp = mfma4(vp[kb * 4 * G::PITCH + 4 * (kb & 3)], greg[o][kb], dp);
                    }
                    read_ahead<D / 2>();
                    const float *kq = Kc + n * G::PITCH + 4 * ((n >> 2) & 3) + col0 + 4 * g;
                    f32x4 ka[D / 16];
#pragma unroll
                    for (int mt = 0; mt < D / 16; ++mt) ka[mt] = *reinterpret_cast<const f32x4 *>(kq + mt * 16 * G::PITCH);
                    float ds[4];
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr) ds[rr] = __builtin_amdgcn_exp2f(fmaf(sc[rr], c2, -L2[o])) * dp[rr];
                    if (tr.mask(Xt)) {
                        bool keep[4];
                        tr.keep(keep, Xt, 4 * g, n);
#pragma unroll
                        for (int rr = 0; rr < 4; ++rr) ds[rr] = keep[rr] ? ds[rr] : 0.f;
                    }
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int mt = 0; mt < D / 16; ++mt) acc[o][mt] = mfma4(ka[mt][j], ds[j], acc[o][mt]);
                }
            }
        };
        tiles(std::integral_constant<int, kAnyTiles>());
    }
    if (!w.active) return;
    unsigned again[NO];                  // owners whose sums took in a non-finite value (s2_nattn_exact.h)
#pragma unroll
    for (int o = 0; o < NO; ++o) {
        const int u = w.W0 + 16 * o + n;
        again[o] = not_finite(acc[o], u < nU);
        if (u >= nU || (again[o] >> n & 1)) continue;
        float *ob = dq + slice_q + w.c_own * u;
#pragma unroll
        for (int mt = 0; mt < D / 16; ++mt)
#pragma unroll
            for (int rr = 0; rr < 4; ++rr)
                if (has<MODE>(16 * mt + 4 * g + rr, a.d)) *(ob + size_t(16 * mt + 4 * g + rr) * w.plane_own) = acc[o][mt][rr] * a.scale;
    }
    exact_dq<float, G::OW>(again, w.wave);
}

// ---------------------------------------------------------------------------------------------------------------
// Backward, key side: owners are input points, the transposed band gives the output latitudes; q, dout, lse and D
// of a stage's outputs are staged together.
template <int D, int NO, int MODE>
__global__ void __launch_bounds__(256, D == 16 && MODE != kRagged ? 6 : 2)
nattn_bwd_dkdv_band(BandArgs a, const float *__restrict__ q, const float *__restrict__ k, const float *__restrict__ v,
                    const float *__restrict__ lse, const float *__restrict__ go, const float *__restrict__ Dws,
                    float *__restrict__ dk, float *__restrict__ dv)
{
    using G = Geo<D, NO>;
    extern __shared__ __attribute__((aligned(16))) float lds[];
    float *Qc = lds, *Gc = lds + G::TILE, *Ls = lds + 2 * G::TILE, *Dn = Ls + G::COLS;
    BandWhere w;
    w.set<G::OW>(a);
    const int nU = w.nU, n = w.n, g = w.g;
    const float c2 = a.scale * kLog2e, lref = a.ln_omega_ref;
    const size_t slice_k = size_t(w.bh) * (MODE == kRagged ? a.d : D) * w.plane_own + w.own_at, slice_v = size_t(w.bh) * (MODE == kRagged ? a.e : D) * w.plane_own + w.own_at;
    const float *qs = q + size_t(w.bh) * (MODE == kRagged ? a.d : D) * w.plane_walk, *gs = go + size_t(w.bh) * (MODE == kRagged ? a.e : D) * w.plane_walk;
    const float *ls = lse + size_t(w.bh) * w.plane_walk, *Ds = Dws + size_t(w.bh) * w.plane_walk;
    // the quadrature weight is the owner's own here: it multiplies the finished sums (one rounding instead of one in every
    // exponent; a latitude of weight zero has no arcs)
    const float omega = w.active ? a.omega_rel[w.own / w.c_own] : 0.f;

    float kreg[NO][D / 4], vreg[NO][D / 4];
    f32x4 adk[NO][D / 16], adv[NO][D / 16];
#pragma unroll
    for (int o = 0; o < NO; ++o) {
        const int u = w.W0 + 16 * o + n;
        const bool own = w.active && u < nU;
#pragma unroll
        for (int mt = 0; mt < D / 16; ++mt) adk[o][mt] = adv[o][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kb = 0; kb < D / 4; ++kb) {
            const int c = 4 * kb + g;
            const size_t at = size_t(c) * w.plane_own + w.c_own * u;
            kreg[o][kb] = own && has<MODE>(c, a.d) ? *(k + slice_k + at) : 0.f;
            vreg[o][kb] = own && has<MODE>(c, a.e) ? *(v + slice_v + at) : 0.f;
        }
    }
    // minus the logsumexp (base 2, relative) and -D of a stage's columns: one pair per thread, turned into that on the way to LDS
    // (arithmetic on a value just requested would wait for it and for the whole stage requested before it)
    static_assert(G::SW <= 256, "stage width");
    float rl = 0.f, rd = 0.f;
    auto load_stat = [&](size_t row, int Xs) {
        if (w.tid < G::SW) {
            const size_t at = row + w.c_walk * wrap_stage(Xs, w.tid, G::SW, nU, w.inv_nU);
            rl = ls[at];
            rd = Ds[at];
        }
    };
    Walker wk;
    typename Stage<D, NO, MODE>::Idx at;
    at.init(w);
    Stage<D, NO, MODE> rq, rg;
    bool more = wk.start<G::OW, G::SW>(a.b, w.first, w.own, nullptr, w.lane, w.Wb);
    if (more) {
        const size_t row = w.walk_at(wk.r);
        at.set(w, wk.cur.Xs0);
        rq.load(w, at, qs + row, a.d);
        rg.load(w, at, gs + row, a.e);
        load_stat(row, wk.cur.Xs0);
    }
    for (int i = w.tid; i < 2 * G::TILE + 2 * G::COLS; i += 256) lds[i] = 0.f;
    while (more) {
        __syncthreads();
        rq.store(w, Qc, a.d);
        rg.store(w, Gc, a.e);
        if (w.tid < G::SW) {
            Ls[w.tid] = (lref - rl) * kLog2e;
            Dn[w.tid] = -rd;
        }
        __syncthreads();
        const RowPlan p = wk.cur;
        const int Xst = p.Xs0 + wk.s * G::SW;
        int lo, cnt;
        wk.rows.arc(wk.r, lo, cnt);
        more = wk.next<G::OW, G::SW>(nU, w.Wb);
        if (more) {
            const size_t row = w.walk_at(wk.r);
            at.set(w, wk.cur.Xs0 + wk.s * G::SW);
            rq.load(w, at, qs + row, a.d);
            rg.load(w, at, gs + row, a.e);
            load_stat(row, wk.cur.Xs0 + wk.s * G::SW);
        }
        if (cnt <= 0) continue;
        // one copy of the tile loop for rows on the common grid, one for rows whose tiles follow their owners (backward: one
        // copy for both; two take the registers of a wavefront: d = 64 dk/dv on 129 x 256, 32 slices, 3.67 against 2.47 ms)
        auto tiles = [&](auto kind) {
            constexpr int KIND = decltype(kind)::value;
#pragma unroll
            for (int o = 0; o < NO; ++o) {
                if (w.W0 + 16 * o >= nU) break;
                const int Wo = w.Wb + 16 * o;
                const int T0 = on_grid<KIND>(p) ? Xst : (Wo + lo) & ~3;
                const int Tend = on_grid<KIND>(p) ? imin(Xst + G::SW, p.Xend) : Wo + 15 + lo + cnt;
                TileRow<KIND> tr;
                tr.start(p, T0, Wo, lo, cnt, nU);
                for (int Xt = T0; Xt < Tend; Xt += 16, tr.next()) {
                    if (!tr.touch()) continue;
                    const int col0 = Xt - Xst;
                    const float *qp = Qc + g * G::PITCH + col0 + n, *gp = Gc + g * G::PITCH + col0 + n;
                    const f32x4 L = *reinterpret_cast<const f32x4 *>(Ls + col0 + 4 * g);
                    f32x4 sc = {0.f, 0.f, 0.f, 0.f}, dp = *reinterpret_cast<const f32x4 *>(Dn + col0 + 4 * g);
#pragma unroll
                    for (int kb = 0; kb < D / 4; ++kb) {
                        sc = mfma4(qp[kb * 4 * G::PITCH + 4 * (kb & 3)], kreg[o][kb], sc);
                        dp = mfma4(gp[kb * 4 * G::PITCH + 4 * (kb & 3)], vreg[o][kb], dp);
                    }
                    if constexpr (D < 64 || MODE == kWide) read_ahead<D / 2>();       // else no registers left for it
                    float pr[4], ds[4];
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr) {
                        pr[rr] = __builtin_amdgcn_exp2f(fmaf(sc[rr], c2, L[rr]));
                        ds[rr] = pr[rr] * dp[rr];
                    }
                    if (tr.mask(Xt)) {
                        bool keep[4];
                        tr.keep(keep, Xt, 4 * g, n);
#pragma unroll
                        for (int rr = 0; rr < 4; ++rr) {
                            pr[rr] = keep[rr] ? pr[rr] : 0.f;
                            ds[rr] = keep[rr] ? ds[rr] : 0.f;
                        }
                    }
                    const int at = n * G::PITCH + 4 * ((n >> 2) & 3) + col0 + 4 * g;
                    f32x4 ga[D / 16], qa[D / 16];
#pragma unroll
                    for (int mt = 0; mt < D / 16; ++mt) {
                        ga[mt] = *reinterpret_cast<const f32x4 *>(Gc + at + mt * 16 * G::PITCH);
                        qa[mt] = *reinterpret_cast<const f32x4 *>(Qc + at + mt * 16 * G::PITCH);
                    }
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int mt = 0; mt < D / 16; ++mt) {
                            adv[o][mt] = mfma4(ga[mt][j], pr[j], adv[o][mt]);
                            adk[o][mt] = mfma4(qa[mt][j], ds[j], adk[o][mt]);
                        }
                }
            }
        };
        tiles(std::integral_constant<int, kAnyTiles>());
    }
    if (!w.active) return;
    unsigned again[NO];                  // owners whose sums took in a non-finite value (s2_nattn_exact.h)
#pragma unroll
    for (int o = 0; o < NO; ++o) {
        const int u = w.W0 + 16 * o + n;
        again[o] = not_finite(adk[o], u < nU) | not_finite(adv[o], u < nU);
        if (u >= nU || (again[o] >> n & 1)) continue;
#pragma unroll
        for (int mt = 0; mt < D / 16; ++mt)
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                const int c = 16 * mt + 4 * g + rr;
                const size_t at = size_t(c) * w.plane_own + w.c_own * u;
                if (has<MODE>(c, a.d)) *(dk + slice_k + at) = adk[o][mt][rr] * (omega * a.scale);
                if (has<MODE>(c, a.e)) *(dv + slice_v + at) = adv[o][mt][rr] * omega;
            }
    }
    exact_dkdv<float, G::OW>(again, w.wave);
}

template <int D, int NO>
constexpr size_t fwd_lds() { return size_t(2) * Geo<D, NO>::TILE * sizeof(float); }
template <int D, int NO>
constexpr size_t dkdv_lds() { return (size_t(2) * Geo<D, NO>::TILE + 2 * Geo<D, NO>::COLS) * sizeof(float); }

template <int D, int NO, int MODE, bool DKDV>
int configure_one()
{
    auto raise = [](const void *f, size_t bytes) {
        return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes)) != hipSuccess;
    };
    int rc = 0;
    if constexpr (DKDV) rc = raise(reinterpret_cast<const void *>(nattn_bwd_dkdv_band<D, NO, MODE>), dkdv_lds<D, NO>());
    return rc || raise(reinterpret_cast<const void *>(nattn_bwd_dq_band<D, NO, MODE>), fwd_lds<D, NO>()) ||
           raise(reinterpret_cast<const void *>(nattn_fwd_band<D, NO, MODE>), fwd_lds<D, NO>());
}

template <int D, int NO>
unsigned blocks(const S2BandSide &b, int nbh)
{
    return unsigned(long((b.n_own + 3) / 4) * nbh * ((b.nU + Geo<D, NO>::OW - 1) / Geo<D, NO>::OW));
}
inline BandArgs band_args(const S2DeviceTables &t, const S2BandSide &b, int nbh, int d, int e, float scale)
{
    return {b, t.omega_rel, t.ln_omega_ref, t.omega_ref, scale, nbh, d, e};
}
inline double pair_count(const double (&p)[4], int nbh) { return nbh * (p[0] + p[1] + p[2] + p[3]); }

// Calls f with the geometry for a head dimension and a launch: owner tiles per wavefront (NO), one or two.  Two share a
// staged row, one makes twice the workgroups and needs fewer registers.  d = 16: two in the forward and dq from four workgroups
// per compute unit on (129 x 256, 32 slices: 0.43 against 0.50 and 0.53 against 0.56 ms), one in dk/dv (0.66 against 0.70; four
// were slower throughout); d = 32: two from four, d = 64: two from two workgroups per compute unit on (129 x 256: 2.8 against
// 3.3 and 5.9 against 7.5 ms per step; 64 x 128, 8 slices, d = 32: 0.41 against 0.31).
template <int D_, int NO_>
struct Shape {
    static constexpr int D = D_, NO = NO_;
};
enum Launch { kFwd, kDq, kDkdv };
template <Launch WHICH, class F>
void by_shape(const S2BandSide &b, int nbh, int dmax, F &&f)
{
    const unsigned ncu = s2_compute_units();
    const unsigned two = blocks<16, 2>(b, nbh);
    if (dmax <= 16) {
        if constexpr (WHICH != kDkdv)
            if (two >= 4 * ncu) return f(Shape<16, 2>());
        f(Shape<16, 1>());
    } else if (dmax <= 32) {
        if (two >= 4 * ncu) f(Shape<32, 2>());
        else f(Shape<32, 1>());
    } else {
        if (two >= 2 * ncu) f(Shape<64, 2>());
        else f(Shape<64, 1>());
    }
}

}  // namespace

// One instantiation (storage type, staging mode) per translation unit: BandSet<MODE> in s2_nattn_band.h.
template <int MODE>
int BandSet<MODE>::configure()
{
    return configure_one<16, 1, MODE, true>() || configure_one<16, 2, MODE, false>() || configure_one<32, 1, MODE, true>() ||
           configure_one<32, 2, MODE, true>() || configure_one<64, 1, MODE, true>() || configure_one<64, 2, MODE, true>();
}
template <int MODE>
void BandSet<MODE>::fwd(const S2DeviceTables &t, int nbh, int d, int e, float scale, const float *q, const float *k, const float *v,
                          float *out, float *lse, hipStream_t st)
{
    S2TraceScope tr("nattn_fwd_band", pair_count(t.fwd_pairs, nbh), st);
    by_shape<kFwd>(t.side_out, nbh, d > e ? d : e, [&](auto s) {
        constexpr int D = decltype(s)::D, NO = decltype(s)::NO;
        hipLaunchKernelGGL((nattn_fwd_band<D, NO, MODE>), dim3(blocks<D, NO>(t.side_out, nbh)), dim3(256),
                           (fwd_lds<D, NO>()), st, band_args(t, t.side_out, nbh, d, e, scale), q, k, v, out, lse);
    });
}
template <int MODE>
void BandSet<MODE>::dq(const S2DeviceTables &t, int nbh, int d, int e, float scale, const float *q, const float *k, const float *v,
                         const float *o, const float *lse, const float *go, float *dq, float *Dws, hipStream_t st)
{
    S2TraceScope tr("nattn_bwd_dq_band", pair_count(t.fwd_pairs, nbh), st);
    by_shape<kDq>(t.side_out, nbh, d > e ? d : e, [&](auto s) {
        constexpr int D = decltype(s)::D, NO = decltype(s)::NO;
        hipLaunchKernelGGL((nattn_bwd_dq_band<D, NO, MODE>), dim3(blocks<D, NO>(t.side_out, nbh)), dim3(256),
                           (fwd_lds<D, NO>()), st, band_args(t, t.side_out, nbh, d, e, scale), q, k, v, o, lse, go, dq, Dws);
    });
}
template <int MODE>
void BandSet<MODE>::dkdv(const S2DeviceTables &t, int nbh, int d, int e, float scale, const float *q, const float *k, const float *v,
                           const float *lse, const float *go, const float *Dws, float *dk, float *dv, hipStream_t st)
{
    S2TraceScope tr("nattn_bwd_dkdv_band", pair_count(t.bwd_pairs, nbh), st);
    by_shape<kDkdv>(t.side_in, nbh, d > e ? d : e, [&](auto s) {
        constexpr int D = decltype(s)::D, NO = decltype(s)::NO;
        hipLaunchKernelGGL((nattn_bwd_dkdv_band<D, NO, MODE>), dim3(blocks<D, NO>(t.side_in, nbh)), dim3(256),
                           (dkdv_lds<D, NO>()), st, band_args(t, t.side_in, nbh, d, e, scale), q, k, v, lse, go, Dws, dk, dv);
    });
}
