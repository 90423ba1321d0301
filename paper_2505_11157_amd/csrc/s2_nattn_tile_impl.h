// Neighborhood attention (Sec. 3.3, eq. (9)-(10); gradients App. B.4) on the bf16 matrix cores: band tiles of 16 keys x 16
// outputs, two key tiles (32 keys) per step, for d, e <= 64 (rounded up to 16, 32 or 64 channels) and any pair of grids.
// s2_nattn_walk.h describes the walk.
//
// Precision.  q, k, v and dout enter the matrix cores as they are; probabilities and dS, which multiply them, are float32
// values cut into three bf16 terms, which hold the 24 bits exactly, so that every product is the float32 one; logits, softmax,
// logsumexp, D and all accumulators are float32.  Share of `out` and dv that differ from the correctly rounded result: 1.3e-4
// and 3e-4, as on the fp32 matrix cores (with two terms 2.3e-3 both).  The third term costs 4 to 14 % (129 x 256, 32 slices,
// d = 16: 0.93 -> 1.03 ms per step, d = 64: 3.11 -> 3.23 ms); cut off bit by bit it is cheaper than rounded (1.06 ms).
//
// Operands of v_mfma_f32_16x16x32_bf16 (A: 16 x 32, lane (row n = lane & 15, g = lane >> 4) holds k = 8 g .. 8 g + 7; B the
// same with columns; C/D: lane holds rows 4 g .. 4 g + 3 of column n):
//   S^T = K Q^T      A = K[key n][channels 8 g ..]: a staged row is channel-major, as in memory, and ds_read_b64_tr_b16
//                    turns a block of 4 channels x 16 keys on its way to the registers (no scatter, no second copy);
//                    B = q of the lane's output: lane (n, g) ends with the logits of keys 4 g .. 4 g + 3 for output n;
//   O^T += V P^T     the 8 contraction indices of a lane are keys 4 g .. of the first tile and keys 4 g .. of the second, so
//                    B is the lane's own eight probabilities and A = V[channel n][those keys], two 8-byte LDS reads.
// 16 channels use the 16x16x16 instruction for the first product (four channels per lane).
// Channel rows have a pitch of 4 mod 8 words.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "s2_internal.h"
#include "s2_nattn_tile.h"
#include "s2_nattn_exact.h"
#include "s2_nattn_walk.h"

namespace {

using namespace s2walk;
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

template <int D, int NO>
struct Geo {
    static constexpr int OW = 16 * NO, SW = OW + 64;        // owners per workgroup and latitude, staged columns
    static constexpr int COLS = SW + 32;                    // + zeroed padding (a step may reach past the window)
    static constexpr int PITCH = COLS + 8;                  // bf16 values per channel row
    static constexpr int TILE = D * PITCH;                  // ... per staged tensor
    static constexpr int KC = D == 16 ? 1 : D / 32;         // first product: steps over the channels
    static_assert(PITCH % 16 == 8, "pitch");
};
// Wavefronts per SIMD the registers are held to: as many as fit without spills (the owners' registers grow with D and NO; the
// column-by-column stage of 64 channels takes 64 more).
template <int D, int NO, int MODE>
struct Occ {
    static constexpr int regs = D * NO + (MODE != kWide && D == 64 ? 64 : 0);
    static constexpr int fwd = regs <= 64 ? 4 : regs <= 128 ? 3 : 2, bwd = regs <= 48 ? 4 : regs <= 64 ? 3 : 2;
    static constexpr int dq = D <= 32 && NO <= 2 ? 4 : bwd;
};
// first-product operand of one point or one key: 8 channels per lane and step (16 channels: 4)
template <int D>
struct Chan {
    bf16x8 v[D / 32];
};
template <>
struct Chan<16> {
    bf16x4 v[1];
};

__device__ __forceinline__ float ldx(const bf16raw *p) { return __builtin_bit_cast(float, unsigned(*p) << 16); }
__device__ __forceinline__ void stx(bf16raw *p, float x) { *p = __builtin_bit_cast(bf16raw, (__bf16)x); }

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f32x4 mma(bf16x8 a, bf16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f32x4 mma(bf16x4 a, bf16x4 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4, a), __builtin_bit_cast(s16x4, b), c, 0, 0, 0);
}
__device__ __forceinline__ bf16x4 lds_tr(const __bf16 *p)
{
    typedef __attribute__((address_space(3))) s16x4 *ptr;
    return __builtin_bit_cast(bf16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((ptr)(__attribute__((address_space(3))) void *)p));
}
__device__ __forceinline__ bf16x8 join(bf16x4 a, bf16x4 b) { return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7); }

template <int D, int NO>
struct Tile {
    using G = Geo<D, NO>;
    // acc += (columns col .. col + 15 of a staged tensor, col a multiple of four) . (the lane's own point)
    static __device__ __forceinline__ f32x4 dot(const __bf16 *tile, int col, const Chan<D> &own, f32x4 acc, int n, int g)
    {
        const __bf16 *p = tile + col + 4 * (n & 3);
        if constexpr (D == 16) {
            acc = mma(lds_tr(p + (4 * g + (n >> 2)) * G::PITCH), own.v[0], acc);
        } else {
            p += (8 * g + (n >> 2)) * G::PITCH;
#pragma unroll
            for (int s = 0; s < G::KC; ++s)
                acc = mma(join(lds_tr(p + 32 * s * G::PITCH), lds_tr(p + (32 * s + 4) * G::PITCH)), own.v[s], acc);
        }
        return acc;
    }
    // acc[mt] += (channels 16 mt ..) . (the lane's eight float32 values of the columns of two tiles), smallest terms first
    static __device__ __forceinline__ void sum(const __bf16 *tile, int col, const bf16x8 (&b)[3], f32x4 (&acc)[D / 16], int n, int g)
    {
        const __bf16 *p = tile + n * G::PITCH + col + 4 * g;
        bf16x8 a[D / 16];
#pragma unroll
        for (int mt = 0; mt < D / 16; ++mt) {
            const __bf16 *q = p + 16 * mt * G::PITCH;
            a[mt] = join(*reinterpret_cast<const bf16x4 *>(q), *reinterpret_cast<const bf16x4 *>(q + 16));
        }
#pragma unroll
        for (int k = 2; k >= 0; --k)
#pragma unroll
            for (int mt = 0; mt < D / 16; ++mt) acc[mt] = mma(a[mt], b[k], acc[mt]);
    }
    // the lane's own point as first-product operand; p: channel 0 of the point (any valid address if !own)
    template <int MODE>
    static __device__ __forceinline__ void own_point(Chan<D> &f, const bf16raw *p, size_t plane, int nch, bool own, int g)
    {
        constexpr int W = D == 16 ? 4 : 8;
#pragma unroll
        for (int s = 0; s < G::KC; ++s) {
            bf16raw x[W];
#pragma unroll
            for (int i = 0; i < W; ++i) {
                const int c = 32 * s + W * g + i;
                x[i] = own && has<MODE>(c, nch) ? p[size_t(c) * plane] : bf16raw(0);
            }
#pragma unroll
            for (int i = 0; i < W; ++i) f.v[s][i] = __builtin_bit_cast(__bf16, x[i]);
        }
    }
};
// eight float32 values as three bf16 terms, cut off bit by bit (8 of the 24 each), so that the last one is exact as well
__device__ __forceinline__ void pack(const float (&x)[8], bf16x8 (&b)[3])
{
    unsigned u[3][4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float lo = x[2 * i], hi = x[2 * i + 1];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const unsigned a = __builtin_bit_cast(unsigned, lo), c = __builtin_bit_cast(unsigned, hi);
            u[k][i] = __builtin_amdgcn_perm(c, a, 0x07060302u);           // the two upper halves
            lo -= __builtin_bit_cast(float, a & 0xffff0000u);
            hi -= __builtin_bit_cast(float, c & 0xffff0000u);
        }
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) b[k] = __builtin_bit_cast(bf16x8, u32x4{u[k][0], u[k][1], u[k][2], u[k][3]});
}


// One tensor's stage in registers, and its way to LDS.
template <int D, int NO, int MODE>
struct Stage {
    using G = Geo<D, NO>;
    using Idx = StageIdx<bf16raw, D, G::SW, MODE>;
    static constexpr bool WIDE = MODE == kWide;
    static constexpr int NC = Idx::NC, NJ = D / 4;
    std::conditional_t<WIDE, uint2, unsigned> r[WIDE ? Idx::NP : NJ * NC];
    __device__ __forceinline__ void load(const BandWhere &w, const Idx &at, const bf16raw *row, int nch)
    {
        if constexpr (WIDE) {
#pragma unroll
            for (int j = 0; j < Idx::NP; ++j) r[j] = load_at<uint2>(row, at.at(j));
        } else {
            size_t step = w.plane_walk;
            asm volatile("" : "+s"(step));   // else the compiler keeps every channel's address in (spilled) scalar registers
            int c = MODE == kRagged ? imin(w.wave, nch - 1) : w.wave;
            const bf16raw *p = row + c * step;
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
#pragma unroll
                for (int i = 0; i < NC; ++i) r[j * NC + i] = load_at<bf16raw>(p, at.at(i));
                // past the last channel: that channel again (not stored); a branch around a load would make the compiler
                // wait for all loads in flight where its sides meet
                const int up = MODE == kRagged ? imin(w.wave + 4 * j + 4, nch - 1) - c : 4;
                p += up * step;
                c += up;
            }
        }
    }
    __device__ __forceinline__ void store(const BandWhere &w, __bf16 *tile, int nch) const
    {
        if constexpr (WIDE) {
#pragma unroll
            for (int j = 0; j < Idx::NP; ++j) {
                const int i = w.tid + 256 * j, c = i / Idx::P4, pc = i % Idx::P4;
                if (Idx::EVEN || i < D * Idx::P4) *reinterpret_cast<uint2 *>(tile + c * G::PITCH + 4 * pc) = r[j];
            }
        } else {
            __bf16 *p = tile + w.wave * G::PITCH + w.lane;
#pragma unroll
            for (int i = 0; i < NC; ++i) {
                if (64 * i + 64 > G::SW && w.lane + 64 * i >= G::SW) break;
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                    if (MODE != kRagged || w.wave + 4 * j < nch)
                        p[4 * j * G::PITCH + 64 * i] = __builtin_bit_cast(__bf16, bf16raw(r[j * NC + i]));
            }
        }
    }
};

// Position of a tile on the common grid (columns Xt .. Xt + 15) relative to 16 owners at Wo: b = smallest offset in the tile
// minus the arc's first offset (around the circle where the plan says so), whether the band touches it, whether it needs the
// mask.  Found anew for every tile: the owner tiles of a step follow each other here, and a position kept for each of them
// (TileRow) costs more scalar registers than it saves instructions (91 x 180, 16 slices, d = 16: 347 against 328 us per step).
struct GridTile {
    int b;
    bool touch, mask, tail;              // tail: columns past Xend inside the tile
    __device__ __forceinline__ void set(const RowPlan &p, int Xt, int Wo, int lo, int cnt, int nU)
    {
        b = Xt - Wo - lo - 15;
        tail = false;
        if (p.circle) {
            if (nU < 32) {
                b = (b + 16 * nU) % nU;
            } else {
                b = b < 0 ? b + nU : b;
                b = b < 0 ? b + nU : b;
                b = b >= nU ? b - nU : b;
                b = b >= nU ? b - nU : b;
            }
            tail = Xt + 16 > p.Xend;
            touch = b < cnt || b + 30 >= nU;                    // always for a whole circle: b < nU = cnt
            mask = tail || (cnt < nU && b + 30 >= cnt);
        } else {
            touch = b + 30 >= 0 && b < cnt;
            mask = b < 0 || b + 30 >= cnt;
        }
    }
    // keep[rr]: is column Xt + k0 + rr a neighbor of owner Wo + n
    template <int N>
    __device__ __forceinline__ void keep(bool (&keep)[N], const RowPlan &p, int Xt, int cnt, int nU, int k0, int n) const
    {
        const int uu = b + k0 - n + 15;
        if (p.circle && (tail || nU < 32)) {
            const int nvalid = p.Xend - Xt - k0;
#pragma unroll
            for (int rr = 0; rr < N; ++rr) keep[rr] = unsigned((uu + rr) % nU) < unsigned(cnt) && rr < nvalid;
        } else if (p.circle) {
#pragma unroll
            for (int rr = 0; rr < N; ++rr) {
                const int v = uu + rr;
                keep[rr] = unsigned(v >= nU ? v - nU : v) < unsigned(cnt);
            }
        } else {
#pragma unroll
            for (int rr = 0; rr < N; ++rr) keep[rr] = unsigned(uu + rr) < unsigned(cnt);
        }
    }
};

// Walks one staged row: calls f(o, col0, keep) for every step (32 walked columns from staged column col0 on) that touches
// owner tile o.  keep[0..3], keep[4..7]: are the lane's columns 4 g + 0..3 of the step's two tiles neighbors of the lane's
// owner.  On rows whose tiles follow their owners every owner tile sees the same masks (Wo + lo is the same mod 4 for all
// of them), so a step's masks are made once for all owner tiles.
template <int NO, int SW, class F>
__device__ __forceinline__ void walk_row(const BandWhere &w, const RowPlan &p, int Xst, int lo, int cnt, F &&f)
{
    if (cnt <= 0) return;
    const int nU = w.nU, a = (w.Wb + lo) & 3;
    const int x0 = p.multi ? 0 : w.Wb + lo - a - Xst, xend = p.multi ? imin(SW, p.Xend - Xst) : x0 + a + 15 + cnt;
    const int across = p.multi ? 0 : 16;
    for (int x = x0; x < xend; x += 32) {
        bool keep[8];
        const int uu = x - x0 - a + 4 * w.g - w.n;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            keep[i] = unsigned(uu + i) < unsigned(cnt);
            keep[4 + i] = unsigned(uu + 16 + i) < unsigned(cnt);
        }
#pragma unroll
        for (int o = 0; o < NO; ++o) {
            if (o >= w.no) break;
            if (p.multi) {
                const int Xt = Xst + x;
                GridTile ta, tb;
                ta.set(p, Xt, w.Wb + 16 * o, lo, cnt, nU);
                tb.set(p, Xt + 16, w.Wb + 16 * o, lo, cnt, nU);
                const bool second = x + 16 < xend;
                if (!ta.touch && !(second && tb.touch)) continue;
#pragma unroll
                for (int i = 0; i < 8; ++i) keep[i] = true;
                if (ta.mask || tb.mask || !second) {
                    bool ka[4], kb[4];
                    ta.keep(ka, p, Xt, cnt, nU, 4 * w.g, w.n);
                    tb.keep(kb, p, Xt + 16, cnt, nU, 4 * w.g, w.n);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        keep[i] = ka[i];
                        keep[4 + i] = kb[i] && second;
                    }
                }
            }
            f(o, x + across * o, keep);
        }
    }
}

// ---------------------------------------------------------------------------------------------------------------
// Forward.
template <int D, int NO, int MODE>
__global__ void __launch_bounds__(256, (Occ<D, NO, MODE>::fwd))
nattn_fwd_tile(BandArgs a, const bf16raw *__restrict__ q, const bf16raw *__restrict__ k, const bf16raw *__restrict__ v, bf16raw *__restrict__ out,
               float *__restrict__ lse)
{
    using G = Geo<D, NO>;
    using TL = Tile<D, NO>;
    extern __shared__ __attribute__((aligned(16))) __bf16 lds[];
    BandWhere w;
    w.set<G::OW>(a);
    const int nU = w.nU, n = w.n, g = w.g;
    const float c2 = a.scale * kLog2e;
    const bf16raw *qs = q + size_t(w.bh) * (MODE == kRagged ? a.d : D) * w.plane_own + w.own_at;
    const bf16raw *ks = k + size_t(w.bh) * (MODE == kRagged ? a.d : D) * w.plane_walk, *vs = v + size_t(w.bh) * (MODE == kRagged ? a.e : D) * w.plane_walk;

    Chan<D> qf[NO];
    f32x4 acc[NO][D / 16];
    float m[NO], l[NO];
#pragma unroll
    for (int o = 0; o < NO; ++o) {
        const int u = w.W0 + 16 * o + n;
        const bool own = w.active && u < nU;
        TL::template own_point<MODE>(qf[o], qs + w.c_own * (own ? u : 0), w.plane_own, a.d, own, g);
#pragma unroll
        for (int mt = 0; mt < D / 16; ++mt) acc[o][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
        m[o] = kMinRef;
        l[o] = 0.f;
    }
    Walker wk;
    Stage<D, NO, MODE> rk, rv;
    typename Stage<D, NO, MODE>::Idx at;
    at.init(w);
    bool more = wk.start<G::OW, G::SW>(a.b, w.first, w.own, a.omega_rel, w.lane, w.Wb);
    auto load = [&]() {
        const size_t row = w.walk_at(wk.r);
        const int Xs = wk.cur.Xs0 + wk.s * G::SW;
        at.set(w, Xs);
        rk.load(w, at, ks + row, a.d);
        rv.load(w, at, vs + row, a.e);
    };
    auto store = [&](int b) {
        rk.store(w, lds + b * 2 * G::TILE, a.d);
        rv.store(w, lds + b * 2 * G::TILE + G::TILE, a.e);
    };
    // two stages in LDS: while one is worked on the next is stored and the one after is on its way to the registers; one
    // barrier per stage, and a wavefront may run ahead of the slowest by one
    if (more) load();
    for (int i = w.tid; i < 2 * G::TILE; i += 256) reinterpret_cast<unsigned *>(lds)[i] = 0u;
    __syncthreads();
    if (more) store(0);
    for (int buf = 0; more; buf ^= 1) {
        const RowPlan p = wk.cur;
        const int Xst = p.Xs0 + wk.s * G::SW;
        int lo, cnt;
        wk.rows.arc(wk.r, lo, cnt);
        const float lw2 = __log2f(wk.rows.weight(wk.r));
        more = wk.next<G::OW, G::SW>(nU, w.Wb);
        if (more) load();
        __syncthreads();
        const __bf16 *Kc = lds + buf * 2 * G::TILE, *Vc = Kc + G::TILE;
        walk_row<NO, G::SW>(w, p, Xst, lo, cnt, [&](int o, int col0, const bool (&keep)[8]) {
            __builtin_amdgcn_sched_barrier(0);       // owner tiles one after the other: interleaved they take twice the registers
            const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
            const f32x4 s0 = TL::dot(Kc, col0, qf[o], zero, n, g);
            const f32x4 s1 = TL::dot(Kc, col0 + 16, qf[o], zero, n, g);
            const float s[8] = {s0[0], s0[1], s0[2], s0[3], s1[0], s1[1], s1[2], s1[3]};
            float x[8];
            // probabilities against the reference maximum so far; their sum tells whether it has to move
            auto probabilities = [&]() {
                const float bias = lw2 - m[o];
                float sum = 0.f;
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const float p = __builtin_amdgcn_exp2f(fmaf(s[i], c2, bias));
                    x[i] = keep[i] ? p : 0.f;
                    sum += x[i];
                }
                return sum;
            };
            float sum = probabilities();
            if (__any(sum > 2048.f)) {
                float mx = -INFINITY;
#pragma unroll
                for (int i = 0; i < 8; ++i) mx = keep[i] ? fmaxf(mx, fmaf(s[i], c2, lw2)) : mx;
                mx = group_max(mx);
                const float m_new = mx > m[o] + 8.f ? mx : m[o];
                const float corr = __builtin_amdgcn_exp2f(m[o] - m_new);
                m[o] = m_new;
                l[o] *= corr;
#pragma unroll
                for (int mt = 0; mt < D / 16; ++mt)
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr) acc[o][mt][rr] *= corr;
                sum = probabilities();
            }
            l[o] += sum;
            bf16x8 pb[3];
            pack(x, pb);
            TL::sum(Vc, col0, pb, acc[o], n, g);
            settle(acc[o]);
        });
        if (more) store(buf ^ 1);
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
        bf16raw *ob = out + size_t(w.bh) * (MODE == kRagged ? a.e : D) * w.plane_own + w.own_at + w.c_own * u;
#pragma unroll
        for (int mt = 0; mt < D / 16; ++mt)
#pragma unroll
            for (int rr = 0; rr < 4; ++rr)
                if (has<MODE>(16 * mt + 4 * g + rr, a.e)) stx(ob + size_t(16 * mt + 4 * g + rr) * w.plane_own, acc[o][mt][rr] * inv);
        if (g == 0)
            lse[size_t(w.bh) * w.plane_own + w.own_at + w.c_own * u] = (m[o] + log2f(lt * a.omega_ref)) * 0.6931471805599453f;
    }
    exact_fwd<bf16raw, BandPlace<G::OW>>(again, w.wave);
}

// ---------------------------------------------------------------------------------------------------------------
// Backward, query side: dq and D_i = dout_i . out_i (written for the key-side launch).
template <int D, int NO, int MODE>
__global__ void __launch_bounds__(256, (Occ<D, NO, MODE>::dq))
nattn_bwd_dq_tile(BandArgs a, const bf16raw *__restrict__ q, const bf16raw *__restrict__ k, const bf16raw *__restrict__ v,
                  const bf16raw *__restrict__ o_, const float *__restrict__ lse, const bf16raw *__restrict__ go, bf16raw *__restrict__ dq,
                  float *__restrict__ Dws)
{
    using G = Geo<D, NO>;
    using TL = Tile<D, NO>;
    extern __shared__ __attribute__((aligned(16))) __bf16 lds[];
    BandWhere w;
    w.set<G::OW>(a);
    const int nU = w.nU, n = w.n, g = w.g;
    const float c2 = a.scale * kLog2e;
    const size_t slice_q = size_t(w.bh) * (MODE == kRagged ? a.d : D) * w.plane_own + w.own_at, slice_o = size_t(w.bh) * (MODE == kRagged ? a.e : D) * w.plane_own + w.own_at;
    const bf16raw *ks = k + size_t(w.bh) * (MODE == kRagged ? a.d : D) * w.plane_walk, *vs = v + size_t(w.bh) * (MODE == kRagged ? a.e : D) * w.plane_walk;

    Chan<D> qf[NO], gf[NO];
    f32x4 acc[NO][D / 16];
    float L2[NO], Dn[NO];
#pragma unroll
    for (int o = 0; o < NO; ++o) {
#pragma unroll
        for (int mt = 0; mt < D / 16; ++mt) acc[o][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
        L2[o] = 0.f;
        Dn[o] = 0.f;
        const int u = w.W0 + 16 * o + n;
        const bool own = w.active && u < nU;
        const size_t at = w.c_own * (own ? u : 0);
        TL::template own_point<MODE>(qf[o], q + slice_q + at, w.plane_own, a.d, own, g);
        TL::template own_point<MODE>(gf[o], go + slice_o + at, w.plane_own, a.e, own, g);
        float dsum = 0.f;
#pragma unroll
        for (int i = 0; i < D / 4; ++i) {
            const int c = (D / 4) * g + i;
            const bool on = own && has<MODE>(c, a.e);
            const size_t e = at + size_t(c) * w.plane_own;
            if (on) dsum = fmaf(ldx(go + slice_o + e), ldx(o_ + slice_o + e), dsum);
        }
        dsum = group_sum(dsum);
        if (own) {
            const size_t e = size_t(w.bh) * w.plane_own + w.own_at + at;
            if (g == 0) Dws[e] = dsum;
            Dn[o] = -dsum;
            L2[o] = (lse[e] - a.ln_omega_ref) * kLog2e;
        }
    }
    Walker wk;
    Stage<D, NO, MODE> rk, rv;
    typename Stage<D, NO, MODE>::Idx at;
    at.init(w);
    bool more = wk.start<G::OW, G::SW>(a.b, w.first, w.own, a.omega_rel, w.lane, w.Wb);
    auto load = [&]() {
        const size_t row = w.walk_at(wk.r);
        const int Xs = wk.cur.Xs0 + wk.s * G::SW;
        at.set(w, Xs);
        rk.load(w, at, ks + row, a.d);
        rv.load(w, at, vs + row, a.e);
    };
    auto store = [&](int b) {
        rk.store(w, lds + b * 2 * G::TILE, a.d);
        rv.store(w, lds + b * 2 * G::TILE + G::TILE, a.e);
    };
    // two stages in LDS: while one is worked on the next is stored and the one after is on its way to the registers; one
    // barrier per stage, and a wavefront may run ahead of the slowest by one
    if (more) load();
    for (int i = w.tid; i < 2 * G::TILE; i += 256) reinterpret_cast<unsigned *>(lds)[i] = 0u;
    __syncthreads();
    if (more) store(0);
    for (int buf = 0; more; buf ^= 1) {
        const RowPlan p = wk.cur;
        const int Xst = p.Xs0 + wk.s * G::SW;
        int lo, cnt;
        wk.rows.arc(wk.r, lo, cnt);
        const float lw2 = __log2f(wk.rows.weight(wk.r));
        more = wk.next<G::OW, G::SW>(nU, w.Wb);
        if (more) load();
        __syncthreads();
        const __bf16 *Kc = lds + buf * 2 * G::TILE, *Vc = Kc + G::TILE;
        walk_row<NO, G::SW>(w, p, Xst, lo, cnt, [&](int o, int col0, const bool (&keep)[8]) {
            __builtin_amdgcn_sched_barrier(0);       // owner tiles one after the other: interleaved they take twice the registers
            const float bias = lw2 - L2[o], Dw = Dn[o];
            const f32x4 zero = {0.f, 0.f, 0.f, 0.f}, d0 = {Dw, Dw, Dw, Dw};
            const f32x4 s0 = TL::dot(Kc, col0, qf[o], zero, n, g), e0 = TL::dot(Vc, col0, gf[o], d0, n, g);
            const f32x4 s1 = TL::dot(Kc, col0 + 16, qf[o], zero, n, g);
            const f32x4 e1 = TL::dot(Vc, col0 + 16, gf[o], d0, n, g);
            float ds[8];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float x = __builtin_amdgcn_exp2f(fmaf(s0[i], c2, bias)) * e0[i];
                ds[i] = keep[i] ? x : 0.f;
                const float y = __builtin_amdgcn_exp2f(fmaf(s1[i], c2, bias)) * e1[i];
                ds[4 + i] = keep[4 + i] ? y : 0.f;
            }
            bf16x8 db[3];
            pack(ds, db);
            TL::sum(Kc, col0, db, acc[o], n, g);
            settle(acc[o]);
        });
        if (more) store(buf ^ 1);
    }
    if (!w.active) return;
    unsigned again[NO];                  // owners whose sums took in a non-finite value (s2_nattn_exact.h)
#pragma unroll
    for (int o = 0; o < NO; ++o) {
        const int u = w.W0 + 16 * o + n;
        again[o] = not_finite(acc[o], u < nU);
        if (u >= nU || (again[o] >> n & 1)) continue;
        bf16raw *ob = dq + slice_q + w.c_own * u;
#pragma unroll
        for (int mt = 0; mt < D / 16; ++mt)
#pragma unroll
            for (int rr = 0; rr < 4; ++rr)
                if (has<MODE>(16 * mt + 4 * g + rr, a.d)) stx(ob + size_t(16 * mt + 4 * g + rr) * w.plane_own, acc[o][mt][rr] * a.scale);
    }
    exact_dq<bf16raw, BandPlace<G::OW>>(again, w.wave);
}

// ---------------------------------------------------------------------------------------------------------------
// Backward, key side: owners are input points, the transposed band gives the output latitudes; q, dout, lse and D
// of a stage's outputs are staged together.
template <int D, int NO, int MODE>
__global__ void __launch_bounds__(256, (Occ<D, NO, MODE>::bwd))
nattn_bwd_dkdv_tile(BandArgs a, const bf16raw *__restrict__ q, const bf16raw *__restrict__ k, const bf16raw *__restrict__ v,
                    const float *__restrict__ lse, const bf16raw *__restrict__ go, const float *__restrict__ Dws,
                    bf16raw *__restrict__ dk, bf16raw *__restrict__ dv)
{
    using G = Geo<D, NO>;
    using TL = Tile<D, NO>;
    extern __shared__ __attribute__((aligned(16))) __bf16 lds[];
    float *Ls = reinterpret_cast<float *>(lds + 4 * G::TILE);        // per stage: -L, then -D
    BandWhere w;
    w.set<G::OW>(a);
    const int nU = w.nU, n = w.n, g = w.g;
    const float c2 = a.scale * kLog2e, lref = a.ln_omega_ref;
    const size_t slice_k = size_t(w.bh) * (MODE == kRagged ? a.d : D) * w.plane_own + w.own_at, slice_v = size_t(w.bh) * (MODE == kRagged ? a.e : D) * w.plane_own + w.own_at;
    const bf16raw *qs = q + size_t(w.bh) * (MODE == kRagged ? a.d : D) * w.plane_walk, *gs = go + size_t(w.bh) * (MODE == kRagged ? a.e : D) * w.plane_walk;
    const float *ls = lse + size_t(w.bh) * w.plane_walk, *Ds = Dws + size_t(w.bh) * w.plane_walk;
    // the quadrature weight is the owner's own here: it multiplies the finished sums (a latitude of weight zero has no arcs)
    const float omega = w.active ? a.omega_rel[w.own / w.c_own] : 0.f;

    Chan<D> kf[NO], vf[NO];
    f32x4 adk[NO][D / 16], adv[NO][D / 16];
#pragma unroll
    for (int o = 0; o < NO; ++o) {
        const int u = w.W0 + 16 * o + n;
        const bool own = w.active && u < nU;
        const size_t at = w.c_own * (own ? u : 0);
#pragma unroll
        for (int mt = 0; mt < D / 16; ++mt) adk[o][mt] = adv[o][mt] = f32x4{0.f, 0.f, 0.f, 0.f};
        TL::template own_point<MODE>(kf[o], k + slice_k + at, w.plane_own, a.d, own, g);
        TL::template own_point<MODE>(vf[o], v + slice_v + at, w.plane_own, a.e, own, g);
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
    Stage<D, NO, MODE> rq, rg;
    typename Stage<D, NO, MODE>::Idx at;
    at.init(w);
    bool more = wk.start<G::OW, G::SW>(a.b, w.first, w.own, nullptr, w.lane, w.Wb);
    auto load = [&]() {
        const size_t row = w.walk_at(wk.r);
        const int Xs = wk.cur.Xs0 + wk.s * G::SW;
        at.set(w, Xs);
        rq.load(w, at, qs + row, a.d);
        rg.load(w, at, gs + row, a.e);
        load_stat(row, Xs);
    };
    auto store = [&](int b) {
        rq.store(w, lds + b * 2 * G::TILE, a.d);
        rg.store(w, lds + b * 2 * G::TILE + G::TILE, a.e);
        if (w.tid < G::SW) {
            Ls[b * 2 * G::COLS + w.tid] = (lref - rl) * kLog2e;
            Ls[b * 2 * G::COLS + G::COLS + w.tid] = -rd;
        }
    };
    // two stages in LDS: while one is worked on the next is stored and the one after is on its way to the registers; one
    // barrier per stage, and a wavefront may run ahead of the slowest by one
    if (more) load();
    for (int i = w.tid; i < 2 * G::TILE + 4 * G::COLS; i += 256) reinterpret_cast<unsigned *>(lds)[i] = 0u;
    __syncthreads();
    if (more) store(0);
    for (int buf = 0; more; buf ^= 1) {
        const RowPlan p = wk.cur;
        const int Xst = p.Xs0 + wk.s * G::SW;
        int lo, cnt;
        wk.rows.arc(wk.r, lo, cnt);
        more = wk.next<G::OW, G::SW>(nU, w.Wb);
        if (more) load();
        __syncthreads();
        const __bf16 *Qc = lds + buf * 2 * G::TILE, *Gc = Qc + G::TILE;
        const float *Ls_ = Ls + buf * 2 * G::COLS, *Dn_ = Ls_ + G::COLS;
        walk_row<NO, G::SW>(w, p, Xst, lo, cnt, [&](int o, int col0, const bool (&keep)[8]) {
            __builtin_amdgcn_sched_barrier(0);       // owner tiles one after the other: interleaved they take twice the registers
            const float *Lp = Ls_ + col0 + 4 * g, *Dp = Dn_ + col0 + 4 * g;
            const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
            const f32x4 L0 = *reinterpret_cast<const f32x4 *>(Lp), L1 = *reinterpret_cast<const f32x4 *>(Lp + 16);
            const f32x4 s0 = TL::dot(Qc, col0, kf[o], zero, n, g);
            const f32x4 e0 = TL::dot(Gc, col0, vf[o], *reinterpret_cast<const f32x4 *>(Dp), n, g);
            const f32x4 s1 = TL::dot(Qc, col0 + 16, kf[o], zero, n, g);
            const f32x4 e1 = TL::dot(Gc, col0 + 16, vf[o], *reinterpret_cast<const f32x4 *>(Dp + 16), n, g);
            float pr[8], ds[8];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float x = __builtin_amdgcn_exp2f(fmaf(s0[i], c2, L0[i]));
                pr[i] = keep[i] ? x : 0.f;
                ds[i] = pr[i] * e0[i];
                const float y = __builtin_amdgcn_exp2f(fmaf(s1[i], c2, L1[i]));
                pr[4 + i] = keep[4 + i] ? y : 0.f;
                ds[4 + i] = pr[4 + i] * e1[i];
            }
            bf16x8 pb[3];
            pack(pr, pb);
            TL::sum(Gc, col0, pb, adv[o], n, g);
            pack(ds, pb);
            TL::sum(Qc, col0, pb, adk[o], n, g);
            settle(adv[o]);
            settle(adk[o]);
        });
        if (more) store(buf ^ 1);
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
                if (has<MODE>(c, a.d)) stx(dk + slice_k + at, adk[o][mt][rr] * (omega * a.scale));
                if (has<MODE>(c, a.e)) stx(dv + slice_v + at, adv[o][mt][rr] * omega);
            }
    }
    exact_dkdv<bf16raw, BandPlace<G::OW>>(again, w.wave);
}

template <int D, int NO>
constexpr size_t fwd_lds() { return size_t(4) * Geo<D, NO>::TILE * sizeof(__bf16); }
template <int D, int NO>
constexpr size_t dkdv_lds() { return fwd_lds<D, NO>() + 4 * Geo<D, NO>::COLS * sizeof(float); }

inline int raise_lds(const void *f, size_t bytes)
{
    return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes)) != hipSuccess;
}
template <int D, int NO, int MODE, bool BWD>
int configure_one()
{
    int rc = 0;
    if constexpr (BWD)
        rc = raise_lds(reinterpret_cast<const void *>(nattn_bwd_dq_tile<D, NO, MODE>), fwd_lds<D, NO>()) ||
             raise_lds(reinterpret_cast<const void *>(nattn_bwd_dkdv_tile<D, NO, MODE>), dkdv_lds<D, NO>());
    return rc || raise_lds(reinterpret_cast<const void *>(nattn_fwd_tile<D, NO, MODE>), fwd_lds<D, NO>());
}

template <int NO>
unsigned blocks(const S2BandSide &b, int nbh)
{
    return unsigned(long((b.n_own + 3) / 4) * nbh * ((b.nU + 16 * NO - 1) / (16 * NO)));
}
inline BandArgs band_args(const S2DeviceTables &t, const S2BandSide &b, int nbh, int d, int e, float scale)
{
    return {b, t.omega_rel, t.ln_omega_ref, t.omega_ref, scale, nbh, d, e};
}
inline double pair_count(const double (&p)[4], int nbh) { return nbh * (p[0] + p[1] + p[2] + p[3]); }

// Calls f with the geometry for a head dimension and a launch: owner tiles per wavefront (NO).  More of them share a staged
// row and its masks, fewer make more workgroups.  Measured on seven grids with 6 to 32 slices: four from eight workgroups per
// compute unit on (129 x 256, 32 slices, d = 16: 0.95 against 1.04 ms per step; 91 x 180, 16 slices: 0.32 against 0.31), two
// from three per compute unit on (91 x 181, 8 slices, d = 32: 0.24 against 0.28; 64 x 128, 8 slices: 0.24 against 0.21).  The
// backward keeps 32 channels at two (0.86 against 0.90 ms on 161 x 320 with 18 slices).  64 channels: two from two per compute
// unit on (64 x 128, 8 slices: 302 against 341 us per step; 91 x 181, 4 slices: 319 against 383), else one (64 x 128, 4 slices:
// 208 against 282; 91 x 180, 2 slices: 205 against 264; 46 x 90, 4 slices: 156 against 180).
template <int D_, int NO_>
struct Shape {
    static constexpr int D = D_, NO = NO_;
};
template <bool BWD, class F>
void by_shape(const S2BandSide &b, int nbh, int dmax, F &&f)
{
    const unsigned ncu = s2_compute_units();
    const bool two = blocks<2>(b, nbh) >= 3 * ncu, four = blocks<4>(b, nbh) >= 8 * ncu;
    if (dmax <= 16) {
        if (four) f(Shape<16, 4>());
        else if (two) f(Shape<16, 2>());
        else f(Shape<16, 1>());
    } else if (dmax <= 32) {
        if constexpr (!BWD)
            if (four) return f(Shape<32, 4>());
        if (two) f(Shape<32, 2>());
        else f(Shape<32, 1>());
    } else {
        if (blocks<2>(b, nbh) >= 2 * ncu) f(Shape<64, 2>());
        else f(Shape<64, 1>());
    }
}

}  // namespace

// One instantiation (storage type, staging mode) per translation unit: TileSet<MODE> in s2_nattn_tile.h.
template <int MODE>
int TileSet<MODE>::configure()
{
    return configure_one<16, 1, MODE, true>() || configure_one<16, 2, MODE, true>() || configure_one<16, 4, MODE, true>() ||
           configure_one<32, 1, MODE, true>() || configure_one<32, 2, MODE, true>() || configure_one<32, 4, MODE, false>() ||
           configure_one<64, 1, MODE, true>() || configure_one<64, 2, MODE, true>();
}
template <int MODE>
void TileSet<MODE>::fwd(const S2DeviceTables &t, int nbh, int d, int e, float scale, const bf16raw *q, const bf16raw *k, const bf16raw *v,
                           bf16raw *out, float *lse, hipStream_t st)
{
    S2TraceScope tr("nattn_fwd_tile", pair_count(t.fwd_pairs, nbh), st);
    by_shape<false>(t.side_out, nbh, d > e ? d : e, [&](auto s) {
        constexpr int D = decltype(s)::D, NO = decltype(s)::NO;
        hipLaunchKernelGGL((nattn_fwd_tile<D, NO, MODE>), dim3(blocks<NO>(t.side_out, nbh)), dim3(256), (fwd_lds<D, NO>()), st,
                           band_args(t, t.side_out, nbh, d, e, scale), q, k, v, out, lse);
    });
}
template <int MODE>
void TileSet<MODE>::dq(const S2DeviceTables &t, int nbh, int d, int e, float scale, const bf16raw *q, const bf16raw *k, const bf16raw *v,
                          const bf16raw *o, const float *lse, const bf16raw *go, bf16raw *dq, float *Dws, hipStream_t st)
{
    S2TraceScope tr("nattn_bwd_dq_tile", pair_count(t.fwd_pairs, nbh), st);
    by_shape<true>(t.side_out, nbh, d > e ? d : e, [&](auto s) {
        constexpr int D = decltype(s)::D, NO = decltype(s)::NO;
        hipLaunchKernelGGL((nattn_bwd_dq_tile<D, NO, MODE>), dim3(blocks<NO>(t.side_out, nbh)), dim3(256), (fwd_lds<D, NO>()), st,
                           band_args(t, t.side_out, nbh, d, e, scale), q, k, v, o, lse, go, dq, Dws);
    });
}
template <int MODE>
void TileSet<MODE>::dkdv(const S2DeviceTables &t, int nbh, int d, int e, float scale, const bf16raw *q, const bf16raw *k, const bf16raw *v,
                            const float *lse, const bf16raw *go, const float *Dws, bf16raw *dk, bf16raw *dv, hipStream_t st)
{
    S2TraceScope tr("nattn_bwd_dkdv_tile", pair_count(t.bwd_pairs, nbh), st);
    by_shape<true>(t.side_in, nbh, d > e ? d : e, [&](auto s) {
        constexpr int D = decltype(s)::D, NO = decltype(s)::NO;
        hipLaunchKernelGGL((nattn_bwd_dkdv_tile<D, NO, MODE>), dim3(blocks<NO>(t.side_in, nbh)), dim3(256), (dkdv_lds<D, NO>()), st,
                           band_args(t, t.side_in, nbh, d, e, scale), q, k, v, lse, go, Dws, dk, dv);
    });
}
