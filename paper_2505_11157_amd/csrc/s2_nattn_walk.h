// How the tile kernels of the neighborhood attention walk a neighborhood (device side, shared by the float32 and the
// bf16 matrix-core kernels).
//
// Both directions and all grid ratios are one problem (S2BandSide): owners (the points a wavefront accumulates for) and
// walked points lie on grids of the same longitude count nU.  Equal grids are that already; where one grid has r times
// the longitudes of the other, its latitude is cut into r interleaved classes s (longitudes r u + s, u < nU), each of
// them a row of its own.  On walked row r the neighbors of owner u are the columns u + lo .. u + lo + cnt - 1 around the
// circle of nU.
//
// A workgroup of four wavefronts owns OW consecutive columns of FOUR consecutive owner rows, one row per wavefront, and
// walks the union of the four bands row by row in stages of SW = OW + 64 columns held in LDS:
//   * rows whose arcs all fit (union of at most kSpan offsets) are ONE stage that holds the window of all owners; every
//     16-owner tile walks its own key tiles from the first column of its band rounded down to a multiple of four;
//   * rows with longer arcs or whole circles are walked in stages on a common 16-column grid: over the linear window
//     while that is shorter than the circle, else over the circle itself, every column once, with distances taken
//     around the circle.
// For 16 owners the walked columns of one row form a band of the 16 x 16 score tiles: a tile the band does not touch is
// skipped (wavefront-uniform), a tile it cuts gets a per-element mask, a tile inside it none.
#pragma once
#include <hip/hip_runtime.h>

#include "s2_internal.h"
#include "s2_nattn_band.h"

namespace s2walk {

constexpr int kSpan = 57;            // widest union of arcs that is served by a single stage

typedef float f32x4 __attribute__((ext_vector_type(4)));
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kMinRef = -1e30f;    // start value of the reference maximum: finite, so that x - m needs no guard (exp2(-inf) = 0)

__device__ __forceinline__ float group_max(float x)     // over the four lanes (g = 0..3) of a point
{
    x = fmaxf(x, __shfl_xor(x, 16));
    return fmaxf(x, __shfl_xor(x, 32));
}
__device__ __forceinline__ float group_sum(float x)
{
    x += __shfl_xor(x, 16);
    return x + __shfl_xor(x, 32);
}
// Matrix results that a branch may lead to a reader of: the compiler pads the wait states of an instruction on one side of
// a branch only.  Ten wait states here, after the last instruction of the tile.
template <int N>
__device__ __forceinline__ void settle(f32x4 (&a)[N])
{
#pragma unroll
    for (int i = 0; i + 1 < N; ++i) asm volatile("" : "+v"(a[i]));
    asm volatile("s_nop 9" : "+v"(a[N - 1]));
}

__device__ __forceinline__ int imin(int a, int b) { return a < b ? a : b; }
__device__ __forceinline__ int imax(int a, int b) { return a > b ? a : b; }

// x mod n for 0 <= x < 2^22: the float32 quotient is off by at most one
__device__ __forceinline__ int wrap_col(int x, int n, float inv_n)
{
    const int r = x - int(float(x) * inv_n) * n;
    return r < 0 ? r + n : r >= n ? r - n : r;
}

// (Xs + col) mod n, Xs uniform and below 4 n (2^22), 0 <= col < width
__device__ __forceinline__ int wrap_stage(int Xs, int col, int width, int n, float inv_n)
{
    if (n < width) return wrap_col(Xs + col, n, inv_n);
    int x = Xs >= 2 * n ? Xs - 2 * n : Xs;
    x = (x >= n ? x - n : x) + col;
    return x >= n ? x - n : x;
}

// polar segments (the heaviest) first, from both ends
__device__ __forceinline__ int segment_of(int sk, int nseg) { return (sk & 1) ? nseg - 1 - (sk >> 1) : (sk >> 1); }

// Rows a workgroup has to stage and their metadata, read from the grid tables once and kept one row per lane in two sets of
// registers (a table read inside the row loop would be a vector load whose wait also waits for the prefetch in flight):
// at most kMaxRows rows, longitude counts below 2^15.
constexpr int kMaxRows = 128;
struct BandRows {
    int rmin, rmax;          // of the whole union
    int arc_v[2];            // row rmin + 64 s + lane: own arc, first offset (low half) and number of offsets
    int uni_v[2];            // ... first and last offset over the four owner rows (last < first: no arc; 0x7fff: the circle)
    float omega_v[2];        // ... the row's relative quadrature weight (1 where the owners carry the weight)

    __device__ __forceinline__ void load(const S2BandSide &b, int first, int own, const float *omega_rel, int lane)
    {
        rmin = 1 << 30;
        rmax = -1;
        for (int w = 0; w < 4; ++w) {
            if (first + w >= b.n_own) break;
            const int lo = b.blo[first + w], n = b.bn[first + w];
            if (n > 0) {
                rmin = imin(rmin, lo);
                rmax = imax(rmax, lo + n - 1);
            }
        }
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            const int r = rmin + 64 * s + lane;
            int wlo = 0x7ffe, whi = -0x7fff;
            arc_v[s] = 0;
            omega_v[s] = 1.f;
            if (64 * s <= rmax - rmin) {
                for (int w = 0; w < 4; ++w) {
                    const int vl = first + w;
                    if (vl >= b.n_own) break;
                    const int i = r - b.blo[vl];
                    if (r <= rmax && i >= 0 && i < b.bn[vl]) {
                        const int2 a = b.arc[vl * b.bmax + i];
                        if (a.y > 0) {
                            wlo = imin(wlo, a.x);
                            whi = imax(whi, a.y >= b.nU ? 0x7fff : a.x + a.y - 1);
                            if (vl == own) arc_v[s] = (a.x & 0xffff) | a.y << 16;
                        }
                    }
                }
                if (omega_rel && r <= rmax) omega_v[s] = omega_rel[r / b.c_walk];
            }
            uni_v[s] = (wlo & 0xffff) | whi << 16;
        }
    }
    __device__ __forceinline__ int pick(const int (&v)[2], int r) const
    {
        const int i = r - rmin, x = __builtin_amdgcn_readlane(v[0], i & 63), y = __builtin_amdgcn_readlane(v[1], i & 63);
        return i < 64 ? x : y;
    }
    __device__ __forceinline__ void arc(int r, int &lo, int &cnt) const
    {
        const int a = pick(arc_v, r);
        lo = int(short(a & 0xffff));
        cnt = a >> 16;
    }
    __device__ __forceinline__ float weight(int r) const
    {
        const int v[2] = {__builtin_bit_cast(int, omega_v[0]), __builtin_bit_cast(int, omega_v[1])};
        return __builtin_bit_cast(float, pick(v, r));
    }
};

// How one row is walked: first staged (unwrapped) column, end of the columns that count, number of stages, and whether
// key tiles lie on the common grid (multi) and distances are taken around the circle (circle).  Unwrapped columns carry
// an offset of nU, so that they stay non-negative; the owners sit at nU + W0 ... = Wb ....
struct RowPlan {
    int Xs0, Xend, nst;
    bool multi, circle;
    template <int OW, int SW>
    __device__ __forceinline__ void set(const BandRows &rows, int r, int nU, int Wb)
    {
        const int u = rows.pick(rows.uni_v, r), wlo = int(short(u & 0xffff)), whi = u >> 16;
        const bool full = whi == 0x7fff;
        const int width = whi - wlo + 1;
        if (width <= 0) {                    // no owner meets this row
            multi = circle = false;
            Xs0 = Xend = nst = 0;
        } else if (!full && width <= kSpan) {
            multi = circle = false;
            Xs0 = (Wb + wlo) & ~3;
            Xend = Xs0 + SW + 32;
            nst = 1;
        } else {
            multi = true;
            circle = full || OW + width + 31 >= nU;
            Xs0 = circle ? nU : (Wb + wlo) & ~15;
            Xend = circle ? 2 * nU : Wb + OW + whi;
            nst = (Xend - Xs0 + SW - 1) / SW;
        }
    }
};

// The stages of a workgroup in order.
struct Walker {
    BandRows rows;
    RowPlan cur;
    int r, s;                            // current row and its current stage
    template <int OW, int SW>
    __device__ __forceinline__ bool settle(int nU, int Wb)
    {
        for (; r <= rows.rmax; ++r) {
            cur.template set<OW, SW>(rows, r, nU, Wb);
            if (cur.nst > 0) return true;
        }
        return false;
    }
    template <int OW, int SW>
    __device__ __forceinline__ bool start(const S2BandSide &b, int first, int own, const float *omega_rel, int lane, int Wb)
    {
        rows.load(b, first, own, omega_rel, lane);
        s = 0;
        r = rows.rmin;
        return settle<OW, SW>(b.nU, Wb);
    }
    template <int OW, int SW>
    __device__ __forceinline__ bool next(int nU, int Wb)
    {
        if (++s < cur.nst) return true;
        s = 0;
        ++r;
        return settle<OW, SW>(nU, Wb);
    }
};

// The key tiles (16 columns from Xt on) of one row as 16 owners at Wo see them, one after the other.
// KIND: rows whose tiles follow their owners (kOwnTiles), rows on the common grid (kGridTiles), or either (kAnyTiles: one
// copy of the tile loop for both, for kernels that have no registers left for two).
// v = (offset of the tile's first column to the last owner) - (the arc's first offset) + 30: the tile's 16 x 16 offsets, counted
// from the arc's first, are v - 30 .. v.  Around the circle v is kept in 0 .. nU - 1 (an offset below zero is then one turn more).
// v moves from tile to tile instead of being found anew from Xt (16 wavefront-uniform instructions, one after the other): together
// with reads ahead of the products, on the fp32 matrix cores, 181 x 360, 2 slices, d = 32: 0.56 -> 0.51 ms per step.
enum { kOwnTiles, kGridTiles, kAnyTiles };
template <int KIND>
__device__ __forceinline__ bool on_grid(const RowPlan &p) { return KIND == kAnyTiles ? p.multi : KIND == kGridTiles; }
template <int KIND>
struct TileRow {
    int v, cnt, nU;
    int step, lim, turn;                 // to the next tile; v wraps at lim; what an offset below zero lacks to its place on the circle
    int low, top;                        // a tile with v in low .. top - 1 lies inside the band
    int tail;                            // a tile from past this column on has columns past the row
    __device__ __forceinline__ void start(const RowPlan &p, int Xt, int Wo, int lo, int count, int n)
    {
        v = Xt - Wo - lo + 15;
        cnt = count;
        nU = n;
        step = 16;
        low = 30;
        top = cnt;
        if (KIND == kOwnTiles) return;
        lim = tail = 0x7fffffff;
        turn = 0;
        if (p.circle) {
            if (nU < 32) {
                v = (v + 16 * nU) % nU;
                step = 16 % nU;
            } else {
                v = v < 0 ? v + nU : v;
                v = v < 0 ? v + nU : v;
                v = v >= nU ? v - nU : v;
                v = v >= nU ? v - nU : v;
            }
            lim = turn = nU;
            tail = p.Xend - 16;
            low = cnt >= nU ? 0 : low;
            top = cnt >= nU ? 0x7fffffff : top;
        }
    }
    __device__ __forceinline__ void next()
    {
        v += step;
        if (KIND != kOwnTiles) v = v >= lim ? v - nU : v;
    }
    // does the band touch the tile (rows of own tiles start and end with the band)
    __device__ __forceinline__ bool touch() const { return KIND == kOwnTiles || unsigned(v) < unsigned(cnt + 30); }
    // does a part of the tile lie outside the band
    __device__ __forceinline__ bool mask(int Xt) const
    {
        return v < low || v >= top || (KIND != kOwnTiles && Xt > tail);
    }
    // keep[rr]: is column Xt + k0 + rr a neighbor of owner Wo + n
    template <int N>
    __device__ __forceinline__ void keep(bool (&keep)[N], int Xt, int k0, int n) const
    {
        const int x = v - 15 + k0 - n;
        if (KIND != kOwnTiles && (Xt > tail || (turn > 0 && nU < 32))) {
            int rest = tail + 16 - Xt;
            asm volatile("" : "+s"(rest));   // found here, not kept in step with Xt in a register of its own
            const int nvalid = rest - k0;
#pragma unroll
            for (int rr = 0; rr < N; ++rr) keep[rr] = unsigned((x + rr + 32 * nU) % nU) < unsigned(cnt) && rr < nvalid;
        } else {
#pragma unroll
            for (int rr = 0; rr < N; ++rr) {
                const int y = x + rr;
                keep[rr] = unsigned(KIND != kOwnTiles && y < 0 ? y + turn : y) < unsigned(cnt);
            }
        }
    }
};

// ---- kernel arguments and the place of a workgroup ----
struct BandArgs {
    S2BandSide b;
    const float *omega_rel;
    float ln_omega_ref, omega_ref, scale;
    int nbh, d, e;
    // patch kernels (S2BandSide::Patches)
    const int4 *seg, *row_rec;
    const int2 *patch;
    int npatch;
};

// Where a wavefront's owners and the walked rows lie.
struct BandWhere {
    int nU, W0, Wb, grp, bh, first, own, lane, wave, n, g, tid;
    int no;                        // owner tiles of this workgroup that hold a point
    bool active;
    float inv_nU;
    size_t plane_own, plane_walk;
    size_t own_at;                 // offset of owner column 0 of the wavefront's row inside a plane
    int nlon_walk, c_own, c_walk;
    template <int OW>
    __device__ __forceinline__ void set(const BandArgs &a, int thread = threadIdx.x)
    {
        nU = a.b.nU;
        const int ngrp = (nU + OW - 1) / OW, nseg = (a.b.n_own + 3) >> 2;
        int id = blockIdx.x;
        grp = id % ngrp; id /= ngrp;
        bh = id % a.nbh;
        first = 4 * segment_of(id / a.nbh, nseg);
        tid = thread; lane = tid & 63; wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        n = lane & 15; g = lane >> 4;
        own = first + wave;
        active = own < a.b.n_own;
        W0 = grp * OW; Wb = nU + W0;
        no = (imin(OW, nU - W0) + 15) >> 4;
        inv_nU = 1.f / float(nU);
        c_own = a.b.c_own; c_walk = a.b.c_walk;
        nlon_walk = nU * c_walk;
        plane_own = size_t(a.b.nlat_own) * nU * c_own;
        plane_walk = size_t(a.b.nlat_walk) * nlon_walk;
        const int lat = own / c_own;
        own_at = size_t(lat) * nU * c_own + (own - lat * c_own);
    }
    // offset of column 0 of walked row r inside a plane
    __device__ __forceinline__ size_t walk_at(int r) const
    {
        if (c_walk == 1) return size_t(r) * nlon_walk;
        const int lat = r / c_walk;
        return size_t(lat) * nlon_walk + (r - lat * c_walk);
    }
};

// is channel c one of the tensor's nch
template <int MODE>
__device__ __forceinline__ bool has(int c, int nch) { return MODE != kRagged || c < nch; }

// Where a thread's pieces of a stage lie: byte offsets into the walked tensor's row, for all stages and both tensors.
// kWide: pieces of four columns, dealt out to the threads channel by channel (past the last channel: that channel again, not
// stored).  Otherwise a wavefront takes 64 columns of one channel at a time.
template <class T, int D, int SW, int MODE>
struct StageIdx {
    static constexpr bool WIDE = MODE == kWide;
    static constexpr int P4 = SW / 4, NP = (D * P4 + 255) / 256, NC = (SW + 63) / 64, N = WIDE ? NP : NC;
    static constexpr bool EVEN = D * P4 % 256 == 0;
    // pieces of a thread repeat their columns every PER (the channel moves on by 256 PER / P4): only PER of them are kept
    static constexpr int gcd(int a, int b) { return b ? gcd(b, a % b) : a; }
    static constexpr int ROUND = P4 / gcd(P4, 256), PER = WIDE && EVEN && ROUND < N ? ROUND : N;
    unsigned base[PER], turn[PER], off[PER];         // channel, column reduced to one turn, sum of both for the current stage
    unsigned up;                                     // from a piece to the one PER pieces later
    __device__ __forceinline__ void init(const BandWhere &w)
    {
        up = WIDE ? unsigned(256 * PER / P4) * unsigned(w.plane_walk) * unsigned(sizeof(T)) : 0u;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            int col;
            if constexpr (WIDE) {
                const int i = w.tid + 256 * j, c = imin(i / P4, D - 1);
                base[j] = unsigned(c) * unsigned(w.plane_walk) * unsigned(sizeof(T));
                col = 4 * (i % P4);
            } else {
                col = w.lane + 64 * j < SW ? w.lane + 64 * j : 0;
                base[j] = 0;
            }
            turn[j] = wrap_col(col, w.nU, w.inv_nU);
        }
    }
    __device__ __forceinline__ void set(const BandWhere &w, int Xs)
    {
        int Xr = Xs >= 2 * w.nU ? Xs - 2 * w.nU : Xs;
        Xr = Xr >= w.nU ? Xr - w.nU : Xr;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const unsigned x = unsigned(Xr) + turn[j], y = x - unsigned(w.nU);       // y wraps to a large value if x < nU
            off[j] = base[j] + (x < y ? x : y) * unsigned(WIDE ? sizeof(T) : sizeof(T) * w.c_walk);
        }
    }
    __device__ __forceinline__ unsigned at(int j) const { return off[j % PER] + unsigned(j / PER) * up; }
};
template <class V>
__device__ __forceinline__ V load_at(const void *row, unsigned off)
{
    return *reinterpret_cast<const V *>(static_cast<const char *>(row) + off);
}

}  // namespace s2walk
