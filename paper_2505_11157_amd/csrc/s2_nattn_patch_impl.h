// Neighborhood attention (Sec. 3.3, eq. (9)-(10); gradients App. B.4) of float32 and bf16 tensors on the bf16 matrix cores, for any
// pair of grids and d, e <= 64 (rounded up to 16, 32 or 64 channels).
//
// Precision.  A float32 value is the sum of three bf16 terms x0 + x1 + x2 of 8 bits each, every one the rounded rest of those
// before, exactly down to 2^-110 (s2_bf16_terms.h).  A product takes the six of nine term products that are not below 2^-26 of it, smallest first;
// sums over keys keep x0 y0 and the other five in accumulators of their own, so that a long sum takes one rounding per 32 keys at
// its own magnitude (v_mfma_f32_16x16x32_bf16 adds its 32 products with less loss than 32 multiply-adds).  Dot products of 32
// and sums over 256 unit-variance values, rms error: multiply-adds and the fp32 matrix cores 1.0e-7 and 2.9e-7 of the result's rms,
// here 3.8e-8 and 9.0e-8 (cut off bit by bit instead of rounded: 7.1e-8, with a bias).  Six bf16 instructions of 32 channels take 96
// cycles where eight fp32 ones (16x16x4) take 262.  Results of the three kernels on 14 grid pairs are 1.5 to 2.8 times closer to
// float64 than those of the kernels that these replaced.
//
// Work.  A wavefront owns 16 points in a patch of 4 x 4, 2 x 8 or 1 x 16 rows x columns (per segment of owner rows, counted on the
// host: s2_grid.cpp), a workgroup four such patches side by side.  Near the equator a square patch meets 32 chunks of four
// columns where 16 points of one row meet 72; near the poles, where arcs are long, a row is as good.  The columns that any owner of
// a workgroup meets are cut into chunks of four, numbered row by row (S2PatchRow), and staged CAP at a time.  Of each stage a
// wavefront lists the chunks its own points meet, four of which are a tile of 16 keys, whatever rows they lie on; masks are per
// element, from the arc of the owner's row.  Owner rows have the smaller longitude count nU of the two grids: classes of a finer
// owner grid are rows of their own (S2BandSide).  Walked rows are whole latitudes, of step columns per owner column: with rows of one
// class of a finer walked grid, a chunk was four loads of every second column (257 x 512 -> 129 x 256, 8 slices, d = 32: forward
// 0.329, dq 0.347 ms, now 0.175 and 0.197; the mirror image's dk/dv 0.397, now 0.258).  Where a latitude's classes make no single
// arc, or 16 bits do not hold its columns, the rows stay classes (step 1).
//
// Columns (kColumns).  A chunk begins at a fixed column, so that the order of a point's sums depends on where its column lies.  The
// float32 forward of d = e = 32 on upsampling grids has results that roll with its inputs bit for bit; there a wavefront owns 16 rows
// of one column, those of a workgroup lie four columns apart, chunks begin at columns counted from the owner's, and stages hold whole
// rows, or pieces of long rows, of all four (S2ColumnRow): every owner meets its tiles in the same order.  129 x 256 -> 257 x 512, 8 slices:
// vector kernels 514 us, by columns 341 (10 tiles in 5.0 stages a wavefront; patches 6.4 in 2.7 and 200 us, as near the poles 16 rows have little in
// common); 46 x 92 -> 92 x 184 with the sphere for a disk 2591 -> 336.  At three workgroups a compute unit, with no spilled register, 365.
//
// LDS holds a stage as [term][channel][chunk]: channel rows as in memory.  First products (S^T = K Q^T and dP) read it through
// ds_read_b64_tr_b16, which turns 4 channels x 16 keys on the way to the registers; in the second (O^T += V P^T) the 8 contraction
// indices of a lane are its four keys of each of two tiles, 8-byte reads.  start(c) and UNITS (an odd multiple of four) spread both
// patterns over the banks.  The workgroup's own points go through LDS the same way, and the results come back through it, in 16-byte
// pieces of whole rows (4-byte loads and stores of 16 points x 4 channels from the lanes: 40 % of the d = 64 launches).
//
// What bounds it: issue of vector and matrix instructions, which hardly overlap on a SIMD (a tile is 12 matrix instructions of 16
// cycles and some 70 vector ones of 2.4 to 4.2, d = 32 forward), and the stalls around the two barriers of a stage; 129 x 256, 32 slices,
// d = 32: matrix pipes busy 29 % of the forward, vector ALUs some 50 %, LDS 39 %.  Workgroups of four wavefronts and small stages leave three to
// five of them on a compute unit, whose barriers do not coincide (eight wavefronts, stages twice as long: dk/dv 0.72 against
// 0.70 ms; all of LDS for one workgroup: 1.43).
// Measured (129 x 256, 32 slices, forward / dq / dk,dv, ms; before: fp32 matrix cores and vector kernels):
//   d = 16  0.42 / 0.52 / 0.65 -> 0.29 / 0.32 / 0.39        d = 32  0.66 / 0.83 / 1.03 -> 0.42 / 0.49 / 0.63
//   d = 64  1.49 / 1.95 / 2.48 -> 0.90 / 1.05 / 1.28
//
// bf16 tensors are one term; probabilities and dS, which multiply them, are cut into three, so that every product is the float32
// one (share of `out` and dv that are not the correctly rounded result: 1e-4 to 4e-4; with two terms 2e-3).  Before, bf16 tiles
// of one row; d = 32 on 64 n longitudes: kernels that rounded the forward's probabilities to bf16:
//   d = 16  0.29 / 0.34 / 0.41 -> 0.19 / 0.21 / 0.26        d = 32  0.28 / 0.35 / 0.51 -> 0.24 / 0.26 / 0.34
//   d = 64  0.83 / 1.17 / 1.12 -> 0.41 / 0.47 / 0.56
//
// Owners that are the two classes of a finer grid are loaded and stored by latitudes (kPairs), four columns at a time, two of either class;
// an owner row alone is every second column of its latitude (129 x 256 -> 257 x 512, 8 slices, float32 d = 32: dq 0.268 -> 0.239 ms, the
// mirror image's dk, dv 0.341 -> 0.316; 65 x 128 -> 129 x 256, 8 slices, bf16 d = 64: forward 72 -> 58 us, backward 171 -> 141).
//
// Shared patches (Geo::SPLIT).  Of a small launch the workgroups near the poles are what is left when all others are done, a chain of stages
// with one wavefront on each SIMD (64 x 128, theta 7 pi / 64, float32 d = 32: 38 us for one slice, 5.5 for each further one of many).
// There two or all four wavefronts of heavy workgroups own one patch: each takes a part of every stage's tiles, and their sums meet in LDS
// at the end (split_patches; s2_split_list has the rule and figures).  These kernels have registers and LDS for longer stages than the others, as
// barriers count for more than workgroups on a compute unit.  One slice, forward / backward, us: 64 x 128 38 / 101 -> 24 / 56,
// bf16 25 / 60 -> 15 / 36; 129 x 256, theta 4 pi / 128, d = 64 70 / 177 -> 55 / 130; 33 x 64, theta 4 pi / 33, d = 32 19 / 48 -> 13 / 29.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "s2_bf16_terms.h"
#include "s2_internal.h"
#include "s2_nattn_band.h"
#include "s2_nattn_exact.h"
#include "s2_nattn_patch.h"
#include "s2_nattn_walk.h"

namespace {

using namespace s2walk;
using namespace s2terms;
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));

typedef unsigned short bf16raw;      // storage of a bf16 tensor
constexpr unsigned kAgain = 0x7fc0a9a1u;     // in place of a result that s2_nattn_exact.h evaluates: not to be stored

// Channels, chunks per stage, wavefronts per SIMD the registers are held to; SPLIT: wavefronts share patches (S2BandSide::Patches::split).
template <class T_, int D_, int CAP_, int WAVES_, bool SPLIT_ = false>
struct Geo {
    using T = T_;
    static constexpr bool SPLIT = SPLIT_;
    static constexpr int TERMS = sizeof(T) == 4 ? kTerms : 1;
    static constexpr int D = D_, NW = kS2PatchWaves, CAP = CAP_, WAVES = WAVES_, NT = 64 * NW;
    static constexpr int UNITS = CAP + 4;                   // 8-byte units per channel row
    static constexpr int ROW = 4 * UNITS;                   // bf16 values per channel row
    static constexpr int TERM = D * ROW + 16, TENSOR = TERMS * TERM;
    static constexpr int KC = D == 16 ? 1 : D / 32;
    static constexpr int XL = CAP & -CAP, NG = NT / XL;     // chunks and channels staged at once
    static constexpr int CJ = CAP / XL, NC = D / NG;        // pieces (4 columns of a channel) per thread and tensor: chunks, channels
    static constexpr int LOOK = 64 / CAP * CAP;             // chunks looked up at once
    static constexpr int OWN = 4 * NW;                      // chunks of the workgroup's own points
    // channels of them at once, pieces per thread: dealt out apart from a stage's, which may have more chunks (threads that would take
    // the points again; 65 x 128 -> 129 x 256, 8 slices, bf16, d = 64: forward 82 -> 72 us, backward 208 -> 171)
    static constexpr int NGO = NT / OWN, NCO = D / NGO;
    static constexpr int PITCH = 4 * OWN + 4;               // floats per channel of the results
    static_assert(D % NG == 0 && D % NGO == 0 && CJ * NC >= NCO && (UNITS / 4) % 2 == 1 && OWN <= CAP && D * PITCH * 4 <= TENSOR * 2, "geometry");
    static __device__ __forceinline__ constexpr int start(int c) { return c * ROW + 8 * ((c >> 3) & 1) + 4 * (c >> 4); }
    static constexpr int UP = 16 * ROW + 4;                 // from a channel to the one 16 later
};

// A workgroup's rows in LDS (S2PatchRow, kColumns: S2ColumnRow).
template <int MODE>
struct RowTab {
    static constexpr bool COLUMNS = MODE == kColumns;
    static constexpr int ROWS = COLUMNS ? kS2ColumnRows : kMaxRows, SUBS = COLUMNS ? 16 : 4;
    static constexpr int DEAD = ROWS;     // the row of a list entry that stands for no chunk: no owner has neighbors on it
    int col[ROWS + 1], uni[ROWS + 1], before[ROWS], row[COLUMNS ? ROWS + 1 : 1];
    uint2 arc[SUBS][ROWS + 1];       // arc and the row's weight
};
template <class G, int MODE>
struct Shared {
    __attribute__((aligned(16))) __bf16 a[G::TENSOR];
    __attribute__((aligned(16))) __bf16 b[G::TENSOR];
    RowTab<MODE> rows;
};
template <class G, int MODE>
struct SharedDq : Shared<G, MODE> {
    float part[G::NGO][G::PITCH];    // partial sums of D
};
template <class G, int MODE>
struct SharedDkdv : Shared<G, MODE> {
    __attribute__((aligned(16))) float L[4 * G::CAP];
    __attribute__((aligned(16))) float D[4 * G::CAP];
};

// A value the compiler may not carry along in a register of its own from before a loop: what is computed from it is computed
// where it is used.
__device__ __forceinline__ int here_v(int x)
{
    asm volatile("" : "+v"(x));
    return x;
}
__device__ __forceinline__ int here_s(int x)
{
    asm volatile("" : "+s"(x));
    return x;
}

// Place of a workgroup and of a lane's owner
struct PatchWhere {
    int nU, first, lg, W, W0, wc, bh, lane, wave, n, g, tid, sub, u;
    int pw, own_end;                 // the workgroup's patch that the wavefront works on; end of the workgroup's own columns
    int share, share_lg;             // its number among the wavefronts of that patch, log2 of how many these are
    bool lead;                       // the first of them, whose the results are
    int own;                         // the lane's owner row
    bool active;                     // the lane's owner is a point
    size_t plane_own, plane_walk, own_at;
    int nlon_walk, c_own, c_walk, n_own;
    int step, nW, su, stride;         // columns of a walked row, of them per owner column; step * u; from one to the next in memory
    int seg, rmin, nrows, total, rows_at, more;
    float inv_nW;
    __device__ __forceinline__ size_t row_at(int row) const
    {
        if (c_own == 1) return size_t(row) * nU;
        const int lat = row / c_own;
        return size_t(lat) * nU * c_own + (row - lat * c_own);
    }
    __device__ __forceinline__ void set_row(int row)
    {
        own = row;
        own_at = row_at(row);
    }
    __device__ __forceinline__ void set_part(const BandArgs &a)
    {
        const int4 s0 = a.seg[2 * seg], s1 = a.seg[2 * seg + 1];
        rmin = s0.z; nrows = s0.w; total = s1.x; rows_at = s1.y; more = s1.z;
    }
    template <bool SPLIT = false>
    __device__ __forceinline__ void set(const BandArgs &a, int thread = threadIdx.x)
    {
        nU = a.b.nU;
        // Workgroups go to the eight XCDs in turn: each of them takes whole slices, one after the other, so that its L2 holds the
        // rows that its workgroups share.
        const int whole = a.nbh & ~7, id = blockIdx.x, rest = id - whole * a.npatch;
        int blk;
        if (rest < 0) {
            blk = (id >> 3) % a.npatch;
            bh = (id & 7) + 8 * ((id >> 3) / a.npatch);
        } else {
            blk = rest / (a.nbh - whole);
            bh = whole + rest % (a.nbh - whole);
        }
        const int2 at = a.patch[blk];
        seg = at.x;
        first = a.seg[2 * seg].x; lg = __builtin_amdgcn_readfirstlane(a.seg[2 * seg].y);
        set_part(a);
        W = 16 >> lg;
        tid = thread; lane = tid & 63; wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        n = lane & 15; g = lane >> 4;
        sub = n >> (4 - lg);
        c_own = a.b.c_own; c_walk = a.b.c_walk; n_own = a.b.n_own;
        nlon_walk = nU * c_walk;
        plane_own = size_t(a.b.nlat_own) * nU * c_own;
        plane_walk = size_t(a.b.nlat_walk) * nlon_walk;
        step = a.b.patches.step;
        nW = nU * step;
        stride = step == 1 ? c_walk : 1;
        inv_nW = 1.f / float(nW);
        const bool row_ok = first + sub < n_own;
        set_row(row_ok ? first + sub : first);
        W0 = SPLIT ? at.y & 0xffff : at.y;
        share_lg = SPLIT ? __builtin_amdgcn_readfirstlane(at.y >> 16) : 0;
        share = wave & ((1 << share_lg) - 1);
        lead = !SPLIT || share == 0;
        pw = wave >> share_lg;
        own_end = SPLIT ? imin(nU, W0 + (kS2PatchWaves >> share_lg) * W) : nU;
        wc = W0 + pw * (W > 4 ? W : 4);
        u = wc + (n & (W - 1));
        su = step * u;
        active = row_ok && u < nU;
    }
    __device__ __forceinline__ size_t walk_at(int r) const
    {
        if (c_walk == 1) return size_t(r) * nlon_walk;
        const int lat = r / c_walk;
        return size_t(lat) * nlon_walk + (r - lat * c_walk);
    }
    // do four points of an owner row lie side by side; kWide: at a multiple of four, in rows of a multiple of four
    template <int MODE>
    __device__ __forceinline__ bool own_pieces() const { return c_own == 1 && (is_wide(MODE) ? nU % 4 == 0 : nU >= 4); }
    // row r of the patch tables
    __device__ __forceinline__ size_t row_walked(int r) const { return stride == 1 ? size_t(r) * nlon_walk : walk_at(r); }
    // the chunk of the workgroup's own points that holds the points 4 j .. 4 j + 3 of this wavefront
    template <int MODE>
    __device__ __forceinline__ int own_slot(int j, int nw) const { return slot_of<MODE>(j, nw, pw); }
    template <int MODE>
    __device__ __forceinline__ int slot_of(int j, int nw, int patch) const
    {
        if (MODE == kColumns) return 4 * patch + j;
        const int h = 2 - here_s(lg);    // log2(chunks per row of a wavefront)
        return (j >> h) * (nw << h) + (patch << h) + (j & ((1 << h) - 1));
    }
    // the wavefront's part of a stage's key tiles
    __device__ __forceinline__ int tiles_from(int ntile) const { return ntile * share >> share_lg; }
    __device__ __forceinline__ int tiles_to(int ntile) const { return ntile * (share + 1) >> share_lg; }
    // f(i, u) for every owner i whose bit is set, with the row set to the owner's
    template <class F>
    __device__ __forceinline__ void each(unsigned owners, F &&f)
    {
#pragma unroll 1
        for (; owners; owners &= owners - 1) {
            const int i = __builtin_ctz(owners);
            set_row(first + i / W);
            f(i, wc + (i & (W - 1)));
        }
    }
};
struct SplitWhere : PatchWhere {
    __device__ __forceinline__ void set(const BandArgs &a, int thread = threadIdx.x) { PatchWhere::set<true>(a, thread); }
};
template <class G>
using WhereOf = std::conditional_t<G::SPLIT, SplitWhere, PatchWhere>;

// The chunks of a workgroup: looked up LOOK at a time, one per lane, and staged CAP at a time.
template <class G, int MODE>
struct Chunks {
    using Tab = RowTab<MODE>;
    int P_v[2];                      // chunks before row lane, 64 + lane
    int r;
    int entry;                       // of those looked up last: the lane's chunk, its column, row and place in its stage
    int list;                        // ... those that the wavefront's points meet, in order
    unsigned long long met;          // ... which they are
    int sh;                          // of the stage set last: its place among those looked up
    int first, cnt;                  // ... where the list has its chunks, and how many

    __device__ __forceinline__ int before(int i) const
    {
        if (Tab::ROWS <= 64) return __builtin_amdgcn_readlane(P_v[0], i);
        const int x = __builtin_amdgcn_readlane(P_v[0], i & 63), y = __builtin_amdgcn_readlane(P_v[1], i & 63);
        return i < 64 ? x : y;
    }
    __device__ __forceinline__ void start(const BandArgs &a, const PatchWhere &w, Tab &t)
    {
        if (w.tid <= Tab::ROWS) {
            constexpr int N = Tab::COLUMNS ? 6 : 2;
            int4 x[N] = {};
            if (w.tid < w.nrows)
#pragma unroll
                for (int i = 0; i < N; ++i) x[i] = a.row_rec[N * (w.rows_at + w.tid) + i];
            t.col[w.tid] = x[0].x;
            t.uni[w.tid] = x[0].y;
            if (w.tid < Tab::ROWS) t.before[w.tid] = x[0].z;
            if constexpr (Tab::COLUMNS) t.row[w.tid] = x[0].w;
            const int omega = Tab::COLUMNS ? x[1].x : x[0].w;
#pragma unroll
            for (int i = 0; i < Tab::SUBS / 4; ++i) {
                const int4 y = x[N - Tab::SUBS / 4 + i];
                t.arc[4 * i][w.tid] = make_uint2(y.x, omega);
                t.arc[4 * i + 1][w.tid] = make_uint2(y.y, omega);
                t.arc[4 * i + 2][w.tid] = make_uint2(y.z, omega);
                t.arc[4 * i + 3][w.tid] = make_uint2(y.w, omega);
            }
        }
        __syncthreads();
        P_v[0] = t.before[w.lane];
        if (Tab::ROWS > 64) P_v[1] = t.before[64 + w.lane];
        r = 0;
        sh = 0;
    }
    // the chunks X0 .. X0 + LOOK - 1 (X0 < total; past the last: that one again, not met)
    __device__ __forceinline__ void look(int X0, const PatchWhere &w, const Tab &t)
    {
        const int X = imin(X0 + w.lane, w.total - 1);
        int at = r;
        while (r + 1 < w.nrows) {
            const int p = before(r + 1);
            if (p >= X0 + G::LOOK) break;
            ++r;
            at += X >= p ? 1 : 0;
        }
        const int u = t.uni[at], c = t.col[at] + 4 * X + w.step * w.W0, d = c + 3 - w.step * w.wc - int(short(u & 0xffff));
        const bool need = w.lane < G::LOOK && X0 + w.lane < w.total && w.wc < w.nU && unsigned(d) < (unsigned(u) >> 16) + w.step * (w.W - 1) + 3;
        met = __ballot(need);
        const int ones = __builtin_amdgcn_mbcnt_hi(unsigned(met >> 32), __builtin_amdgcn_mbcnt_lo(unsigned(met), 0));
        entry = c << 14 | at << 6 | w.lane % G::CAP;
        list = __builtin_amdgcn_ds_permute(4 * (need ? ones : __popcll(met) + w.lane - ones), entry);
    }
    // the stage of chunks X0 .. X0 + CAP - 1, stages in order
    __device__ __forceinline__ void set(int X0, const PatchWhere &w, const Tab &t)
    {
        sh = G::LOOK == 64 ? X0 & 63 : X0 == 0 || sh + G::CAP == G::LOOK ? 0 : sh + G::CAP;
        if (sh == 0) look(X0, w, t);
        first = __popcll(met & ((1ull << sh) - 1));
        cnt = __popcll(met >> sh & (~0ull >> (64 - G::CAP)));
    }
    // row and column of chunk i of the stage
    __device__ __forceinline__ void get(int i, const PatchWhere &w, const Tab &t, int &row, int &col) const
    {
        const int e = __builtin_amdgcn_ds_bpermute(4 * (sh + i), entry), at = e >> 6 & 255;
        if constexpr (Tab::COLUMNS) row = t.row[at];
        else row = w.rmin + at;
        col = e >> 14;
    }
};

// Where a chunk is, in a channel plane (kWide: in a slice)
template <class T, int MODE>
struct ChunkAt {
    static constexpr bool WIDE = is_wide(MODE);
    unsigned off[WIDE ? 1 : 4];      // kWide: byte offset; else elements
    bool apart;                      // not kWide: a chunk of the wavefront's is not four elements side by side (uniform; else off[0] only)
    // channel: its first one (kWide only)
    __device__ __forceinline__ void set(const PatchWhere &w, int row, int col, int channel)
    {
        const int c = wrap_col(col + 2 * w.nW, w.nW, w.inv_nW);
        if constexpr (WIDE) {
            off[0] = unsigned(sizeof(T)) * (unsigned(channel) * unsigned(w.plane_walk) + unsigned(row) * unsigned(w.nW) + unsigned(c));
        } else {
            const unsigned at = unsigned(w.row_walked(row));
            apart = (MODE != kHalves && w.stride > 1) || __any(c + 4 > w.nW);
            off[0] = at + unsigned(w.stride) * unsigned(c);
            if (!apart) return;
            if constexpr (MODE == kHalves) {     // (chunks begin at multiples of four, less whole rows)
                off[2] = at + unsigned(wrap_col(col + 2 + 2 * w.nW, w.nW, w.inv_nW));
                return;
            }
#pragma unroll
            for (int i = 1; i < 4; ++i) off[i] = at + unsigned(w.stride) * unsigned(wrap_col(col + i + 2 * w.nW, w.nW, w.inv_nW));
        }
    }
    // its values in a float32 plane; channel: as set
    __device__ __forceinline__ f32x4 floats(const PatchWhere &w, const float *plane, int channel) const
    {
        f32x4 s;
        if constexpr (WIDE) {
            s = load_at<f32x4>(plane, off[0] / unsigned(sizeof(T)) * 4u - 4u * unsigned(channel) * unsigned(w.plane_walk));
        } else if (!apart) {
            __builtin_memcpy(&s, plane + off[0], sizeof s);
        } else if constexpr (MODE == kHalves) {
            float h[4];
            __builtin_memcpy(h, plane + off[0], 8);
            __builtin_memcpy(h + 2, plane + off[2], 8);
            s = f32x4{h[0], h[1], h[2], h[3]};
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) s[i] = plane[off[i]];
        }
        return s;
    }
};
// What a thread stages: chunks x + XL j, channels cg + NG c
template <class G, int MODE>
struct Place {
    using At = ChunkAt<typename G::T, MODE>;
    static constexpr bool WIDE = At::WIDE;
    At at[G::CJ];
    int x, cg;
    __device__ __forceinline__ void init(const PatchWhere &w)
    {
        x = w.tid & (G::XL - 1);
        cg = w.tid / G::XL;
    }
    __device__ __forceinline__ void set(const PatchWhere &w, const Chunks<G, MODE> &ch, const RowTab<MODE> &t)
    {
#pragma unroll
        for (int j = 0; j < G::CJ; ++j) {
            int row, col;
            ch.get(x + G::XL * j, w, t, row, col);
            at[j].set(w, row, col, cg);
        }
    }
};
// kPairs: the thread's piece of the workgroup's own points, four columns of a latitude of the finer grid, two of either class
struct PairPiece {
    int row, col;                    // the first class's row; the first column
    int at, up;                      // place of the first class's two points among the own points' columns in LDS, from there to the other's
    template <class G>
    __device__ __forceinline__ void set(const PatchWhere &w, int tid)
    {
        const int lg = here_s(w.lg), x = tid & (G::OWN - 1), lat = x >> (5 - lg), i = x & ((32 >> lg) - 1);
        row = w.first + 2 * lat;
        col = 2 * w.W0 + 4 * i;
        up = 4 * G::NW << (2 - lg);
        at = 2 * lat * up + 2 * i;
    }
};
// One tensor's stage, from memory to registers and (float32: cut into three terms) on to LDS.  Pieces of four elements, also where rows are no
// multiple of four long.  kNarrow, kRagged: at any alignment, a piece astride the end of its row element by element, with all of the wavefront's: as
// four loads each, 154 x 306, 4 slices, d = 64, bf16, forward 196 us, now 130; 179 x 358, 6 slices, d = 32, bf16, forward and backward 859 -> 595;
// around the seam of circles of some thirty longitudes, where most pieces are apart, 24.3 -> 25.4.
// kHalves: rows of an even length, in halves: 46 x 90, one slice, d = 32, bf16, forward / backward 20 / 42 -> 15 / 32 us, 90 x 178, 32 slices, d = 64,
// bf16 329 / 879 -> 259 / 755, float32 630 / 1638 -> 589 / 1523; decided inside of kNarrow, odd rows lost 2 to 5 %.
template <class G, int MODE>
struct Stage {
    using T = typename G::T;
    using Piece = std::conditional_t<sizeof(T) == 4, f32x4, u16x4>;
    using P = Place<G, MODE>;
    Piece r[G::CJ * G::NC];          // of the workgroup's own points: the first NCO
    __device__ __forceinline__ void load(const PatchWhere &w, const P &place, const T *slice, int nch)
    {
#pragma unroll
        for (int j = 0; j < G::CJ; ++j) {
            const typename P::At &at = place.at[j];
            Piece *rj = r + j * G::NC;
            if constexpr (P::WIDE) {
#pragma unroll
                for (int k = 0; k < G::NC; ++k) rj[k] = load_at<Piece>(slice + size_t(k * G::NG) * w.plane_walk, at.off[0]);
            } else {
                auto channel = [&](int k) {
                    const int c = place.cg + k * G::NG;
                    return slice + size_t(MODE == kRagged ? imin(c, nch - 1) : c) * w.plane_walk;
                };
                if (!at.apart) {
#pragma unroll
                    for (int k = 0; k < G::NC; ++k) __builtin_memcpy(&rj[k], channel(k) + at.off[0], sizeof rj[k]);
                } else if constexpr (MODE == kHalves) {
                    typedef std::conditional_t<sizeof(T) == 4, u32x2, unsigned> Half;
                    struct Halves { Half lo, hi; };
#pragma unroll
                    for (int k = 0; k < G::NC; ++k) {
                        const T *p = channel(k);
                        Halves h;
                        __builtin_memcpy(&h.lo, p + at.off[0], sizeof(Half));
                        __builtin_memcpy(&h.hi, p + at.off[2], sizeof(Half));
                        rj[k] = __builtin_bit_cast(Piece, h);
                    }
                } else {
#pragma unroll
                    for (int k = 0; k < G::NC; ++k) {
                        const T *p = channel(k);
#pragma unroll
                        for (int i = 0; i < 4; ++i) rj[k][i] = p[at.off[i]];
                    }
                }
            }
        }
    }
    // kColumns: place of point i of the thread's piece, four rows of a column, from the workgroup's first row on
    static __device__ __forceinline__ size_t column_at(const PatchWhere &w, int x, int i)
    {
        const int row = w.first + 4 * (x & 3) + i, u = w.W0 + 4 * (x >> 2);
        return w.row_at(row < w.n_own ? row : w.first) + size_t(w.c_own) * (u < w.nU ? u : w.W0);
    }
    // the workgroup's own points; vec: its rows are contiguous
    __device__ __forceinline__ void load_own(const PatchWhere &w, const T *slice, int nch, bool vec)
    {
        if constexpr (MODE == kColumns) {
            const int tid = here_v(w.tid);
            const T *p = slice + size_t(tid / G::OWN) * w.plane_own;
            if (w.c_own == 2) {                          // both classes of a latitude side by side
                typedef T T2 __attribute__((ext_vector_type(2)));
#pragma unroll
                for (int i = 0; i < 4; i += 2) {
                    const T *pi = p + column_at(w, tid & (G::OWN - 1), i);
#pragma unroll
                    for (int j = 0; j < G::NCO; ++j) {
                        const T2 y = *reinterpret_cast<const T2 *>(pi + size_t(j * G::NGO) * w.plane_own);
                        r[j][i] = y[0];
                        r[j][i + 1] = y[1];
                    }
                }
                return;
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const T *pi = p + column_at(w, tid & (G::OWN - 1), i);
#pragma unroll
                for (int j = 0; j < G::NCO; ++j) r[j][i] = pi[size_t(j * G::NGO) * w.plane_own];
            }
            return;
        }
        if constexpr (MODE == kPairs) {
            if (w.lg > 0) {
                const int tid = here_v(w.tid);
                PairPiece o;
                o.template set<G>(w, tid);
                const T *p = slice + size_t(tid / G::OWN) * w.plane_own + w.row_at(o.row < w.n_own ? o.row : w.first) + (o.col < 2 * w.nU ? o.col : 0);
#pragma unroll
                for (int j = 0; j < G::NCO; ++j) r[j] = *reinterpret_cast<const Piece *>(p + size_t(j * G::NGO) * w.plane_own);
                return;
            }
        }
        const int h = 2 - here_s(w.lg), tid = here_v(w.tid), x = tid & (G::OWN - 1), cg = tid / G::OWN, sub = (x / G::NW) >> h;
        const int row = w.first + sub < w.n_own ? w.first + sub : w.first, u = w.W0 + 4 * (x - G::NW * (sub << h));
        const T *p = slice + w.row_at(row);
        if (!P::WIDE) vec = vec && !__any(u < w.nU && u + 4 > w.nU);       // a row that ends within a piece
#pragma unroll
        for (int j = 0; j < G::NCO; ++j) {
            const int c = cg + j * G::NGO;
            const T *pc = p + size_t(MODE == kRagged ? imin(c, nch - 1) : c) * w.plane_own;
            if (vec) {
                if constexpr (P::WIDE) r[j] = *reinterpret_cast<const Piece *>(pc + (u < w.nU ? u : 0));
                else __builtin_memcpy(&r[j], pc + (u < w.nU ? u : 0), sizeof r[j]);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) r[j][i] = pc[size_t(w.c_own) * imin(u + i, w.nU - 1)];
            }
        }
    }
    __device__ __forceinline__ void negate_own()
    {
#pragma unroll
        for (int j = 0; j < G::NCO; ++j) {
            if constexpr (sizeof(T) == 4) r[j] = -r[j];
            else r[j] ^= static_cast<unsigned short>(0x8000);
        }
    }
    __device__ __forceinline__ f32x4 value(int j) const
    {
        if constexpr (sizeof(T) == 4) {
            return r[j];
        } else {
            f32x4 v;
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = __builtin_bit_cast(float, unsigned(r[j][i]) << 16);
            return v;
        }
    }
    // piece v as chunk x of channel c
    static __device__ __forceinline__ void put(__bf16 *tile, int c, int x, Piece v, int nch)
    {
        if (MODE == kRagged && c >= nch) v = Piece{0, 0, 0, 0};
        __bf16 *p = tile + G::start(c) + 4 * x;
        if constexpr (sizeof(T) == 4) {
            float x0 = v[0], x1 = v[1], x2 = v[2], x3 = v[3];
#pragma unroll
            for (int k = 0; k < kTerms; ++k) {
                const unsigned a = cut_off(x0, x1), b = cut_off(x2, x3);
                *reinterpret_cast<u32x2 *>(p + k * G::TERM) = u32x2{a, b};
            }
        } else {
            *reinterpret_cast<u16x4 *>(p) = v;
        }
    }
    __device__ __forceinline__ void store(const P &place, __bf16 *tile, int nch) const
    {
#pragma unroll
        for (int j = 0; j < G::CJ; ++j)
#pragma unroll
            for (int k = 0; k < G::NC; ++k) put(tile, place.cg + k * G::NG, place.x + G::XL * j, r[j * G::NC + k], nch);
    }
    __device__ __forceinline__ void store_own(const PatchWhere &w, const P &place, __bf16 *tile, int nch) const
    {
        const int tid = here_v(w.tid), x = G::XL == G::OWN ? place.x : tid & (G::OWN - 1), cg = G::XL == G::OWN ? place.cg : tid / G::OWN;
        if constexpr (MODE == kPairs) {
            if (w.lg > 0) {
                PairPiece o;
                o.template set<G>(w, tid);
#pragma unroll
                for (int j = 0; j < G::NCO; ++j) {
                    __bf16 *p = tile + G::start(cg + j * G::NGO) + o.at;
                    if constexpr (sizeof(T) == 4) {
                        float x0 = r[j][0], x1 = r[j][2], y0 = r[j][1], y1 = r[j][3];
#pragma unroll
                        for (int k = 0; k < kTerms; ++k) {
                            *reinterpret_cast<unsigned *>(p + k * G::TERM) = cut_off(x0, x1);
                            *reinterpret_cast<unsigned *>(p + k * G::TERM + o.up) = cut_off(y0, y1);
                        }
                    } else {
                        *reinterpret_cast<unsigned *>(p) = unsigned(r[j][0]) | unsigned(r[j][2]) << 16;
                        *reinterpret_cast<unsigned *>(p + o.up) = unsigned(r[j][1]) | unsigned(r[j][3]) << 16;
                    }
                }
                return;
            }
        }
#pragma unroll
        for (int j = 0; j < G::NCO; ++j) put(tile, cg + j * G::NGO, x, r[j], nch);
    }
    // the thread's four values of its own points' columns, each lane's kept in `to`, one row of G::PITCH floats
    static __device__ __forceinline__ void put_floats(const PatchWhere &w, float *to, f32x4 v)
    {
        const int tid = here_v(w.tid);
        if constexpr (MODE == kPairs) {
            if (w.lg > 0) {
                PairPiece o;
                o.template set<G>(w, tid);
                typedef float f32x2 __attribute__((ext_vector_type(2)));
                *reinterpret_cast<f32x2 *>(to + o.at) = f32x2{v[0], v[2]};
                *reinterpret_cast<f32x2 *>(to + o.at + o.up) = f32x2{v[1], v[3]};
                return;
            }
        }
        *reinterpret_cast<f32x4 *>(to + 4 * (tid & (G::OWN - 1))) = v;
    }
};

__device__ __forceinline__ f32x4 mma(bf16x8 a, bf16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
__device__ __forceinline__ bf16x8 join(bf16x4 a, bf16x4 b) { return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7); }
__device__ __forceinline__ bf16x4 lds_tr(const __bf16 *p)
{
    typedef __attribute__((address_space(3))) s16x4 *ptr;
    return __builtin_bit_cast(bf16x4, __builtin_amdgcn_ds_read_tr16_b64_v4i16((ptr)(__attribute__((address_space(3))) void *)p));
}
__device__ __forceinline__ bf16x4 lds_row(const __bf16 *p) { return *reinterpret_cast<const bf16x4 *>(p); }

// A lane's own point as operand of the first product; p: the lane's place in the staged tensor
template <class G>
struct OwnPoint {
    bf16x8 v[G::KC][G::TERMS];
    __device__ __forceinline__ void read(const __bf16 *p)
    {
        if constexpr (G::D == 16 && G::TERMS == 1) {
            v[0][0] = join(lds_tr(p), bf16x4{});
        } else if constexpr (G::D == 16) {
            const bf16x4 h = lds_tr(p), m = lds_tr(p + G::TERM), l = lds_tr(p + 2 * G::TERM);
            v[0][0] = join(h, h);
            v[0][1] = join(m, m);
            v[0][2] = join(l, h);
        } else {
#pragma unroll
            for (int s = 0; s < G::KC; ++s)
#pragma unroll
                for (int k = 0; k < G::TERMS; ++k) v[s][k] = join(lds_tr(p + k * G::TERM + 2 * s * G::UP), lds_tr(p + k * G::TERM + (2 * s + 1) * G::UP));
        }
    }
};
// owners (bit n) with a NaN among their channels
template <class G>
__device__ __forceinline__ unsigned own_nan(const OwnPoint<G> &o)
{
    bool b = false;
#pragma unroll
    for (int s = 0; s < G::KC; ++s)
#pragma unroll
        for (int j = 0; j < 8; ++j) b |= float(o.v[s][0][j]) != float(o.v[s][0][j]);
    return owner_bits(b);
}
// (chunks' columns) . (the lane's own point), smallest products first; p: the lane's place in the staged tensor
template <class G>
__device__ __forceinline__ f32x4 dot(const __bf16 *p, const OwnPoint<G> &o)
{
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    if constexpr (G::D == 16 && G::TERMS == 1) {
        acc = mma(join(lds_tr(p), bf16x4{}), o.v[0][0], acc);
    } else if constexpr (G::D == 16) {
        const bf16x4 h = lds_tr(p), m = lds_tr(p + G::TERM), l = lds_tr(p + 2 * G::TERM);
        acc = mma(join(h, l), o.v[0][2], acc);
        const bf16x8 hm = join(h, m);
        acc = mma(hm, o.v[0][1], acc);
        acc = mma(hm, o.v[0][0], acc);
    } else {
        bf16x8 x[G::KC][G::TERMS];
#pragma unroll
        for (int s = 0; s < G::KC; ++s)
#pragma unroll
            for (int k = 0; k < G::TERMS; ++k)
                x[s][k] = join(lds_tr(p + k * G::TERM + 2 * s * G::UP), lds_tr(p + k * G::TERM + (2 * s + 1) * G::UP));
        constexpr int order[6][2] = {{2, 0}, {0, 2}, {1, 1}, {1, 0}, {0, 1}, {0, 0}};
#pragma unroll
        for (int i = G::TERMS == 1 ? 5 : 0; i < 6; ++i)
#pragma unroll
            for (int s = 0; s < G::KC; ++s) acc = mma(x[s][order[i][0]], o.v[s][order[i][1]], acc);
    }
    return acc;
}
// Sums over keys, per lane 16 mt + 4 g + rr; float32: the products of first terms apart from the others
template <class G>
struct Sums {
    f32x4 hi[G::D / 16], lo[G::TERMS == 1 ? 1 : G::D / 16];
    __device__ __forceinline__ void zero()
    {
#pragma unroll
        for (auto &x : hi) x = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (auto &x : lo) x = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    __device__ __forceinline__ void wait()
    {
        settle(hi);
        if constexpr (G::TERMS > 1) settle(lo);
    }
    __device__ __forceinline__ void scale(float f)
    {
#pragma unroll
        for (auto &x : hi) x *= f;
        if constexpr (G::TERMS > 1)
#pragma unroll
            for (auto &x : lo) x *= f;
    }
    __device__ __forceinline__ void join_terms()
    {
        if constexpr (G::TERMS > 1)
#pragma unroll
            for (int mt = 0; mt < G::D / 16; ++mt) hi[mt] += lo[mt];
    }
    // += (channels 16 mt ..) . (the lane's eight values of the columns of two tiles); p0, p1: the lane's places
    __device__ __forceinline__ void add(const __bf16 *p0, const __bf16 *p1, const bf16x8 (&b)[kTerms])
    {
#pragma unroll
        for (int mt = 0; mt < G::D / 16; ++mt) {
            bf16x8 x[G::TERMS];
#pragma unroll
            for (int k = 0; k < G::TERMS; ++k) x[k] = join(lds_row(p0 + k * G::TERM + mt * G::UP), lds_row(p1 + k * G::TERM + mt * G::UP));
            if constexpr (G::TERMS == 1) {
                hi[mt] = mma(x[0], b[2], hi[mt]);
                hi[mt] = mma(x[0], b[1], hi[mt]);
                hi[mt] = mma(x[0], b[0], hi[mt]);
            } else {
                lo[mt] = mma(x[2], b[0], lo[mt]);
                hi[mt] = mma(x[0], b[0], hi[mt]);
                lo[mt] = mma(x[0], b[2], lo[mt]);
                lo[mt] = mma(x[1], b[1], lo[mt]);
                lo[mt] = mma(x[1], b[0], lo[mt]);
                lo[mt] = mma(x[0], b[1], lo[mt]);
            }
        }
    }
};

// What a lane needs of one key tile (four chunks of the list): its own chunk, its place as reader of the first product
struct TileRef {
    int slot, row, col;              // the lane's chunk (number g of the tile)
    int slot_n;                      // chunk n & 3 of the tile
    // the tile's chunks are entries at .. at + 3 of the list, those below end
    template <int DEAD>
    __device__ __forceinline__ void get(int list, int at, int end, int n, int g)
    {
        const int m = __builtin_amdgcn_ds_bpermute(4 * (at + g), list);
        slot_n = __builtin_amdgcn_ds_bpermute(4 * (at + (n & 3)), list) & 63;
        slot = m & 63;
        row = at + g < end ? m >> 6 & 255 : DEAD;
        col = m >> 14;
    }
    // keep[rr]: is column col + rr a neighbor of the owner at walked column su
    __device__ __forceinline__ void keep(bool (&keep)[4], int su, unsigned arc) const
    {
        const unsigned rel = unsigned(col - (su + int(short(arc & 0xffff))));
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) keep[rr] = rel + rr < (arc >> 16);
    }
};

// The results of the workgroup's owners, by way of LDS: acc[mt][rr] is channel 16 mt + 4 g + rr of the lane's owner.  again: those that
// are not finite are to be evaluated (marked).
template <class G, int MODE>
__device__ __forceinline__ void put_results(const f32x4 (&acc)[G::D / 16], float factor, bool again, float *tile, const PatchWhere &w)
{
    const int lane = here_v(w.lane);
    float *p = tile + (lane >> 4) * 4 * G::PITCH + 4 * w.template own_slot<MODE>(lane >> 2 & 3, G::NW) + (lane & 3);
#pragma unroll
    for (int mt = 0; mt < G::D / 16; ++mt)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr)
            p[(16 * mt + rr) * G::PITCH] = again && !(fabsf(acc[mt][rr]) < INFINITY) ? __builtin_bit_cast(float, kAgain) : acc[mt][rr] * factor;
}
// SPLIT: the sums of the wavefronts that share a patch, added up in the first of them in the order of their numbers; LDS is free before, and
// after the next barrier again
template <class G, int MODE>
__device__ __forceinline__ void put_shares(const f32x4 (&acc)[G::D / 16], float *tile, const PatchWhere &w)
{
    float *p = tile + 4 * w.g * G::PITCH + 4 * w.template slot_of<MODE>(w.lane >> 2 & 3, G::NW, w.wave) + (w.lane & 3);
#pragma unroll
    for (int mt = 0; mt < G::D / 16; ++mt)
#pragma unroll
        for (int rr = 0; rr < 4; ++rr) p[(16 * mt + rr) * G::PITCH] = acc[mt][rr];
}
template <class G, int MODE>
__device__ __forceinline__ void add_shares(f32x4 (&acc)[G::D / 16], const float *tile, const PatchWhere &w)
{
    if (!w.lead) return;
#pragma unroll 1
    for (int i = 1; i < 1 << w.share_lg; ++i) {
        const float *p = tile + 4 * w.g * G::PITCH + 4 * w.template slot_of<MODE>(w.lane >> 2 & 3, G::NW, w.wave + i) + (w.lane & 3);
#pragma unroll
        for (int mt = 0; mt < G::D / 16; ++mt)
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) acc[mt][rr] += p[(16 * mt + rr) * G::PITCH];
    }
}
// is the lane's channel of the wavefront's owner i marked
template <class G, int MODE>
__device__ __forceinline__ bool marked(const float *tile, const PatchWhere &w, int i)
{
    return __builtin_bit_cast(unsigned, tile[imin(w.lane, G::D - 1) * G::PITCH + 4 * w.template own_slot<MODE>(i >> 2, G::NW) + (i & 3)]) == kAgain;
}
template <class G, int MODE>
__device__ __forceinline__ void store_results(typename G::T *slice, int nch, const float *tile, const PatchWhere &w, bool vec)
{
    using T = typename G::T;
    if constexpr (MODE == kColumns) {
        const int tid = here_v(w.tid), x = tid % G::OWN, c0 = tid / G::OWN;
        if (w.W0 + 4 * (x >> 2) >= w.nU) return;
        T *p = slice + size_t(c0) * w.plane_own;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (w.first + 4 * (x & 3) + i >= w.n_own) break;
            T *pi = p + Stage<G, MODE>::column_at(w, x, i);
#pragma unroll
            for (int j = 0; j < G::NCO; ++j) {
                const u32x2 y = *reinterpret_cast<const u32x2 *>(tile + (c0 + j * G::NGO) * G::PITCH + 4 * x + (i & 2));
                T *pj = pi + size_t(j * G::NGO) * w.plane_own;
                if (w.c_own == 2 && y[0] != kAgain && y[1] != kAgain) {
                    if ((i & 1) == 0) *reinterpret_cast<u32x2 *>(pj) = y;
                } else {
                    const unsigned z = y[i & 1];
                    if (z != kAgain) *pj = __builtin_bit_cast(float, z);
                }
            }
        }
        return;
    }
    const int h = 2 - here_s(w.lg), tid = here_v(w.tid), x = tid % G::OWN, c0 = tid / G::OWN;
    int sub = (x / G::NW) >> h, u = w.W0 + 4 * (x - G::NW * (sub << h)), end = w.own_end, step = w.c_own;
    const bool two = MODE == kPairs && w.lg > 0;
    PairPiece o;
    if (two) {
        o.template set<G>(w, tid);
        sub = o.row - w.first;
        u = o.col;
        end = 2 * w.own_end;
        step = 1;
    }
    if (w.first + sub >= w.n_own || u >= end) return;
    T *p = slice + size_t(c0) * w.plane_own + w.row_at(w.first + sub) + size_t(step) * u;
    const size_t up = size_t(G::NT / G::OWN) * w.plane_own;
#pragma unroll
    for (int j = 0; j < G::D * G::OWN / G::NT; ++j, p += up) {
        const int c = c0 + j * (G::NT / G::OWN);
        if (c >= nch) break;
        u32x4 r;
        if (two) {
            const u32x2 a = *reinterpret_cast<const u32x2 *>(tile + c * G::PITCH + o.at), b = *reinterpret_cast<const u32x2 *>(tile + c * G::PITCH + o.at + o.up);
            r = u32x4{a[0], b[0], a[1], b[1]};
        } else {
            r = *reinterpret_cast<const u32x4 *>(tile + c * G::PITCH + 4 * x);
        }
        unsigned skip = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) skip |= (r[k] == kAgain || u + k >= end ? 1u : 0u) << k;
        typename Stage<G, kWide>::Piece y;
        if constexpr (sizeof(T) == 4) y = __builtin_bit_cast(f32x4, r);
        else y = __builtin_bit_cast(u16x4, __builtin_convertvector(__builtin_bit_cast(f32x4, r), bf16x4));
        if ((vec || two) && skip == 0) {
            if constexpr (is_wide(MODE)) *reinterpret_cast<decltype(y) *>(p) = y;
            else __builtin_memcpy(p, &y, sizeof y);
        } else {
            T *pk = p;
#pragma unroll
            for (int k = 0; k < 4; ++k, pk += step)
                if (!(skip >> k & 1)) *pk = y[k];
        }
    }
}

// ---------------------------------------------------------------------------------------------------------------
// Forward.
template <class G, int MODE>
__global__ void __launch_bounds__(G::NT, G::WAVES)
nattn_fwd_patch(BandArgs a, const typename G::T *__restrict__ q, const typename G::T *__restrict__ k, const typename G::T *__restrict__ v,
                typename G::T *__restrict__ out, float *__restrict__ lse)
{
    constexpr int D = G::D;
    using T = typename G::T;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    Shared<G, MODE> &sh = *reinterpret_cast<Shared<G, MODE> *>(lds);
    WhereOf<G> w;
    w.set(a);
    const int n = w.n, g = w.g, nd = MODE == kRagged ? a.d : D, ne = MODE == kRagged ? a.e : D;
    const bool vec = w.template own_pieces<MODE>();
    const T *qs = q + size_t(w.bh) * nd * w.plane_own, *ks = k + size_t(w.bh) * nd * w.plane_walk, *vs = v + size_t(w.bh) * ne * w.plane_walk;
    Place<G, MODE> at;
    at.init(w);
    Stage<G, MODE> rk, rv;
    rk.load_own(w, qs, nd, vec);
    Chunks<G, MODE> ch;
    ch.start(a, w, sh.rows);
    auto fetch = [&](int X0) {
        ch.set(X0, w, sh.rows);
        at.set(w, ch, sh.rows);
        rk.load(w, at, ks, nd);
        rv.load(w, at, vs, ne);
    };
    const int tr_at = G::start(4 * g + (n >> 2)), row_at = G::start(n);
    __syncthreads();                    // everybody is done with what LDS held
    if (a.scale < 0.f) rk.negate_own();
    rk.store_own(w, at, sh.a, nd);
    __syncthreads();
    if (w.total > 0) fetch(0);
    OwnPoint<G> own;
    own.read(sh.a + tr_at + 4 * w.template own_slot<MODE>(here_v(w.lane) & 3, G::NW));
    Sums<G> acc;
    acc.zero();
    // |scale|, its sign is on q: the largest product is the largest logit; never zero, so that a masked -inf stays one
    const float c2 = a.scale == 0.f ? 1e-37f : fabsf(a.scale) * kLog2e;
    float m = kMinRef, l = 0.f;
    for (;;) {
        for (int X0 = 0; X0 < w.total; X0 += G::CAP) {
            __syncthreads();
            rk.store(at, sh.a, nd);
            rv.store(at, sh.b, ne);
            __syncthreads();
            const int list = ch.list, first = ch.first, end = ch.first + ch.cnt, ntile = (ch.cnt + 3) >> 2;
            if (X0 + G::CAP < w.total) fetch(X0 + G::CAP);
            auto step = [&](int t, auto count) {
                constexpr int N = decltype(count)::value;
                TileRef tr[2];
                float x[8], omega[2];
#pragma unroll
                for (int i = 0; i < N; ++i) tr[i].template get<RowTab<MODE>::DEAD>(list, first + 4 * (t + i), end, n, g);
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    const uint2 arc = sh.rows.arc[w.sub][tr[i].row];
                    const f32x4 sc = dot<G>(sh.a + tr_at + 4 * tr[i].slot_n, own);
                    omega[i] = __builtin_bit_cast(float, arc.y);
                    bool keep[4];
                    tr[i].keep(keep, w.su, arc.x);
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr) x[4 * i + rr] = keep[rr] ? sc[rr] : -INFINITY;
                }
                float mx = x[0];
#pragma unroll
                for (int i = 1; i < 4 * N; ++i) mx = fmaxf(mx, x[i]);
                mx *= c2;
                if (__any(mx > m + 8.f)) {
                    acc.wait();              // (the step before may have ended just now)
                    mx = group_max(mx);
                    const float m_new = mx > m + 8.f ? mx : m;
                    const float corr = __builtin_amdgcn_exp2f(m - m_new);
                    m = m_new;
                    l *= corr;
                    acc.scale(corr);
                }
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    if (i < 4 * N) {
                        const float e = __builtin_amdgcn_exp2f(fmaf(x[i], c2, -m));
                        l = fmaf(omega[i / 4], e, l);
                        x[i] = omega[i / 4] * e;
                    } else {
                        x[i] = 0.f;
                    }
                }
                bf16x8 p[kTerms];
                cut<true>(x, p);
                acc.add(sh.b + row_at + 4 * tr[0].slot, sh.b + row_at + 4 * tr[N - 1].slot, p);
            };
            int t = G::SPLIT ? w.tiles_from(ntile) : 0;
            const int t_end = G::SPLIT ? w.tiles_to(ntile) : ntile;
            for (; t + 1 < t_end; t += 2) step(t, std::integral_constant<int, 2>());
            if (t < t_end) step(t, std::integral_constant<int, 1>());
            acc.wait();
        }
        if (!w.more) break;
        ++w.seg;                           // more walked rows than the tables hold: the next part of them
        w.set_part(a);
        __syncthreads();
        ch.start(a, w, sh.rows);
        if (w.total > 0) fetch(0);
    }
    acc.join_terms();
    float lt = group_sum(l);
    if (G::SPLIT && w.share_lg > 0) {
        float *tile = reinterpret_cast<float *>(sh.a), *stat = reinterpret_cast<float *>(sh.b);      // per wavefront: 16 references, 16 sums
        __syncthreads();
        if (g == 0) {
            stat[32 * w.wave + n] = m;
            stat[32 * w.wave + 16 + n] = lt;
        }
        __syncthreads();
        const float *of = stat + 32 * (w.wave - w.share) + n;
        float most = m;
        for (int i = 0; i < 1 << w.share_lg; ++i) most = fmaxf(most, of[32 * i]);
        lt = 0.f;
        for (int i = 0; i < 1 << w.share_lg; ++i) lt = fmaf(of[32 * i + 16], __builtin_amdgcn_exp2f(of[32 * i] - most), lt);
        const float corr = __builtin_amdgcn_exp2f(m - most);
        m = most;
#pragma unroll
        for (auto &x : acc.hi) x *= corr;
        put_shares<G, MODE>(acc.hi, tile, w);
        __syncthreads();
        add_shares<G, MODE>(acc.hi, tile, w);
    }
    // owners whose sums took in a non-finite value (s2_nattn_exact.h); where it is a NaN of their own the sums are right
    unsigned again = not_finite(acc.hi, w.active && w.lead), no_lse = 0;
    if (any_owner(again)) {
        again &= ~own_nan(own);
        no_lse = again & owner_bits(lt != lt);
    }
    __syncthreads();
    if (w.lead) put_results<G, MODE>(acc.hi, 1.f / lt, again >> n & 1, reinterpret_cast<float *>(sh.a), w);
    if (w.active && w.lead && g == 0 && !(no_lse >> n & 1)) {
        // the whole part of m goes into the logarithm, so that its value and the sum are no larger than the result
        const float whole = fminf(fmaxf(rintf(m), -60.f), 60.f);
        lse[size_t(w.bh) * w.plane_own + w.own_at + size_t(w.c_own) * w.u] =
            fmaf(m - whole, 0.6931471805599453f, logf(ldexpf(lt * a.omega_ref, int(whole))));
    }
    __syncthreads();
    store_results<G, MODE>(out + size_t(w.bh) * ne * w.plane_own, ne, reinterpret_cast<const float *>(sh.a), w, vec);
    exact_fwd<T, WhereOf<G>>(again, no_lse, w.wave, [&](const WhereOf<G> &at, int i) { return marked<G, MODE>(reinterpret_cast<const float *>(sh.a), at, i); });
}

// ---------------------------------------------------------------------------------------------------------------
// Backward, query side: dq and D_i = dout_i . out_i (written for the key-side launch).
template <class G, int MODE>
__global__ void __launch_bounds__(G::NT, G::WAVES)
nattn_bwd_dq_patch(BandArgs a, const typename G::T *__restrict__ q, const typename G::T *__restrict__ k, const typename G::T *__restrict__ v,
                   const typename G::T *__restrict__ o_, const float *__restrict__ lse, const typename G::T *__restrict__ go,
                   typename G::T *__restrict__ dq, float *__restrict__ Dws)
{
    constexpr int D = G::D;
    using T = typename G::T;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    SharedDq<G, MODE> &sh = *reinterpret_cast<SharedDq<G, MODE> *>(lds);
    WhereOf<G> w;
    w.set(a);
    const int n = w.n, g = w.g, nd = MODE == kRagged ? a.d : D, ne = MODE == kRagged ? a.e : D;
    const bool vec = w.template own_pieces<MODE>();
    const float c2 = a.scale * kLog2e;
    const T *qs = q + size_t(w.bh) * nd * w.plane_own, *gs = go + size_t(w.bh) * ne * w.plane_own, *os = o_ + size_t(w.bh) * ne * w.plane_own;
    const T *ks = k + size_t(w.bh) * nd * w.plane_walk, *vs = v + size_t(w.bh) * ne * w.plane_walk;
    Place<G, MODE> at;
    at.init(w);
    Stage<G, MODE> rk, rv;
    rk.load_own(w, qs, nd, vec);
    rv.load_own(w, gs, ne, vec);
    Chunks<G, MODE> ch;
    ch.start(a, w, sh.rows);
    auto fetch = [&](int X0) {
        ch.set(X0, w, sh.rows);
        at.set(w, ch, sh.rows);
        rk.load(w, at, ks, nd);
        rv.load(w, at, vs, ne);
    };
    const int tr_at = G::start(4 * g + (n >> 2)), row_at = G::start(n);
    Stage<G, MODE> ro;
    ro.load_own(w, os, ne, vec);
    const size_t stat = size_t(w.bh) * w.plane_own + w.own_at + size_t(w.c_own) * (w.active ? w.u : 0);
    const float L2 = lse[stat] * kLog2e;         // the weights in the sums are relative ones: max omega multiplies the result
    __syncthreads();
    f32x4 part = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < G::NCO; ++j)
        if (MODE != kRagged || w.tid / G::OWN + j * G::NGO < ne) part += rv.value(j) * ro.value(j);
    Stage<G, MODE>::put_floats(w, sh.part[w.tid / G::OWN], part);
    rk.store_own(w, at, sh.a, nd);
    rv.store_own(w, at, sh.b, ne);
    __syncthreads();
    if (w.total > 0) fetch(0);
    const int slot = w.template own_slot<MODE>(here_v(w.lane) & 3, G::NW), point = 4 * w.template own_slot<MODE>(here_v(w.lane) >> 2 & 3, G::NW) + (n & 3);
    OwnPoint<G> oq, og;
    oq.read(sh.a + tr_at + 4 * slot);
    og.read(sh.b + tr_at + 4 * slot);
    float dsum = 0.f;
#pragma unroll
    for (int i = g; i < G::NGO; i += 4) dsum += sh.part[i][point];
    dsum = group_sum(dsum);
    if (w.active && w.lead && g == 0) Dws[stat] = dsum;
    Sums<G> acc;
    acc.zero();
    for (;;) {
        for (int X0 = 0; X0 < w.total; X0 += G::CAP) {
            __syncthreads();
            rk.store(at, sh.a, nd);
            rv.store(at, sh.b, ne);
            __syncthreads();
            const int list = ch.list, first = ch.first, end = ch.first + ch.cnt, ntile = (ch.cnt + 3) >> 2;
            if (X0 + G::CAP < w.total) fetch(X0 + G::CAP);
            auto step = [&](int t, auto count) {
                constexpr int N = decltype(count)::value;
                TileRef tr[2];
                float x[8];
#pragma unroll
                for (int i = 0; i < N; ++i) tr[i].template get<RowTab<MODE>::DEAD>(list, first + 4 * (t + i), end, n, g);
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    const uint2 arc = sh.rows.arc[w.sub][tr[i].row];
                    const f32x4 sc = dot<G>(sh.a + tr_at + 4 * tr[i].slot_n, oq), dp = dot<G>(sh.b + tr_at + 4 * tr[i].slot_n, og);
                    bool keep[4];
                    tr[i].keep(keep, w.su, arc.x);
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr) {
                        const float ds = __builtin_bit_cast(float, arc.y) * __builtin_amdgcn_exp2f(fmaf(sc[rr], c2, -L2)) * (dp[rr] - dsum);
                        x[4 * i + rr] = keep[rr] ? ds : 0.f;
                    }
                }
#pragma unroll
                for (int i = 4 * N; i < 8; ++i) x[i] = 0.f;
                bf16x8 p[kTerms];
                cut<true>(x, p);
                acc.add(sh.a + row_at + 4 * tr[0].slot, sh.a + row_at + 4 * tr[N - 1].slot, p);
            };
            int t = G::SPLIT ? w.tiles_from(ntile) : 0;
            const int t_end = G::SPLIT ? w.tiles_to(ntile) : ntile;
            for (; t + 1 < t_end; t += 2) step(t, std::integral_constant<int, 2>());
            if (t < t_end) step(t, std::integral_constant<int, 1>());
            acc.wait();
        }
        if (!w.more) break;
        ++w.seg;                           // more walked rows than the tables hold: the next part of them
        w.set_part(a);
        __syncthreads();
        ch.start(a, w, sh.rows);
        if (w.total > 0) fetch(0);
    }
    acc.join_terms();
    if (G::SPLIT && w.share_lg > 0) {
        float *tile = reinterpret_cast<float *>(sh.a);
        __syncthreads();
        put_shares<G, MODE>(acc.hi, tile, w);
        __syncthreads();
        add_shares<G, MODE>(acc.hi, tile, w);
    }
    unsigned again = not_finite(acc.hi, w.active && w.lead);
    if (any_owner(again)) again &= ~(own_nan(oq) | owner_bits(dsum != dsum || L2 != L2));       // (these are NaN throughout, as they are)
    __syncthreads();
    if (w.lead) put_results<G, MODE>(acc.hi, a.scale * a.omega_ref, again >> n & 1, reinterpret_cast<float *>(sh.a), w);
    __syncthreads();
    store_results<G, MODE>(dq + size_t(w.bh) * nd * w.plane_own, nd, reinterpret_cast<const float *>(sh.a), w, vec);
    exact_dq<T, WhereOf<G>>(again, w.wave, [&](const WhereOf<G> &at, int i) { return marked<G, MODE>(reinterpret_cast<const float *>(sh.a), at, i); });
}

// ---------------------------------------------------------------------------------------------------------------
// Backward, key side: owners are input points, the transposed band gives the output latitudes; q, dout, lse and D
// of a stage's outputs are staged together.
template <class G, int MODE>
__global__ void __launch_bounds__(G::NT, G::WAVES)
nattn_bwd_dkdv_patch(BandArgs a, const typename G::T *__restrict__ q, const typename G::T *__restrict__ k, const typename G::T *__restrict__ v,
                     const float *__restrict__ lse, const typename G::T *__restrict__ go, const float *__restrict__ Dws,
                     typename G::T *__restrict__ dk, typename G::T *__restrict__ dv)
{
    constexpr int D = G::D;
    using T = typename G::T;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    SharedDkdv<G, MODE> &sh = *reinterpret_cast<SharedDkdv<G, MODE> *>(lds);
    WhereOf<G> w;
    w.set(a);
    const int n = w.n, g = w.g, nd = MODE == kRagged ? a.d : D, ne = MODE == kRagged ? a.e : D;
    const bool vec = w.template own_pieces<MODE>();
    const float c2 = a.scale * kLog2e;
    const T *ks = k + size_t(w.bh) * nd * w.plane_own, *vs = v + size_t(w.bh) * ne * w.plane_own;
    const T *qs = q + size_t(w.bh) * nd * w.plane_walk, *gs = go + size_t(w.bh) * ne * w.plane_walk;
    const float *ls = lse + size_t(w.bh) * w.plane_walk, *Ds = Dws + size_t(w.bh) * w.plane_walk;
    // the quadrature weight is the owner's own here: it multiplies the finished sums (a latitude of weight zero has no arcs)
    const float omega = a.omega_rel[w.own / w.c_own] * a.omega_ref;
    Place<G, MODE> at;
    at.init(w);
    Stage<G, MODE> rq, rg;
    rq.load_own(w, ks, nd, vec);
    rg.load_own(w, vs, ne, vec);
    Chunks<G, MODE> ch;
    ch.start(a, w, sh.rows);
    f32x4 rs = {0.f, 0.f, 0.f, 0.f};         // first threads: logsumexp or D of a chunk
    auto fetch = [&](int X0) {
        ch.set(X0, w, sh.rows);
        at.set(w, ch, sh.rows);
        rq.load(w, at, qs, nd);
        rg.load(w, at, gs, ne);
        if constexpr (G::CJ == 1) {
            if (w.tid < 2 * G::CAP) rs = at.at[0].floats(w, at.cg ? Ds : ls, at.cg);
        } else if (w.wave < (2 * G::CAP + 63) / 64) {
            int row, col;
            ch.get(w.tid % G::CAP, w, sh.rows, row, col);
            typename Place<G, MODE>::At from;
            from.set(w, row, col, 0);
            if (w.tid < 2 * G::CAP) rs = from.floats(w, w.tid < G::CAP ? ls : Ds, 0);
        }
    };
    const int tr_at = G::start(4 * g + (n >> 2)), row_at = G::start(n);
    __syncthreads();
    rq.store_own(w, at, sh.a, nd);
    rg.store_own(w, at, sh.b, ne);
    __syncthreads();
    if (w.total > 0) fetch(0);
    const int slot = w.template own_slot<MODE>(here_v(w.lane) & 3, G::NW);
    OwnPoint<G> ok, ov;
    ok.read(sh.a + tr_at + 4 * slot);
    ov.read(sh.b + tr_at + 4 * slot);
    Sums<G> dka, dva;
    dka.zero();
    dva.zero();
    for (;;) {
        for (int X0 = 0; X0 < w.total; X0 += G::CAP) {
            __syncthreads();
            rq.store(at, sh.a, nd);
            rg.store(at, sh.b, ne);
            if (w.tid < 2 * G::CAP) {
                if (w.tid < G::CAP) *reinterpret_cast<f32x4 *>(sh.L + 4 * w.tid) = rs * -kLog2e;
                else *reinterpret_cast<f32x4 *>(sh.D + 4 * (w.tid - G::CAP)) = rs;
            }
            __syncthreads();
            const int list = ch.list, first = ch.first, end = ch.first + ch.cnt, ntile = (ch.cnt + 3) >> 2;
            if (X0 + G::CAP < w.total) fetch(X0 + G::CAP);
            auto step = [&](int t, auto count) {
                constexpr int N = decltype(count)::value;
                TileRef tr[2];
                float pr[8], ds[8];
#pragma unroll
                for (int i = 0; i < N; ++i) tr[i].template get<RowTab<MODE>::DEAD>(list, first + 4 * (t + i), end, n, g);
#pragma unroll
                for (int i = 0; i < N; ++i) {
                    const unsigned arc = sh.rows.arc[w.sub][tr[i].row].x;
                    const f32x4 L = *reinterpret_cast<const f32x4 *>(sh.L + 4 * tr[i].slot), Dn = *reinterpret_cast<const f32x4 *>(sh.D + 4 * tr[i].slot);
                    const f32x4 sc = dot<G>(sh.a + tr_at + 4 * tr[i].slot_n, ok), dp = dot<G>(sh.b + tr_at + 4 * tr[i].slot_n, ov);
                    bool keep[4];
                    tr[i].keep(keep, w.su, arc);
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr) {
                        const float x = __builtin_amdgcn_exp2f(fmaf(sc[rr], c2, L[rr]));
                        pr[4 * i + rr] = keep[rr] ? x : 0.f;
                        ds[4 * i + rr] = keep[rr] ? x * (dp[rr] - Dn[rr]) : 0.f;
                    }
                }
#pragma unroll
                for (int i = 4 * N; i < 8; ++i) pr[i] = ds[i] = 0.f;
                bf16x8 p[kTerms];
                cut<true>(pr, p);
                dva.add(sh.b + row_at + 4 * tr[0].slot, sh.b + row_at + 4 * tr[N - 1].slot, p);
                cut<true>(ds, p);
                dka.add(sh.a + row_at + 4 * tr[0].slot, sh.a + row_at + 4 * tr[N - 1].slot, p);
            };
            int t = G::SPLIT ? w.tiles_from(ntile) : 0;
            const int t_end = G::SPLIT ? w.tiles_to(ntile) : ntile;
            for (; t + 1 < t_end; t += 2) step(t, std::integral_constant<int, 2>());
            if (t < t_end) step(t, std::integral_constant<int, 1>());
            dka.wait();
            dva.wait();
        }
        if (!w.more) break;
        ++w.seg;                           // more walked rows than the tables hold: the next part of them
        w.set_part(a);
        __syncthreads();
        ch.start(a, w, sh.rows);
        if (w.total > 0) fetch(0);
    }
    dka.join_terms();
    dva.join_terms();
    if (G::SPLIT && w.share_lg > 0) {
        float *tile_k = reinterpret_cast<float *>(sh.a), *tile_v = reinterpret_cast<float *>(sh.b);
        __syncthreads();
        put_shares<G, MODE>(dka.hi, tile_k, w);
        put_shares<G, MODE>(dva.hi, tile_v, w);
        __syncthreads();
        add_shares<G, MODE>(dka.hi, tile_k, w);
        add_shares<G, MODE>(dva.hi, tile_v, w);
    }
    unsigned again_k = not_finite(dka.hi, w.active && w.lead), again_v = not_finite(dva.hi, w.active && w.lead);
    if (any_owner(again_k | again_v)) {
        const unsigned nan = own_nan(ok);                    // (these are NaN throughout, as they are)
        again_k &= ~(nan | own_nan(ov));
        again_v &= ~nan;
    }
    __syncthreads();
    if (w.lead) {
        put_results<G, MODE>(dka.hi, omega * a.scale, again_k >> n & 1, reinterpret_cast<float *>(sh.a), w);
        put_results<G, MODE>(dva.hi, omega, again_v >> n & 1, reinterpret_cast<float *>(sh.b), w);
    }
    __syncthreads();
    store_results<G, MODE>(dk + size_t(w.bh) * nd * w.plane_own, nd, reinterpret_cast<const float *>(sh.a), w, vec);
    store_results<G, MODE>(dv + size_t(w.bh) * ne * w.plane_own, ne, reinterpret_cast<const float *>(sh.b), w, vec);
    exact_dkdv<T, WhereOf<G>>(
        again_k | again_v, w.wave, [&](const WhereOf<G> &at, int i) { return marked<G, MODE>(reinterpret_cast<const float *>(sh.a), at, i); },
        [&](const WhereOf<G> &at, int i) { return marked<G, MODE>(reinterpret_cast<const float *>(sh.b), at, i); });
}

// Calls f with the geometry for a head dimension.  More workgroups on a compute unit count for more than longer stages (twice the
// chunks per stage: float32 d = 32 0.56 / 0.65 / 0.73 ms, bf16 d = 32 0.27 / 0.35 / 0.40); the register limits are the loosest that do not
// cost a workgroup, and the tightest that spill no more than a few registers (bf16 d = 32 at five
// wavefronts: forward 0.25 -> 0.24, dq 0.28 -> 0.26, dk/dv 0.34 -> 0.45 ms).  kHalves has the limits of kNarrow and spills 28 bytes of scratch in dq of
// float32 d = 32, 20 in that of d = 64 and 12 and 40 in dk/dv of bf16 d = 16 and 32; one wavefront less, 230 shapes, backward: float32 d = 32 1 % slower,
// bf16 d = 16 and 32 1 % faster.  Odd rows take more of them for addresses (128 x 254, 16 slices: dk/dv, float32 d = 16 held to four 0.235 ms, to three 0.217; bf16 d = 64 held to
// three 0.515, to two 0.429; bf16 d = 32 to four 0.214, to three 0.220).
// Stages of 24 chunks where that costs no workgroup, dk/dv of float32 d = 32: the four wavefronts of a workgroup meet more alike numbers of
// whole tiles in a stage and wait less for each other, and there are a third fewer stages (129 x 256, 32 slices: 659 -> 633 us; at three
// workgroups instead of four the forward would take 441 instead of 421, dq 521 instead of 498).  So it is where owners are three or more classes of a
// finer grid (192 x 384 -> 64 x 128, 8 slices: backward 299 us either way; 144 x 288 -> 36 x 72 185 -> 180); two classes are kPairs, whose owners
// meet some 38 chunks: 24 + 14 of them make more odd tiles than 16 + 16 + 6 (257 x 512 -> 129 x 256, 8 slices: 329 -> 350).
enum Launch { kFwd, kDq, kDkdv };
template <class T, int MODE, bool SPLIT, Launch WHICH, class F>
void by_shape(int dmax, F &&f)
{
    if constexpr (SPLIT) {
        constexpr bool F32 = sizeof(T) == 4;
        if (dmax <= 16) f(Geo<T, 16, 64, 2, true>());
        else if (dmax <= 32) f(Geo<T, 32, F32 ? 32 : 64, 2, true>());
        else f(Geo<T, 64, F32 ? 16 : 64, 2, true>());
    } else if constexpr (sizeof(T) == 4) {
        if (dmax <= 16) f(Geo<T, 16, 32, is_wide(MODE) && WHICH == kDkdv ? 4 : 3>());
        else if (dmax <= 32) {
            if constexpr (WHICH == kDkdv && MODE == kWide) f(Geo<T, 32, 24, 3>());
            else f(Geo<T, 32, 16, WHICH == kDq ? 4 : 3>());
        }
        else f(Geo<T, 64, 16, 2>());
    } else {
        if (dmax <= 16) f(Geo<T, 16, 64, 4>());
        else if (dmax <= 32) f(Geo<T, 32, 32, is_wide(MODE) && WHICH != kDkdv ? 5 : 4>());
        else f(Geo<T, 64, 32, !is_wide(MODE) && WHICH == kDkdv ? 2 : 3>());
    }
}
struct PatchLaunch {
    BandArgs a;
    dim3 grid;
};
inline PatchLaunch patch_launch(const S2DeviceTables &t, const S2BandSide &b, int nbh, int d, int e, float scale, const S2BandSide::Patches::Split *s)
{
    const S2BandSide::Patches &p = b.patches;
    const int n = s ? s->n : p.npatch;
    return {{b, t.omega_rel, t.ln_omega_ref, t.omega_ref, scale, nbh, d, e, p.seg, p.row_rec, s ? s->list : p.patch, n},
            dim3(unsigned(n) * unsigned(nbh))};
}
inline bool raise_lds(const void *f, size_t bytes) { return hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, int(bytes)) != hipSuccess; }

}  // namespace

template <class T, int MODE, bool SPLIT>
int PatchKernels<T, MODE, SPLIT>::configure()
{
    bool bad = false;
    for (int d : {16, 32, 64}) {
        by_shape<T, MODE, SPLIT, kFwd>(d, [&](auto g) { bad |= raise_lds(reinterpret_cast<const void *>(nattn_fwd_patch<decltype(g), MODE>), sizeof(Shared<decltype(g), MODE>)); });
        by_shape<T, MODE, SPLIT, kDq>(d, [&](auto g) { bad |= raise_lds(reinterpret_cast<const void *>(nattn_bwd_dq_patch<decltype(g), MODE>), sizeof(SharedDq<decltype(g), MODE>)); });
        by_shape<T, MODE, SPLIT, kDkdv>(d, [&](auto g) { bad |= raise_lds(reinterpret_cast<const void *>(nattn_bwd_dkdv_patch<decltype(g), MODE>), sizeof(SharedDkdv<decltype(g), MODE>)); });
    }
    return bad;
}
template <class T, int MODE, bool SPLIT>
void PatchKernels<T, MODE, SPLIT>::fwd(const S2DeviceTables &t, int nbh, int d, int e, float scale, const T *q, const T *k, const T *v, T *out, float *lse,
                                hipStream_t st)
{
    const PatchLaunch l = patch_launch(t, t.side_out, nbh, d, e, scale, SPLIT ? s2_split_list(t.side_out, nbh, d, e, sizeof(T), false) : nullptr);
    by_shape<T, MODE, SPLIT, kFwd>(d > e ? d : e, [&](auto g) {
        using G = decltype(g);
        hipLaunchKernelGGL((nattn_fwd_patch<G, MODE>), l.grid, dim3(G::NT), sizeof(Shared<G, MODE>), st, l.a, q, k, v, out, lse);
    });
}
template <class T, int MODE, bool SPLIT>
void PatchKernels<T, MODE, SPLIT>::dq(const S2DeviceTables &t, int nbh, int d, int e, float scale, const T *q, const T *k, const T *v, const T *o,
                               const float *lse, const T *go, T *dq, float *Dws, hipStream_t st)
{
    const PatchLaunch l = patch_launch(t, t.side_out, nbh, d, e, scale, SPLIT ? s2_split_list(t.side_out, nbh, d, e, sizeof(T), true) : nullptr);
    by_shape<T, MODE, SPLIT, kDq>(d > e ? d : e, [&](auto g) {
        using G = decltype(g);
        hipLaunchKernelGGL((nattn_bwd_dq_patch<G, MODE>), l.grid, dim3(G::NT), sizeof(SharedDq<G, MODE>), st, l.a, q, k, v, o, lse, go, dq, Dws);
    });
}
template <class T, int MODE, bool SPLIT>
void PatchKernels<T, MODE, SPLIT>::dkdv(const S2DeviceTables &t, int nbh, int d, int e, float scale, const T *q, const T *k, const T *v, const float *lse,
                                 const T *go, const float *Dws, T *dk, T *dv, hipStream_t st)
{
    const PatchLaunch l = patch_launch(t, t.side_in, nbh, d, e, scale, SPLIT ? s2_split_list(t.side_in, nbh, d, e, sizeof(T), true) : nullptr);
    by_shape<T, MODE, SPLIT, kDkdv>(d > e ? d : e, [&](auto g) {
        using G = decltype(g);
        hipLaunchKernelGGL((nattn_bwd_dkdv_patch<G, MODE>), l.grid, dim3(G::NT), sizeof(SharedDkdv<G, MODE>), st, l.a, q, k, v, lse, go, Dws, dk, dv);
    });
}
