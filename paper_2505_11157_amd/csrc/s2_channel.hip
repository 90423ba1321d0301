// Products with channel matrices (1x1 convolutions) of float32 tensors on the bf16 matrix cores (three terms per value, s2_bf16_terms.h;
// v_mfma_f32_32x32x16_bf16), shared by the attention sub-block and the DISCO convolution:
//   forward / input gradients   C[b][m][n] = sum_k A(m, k) X[b][k][n] + bias[m] + R[b][m][n]
//   weight gradients            dW[m][k] = sum_{b, n} dY[b][m][n] X[b][k][n],  dbias[m] = sum_{b, n} dY[b][m][n]
// One launch takes up to three products side by side (q, k and v from the same X), and a forward product may sum over up
// to three (matrix, tensor) pairs (the gradient that q, k and v send back to the same input).
#include <algorithm>
#include <type_traits>

#include "s2_bf16_terms.h"
#include "s2_internal.h"

namespace {

using namespace s2terms;

typedef __attribute__((ext_vector_type(16))) float f32x16;

__device__ __forceinline__ f32x16 mma32(bf16x8 a, bf16x8 b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }

template <int MT>
__device__ __forceinline__ bool not_finite(const f32x16 (&acc)[MT])
{
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) t = fmaf(acc[i][e], 0.f, t);
    return __builtin_expect(!(t == 0.f), 0);
}
// Sums that are not finite.  An infinite factor has terms that give NaN.  So a wavefront that meets such a sum sums its block once
// more over what is not finite about the factors (kinds: zero, +-1, +-infinity, NaN), which is a bf16 product as it stands: where that
// sum is not finite it is the result.  What is left, finite factors whose products overflow or that round to an infinite first term, the
// lane sums one by one.  (DISCO training step of 4 x 33 024 points, 64 to 64 channels, 0.59 ms: one infinite weight 16.3 ms with every
// such sum one by one, 0.84 this way; one NaN of x 3.9 and 0.68.)
__device__ __forceinline__ unsigned kind(float x)
{
    const unsigned u = __builtin_bit_cast(unsigned, x), a = u & 0x7fffffffu;
    return (u >> 16 & 0x8000u) | (a == 0u ? 0u : a < 0x7f800000u ? 0x3f80u : a == 0x7f800000u ? 0x7f80u : 0x7fc0u);
}
__device__ __forceinline__ bf16x8 kinds(const float (&x)[8])
{
    u32x4 u;
#pragma unroll
    for (int i = 0; i < 4; ++i) u[i] = kind(x[2 * i]) | kind(x[2 * i + 1]) << 16;
    return __builtin_bit_cast(bf16x8, u);
}
// the kinds of a block's sums over kinds, two bits each: 0, finite; 1, 2, infinite; 3, NaN
__device__ __forceinline__ unsigned kinds_of(const f32x16 &t)
{
    unsigned c = 0;
#pragma unroll
    for (int e = 0; e < 16; ++e) c |= (t[e] != t[e] ? 3u : t[e] == INFINITY ? 1u : t[e] == -INFINITY ? 2u : 0u) << 2 * e;
    return c;
}
// The sums with these kinds where they are not finite themselves; how many of them have finite factors (and hold nothing of use).
template <int MT>
__device__ __forceinline__ int explain(f32x16 (&acc)[MT], const unsigned (&codes)[MT])
{
    int left = 0;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const unsigned c = codes[i] >> 2 * e & 3u;
            const bool finite = fabsf(acc[i][e]) < INFINITY;
            left += !finite && c == 0u ? 1 : 0;
            acc[i][e] = finite ? acc[i][e] : c == 1u ? INFINITY : c == 2u ? -INFINITY : NAN;
        }
    return left;
}

// ---------------------------------------------------------------------------------------------------------------
// Products with a matrix.  A workgroup of four wavefronts owns 32 MT rows and 128 grid points; a wavefront owns 32 of
// the points and all the rows (MT accumulators).  The matrix goes through LDS in double-buffered slices of 16 along k, cut into
// its three terms on the way ([term][m][16 k], rows 48 bytes apart: the 16 rows that one 16-byte read serves together lie in
// different banks); X does not: lane (column, half) reads X[k0 + 8 half + j][n0 + column] straight into registers, a whole slice
// ahead of its use, every element once, in 128-byte row pieces, and cuts it there.
// Bound by the matrix cores (6 MT instructions of 32 cycles per slice and wavefront; eight fp32 ones of 64 cycles before) and, for
// few products of one X, by the memory X and the results pass through.  The rows per
// workgroup follow M, so 64-row products leave no half of a tile empty, and any k fits.  On the fp32 matrix cores
// before: 64 x 576 onto 4 x 33024 points 112 -> 82 us, three 128 x 128 products of one X 136 -> 101 us, their sum back 125 -> 92 us.
// (In a loop of whole layers part of that is lost: the card then lowers its clock, 2.37 -> 2.14 GHz with these products.)
constexpr int kSlice = 16;
constexpr int kRow = 24;                                   // bf16 values per row of a slice in LDS

// FAR: grids of so many points that a lane's offset takes more than 32 bits: up to 9 rows of X here, in bytes, the rows of a tile in the
// weight gradients, in values (with one row block only: such grids are few)
inline bool far_rows(int N, unsigned long long of_row) { return of_row * N >= 1ull << 32; }

template <bool TRANS, int MT, bool FAR = false>
__device__ __forceinline__ void product_strip(const S2ChannelProduct &a, int strip, int strips_per_batch, int set, int m0, __bf16 *lds)
{
    constexpr int MB = 32 * MT, PIECES = MB * kSlice / (TRANS ? 8 : 4), NP = (PIECES + 255) / 256, TERM = MB * kRow, BUF = kTerms * TERM;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, kk = lane >> 5;
    const int b = strip / strips_per_batch, n = (strip - b * strips_per_batch) * 128 + wave * 32 + col;
    const bool ok = n < a.N;
    using Offset = std::conditional_t<FAR, unsigned long long, unsigned>;
    Offset lane_off = (Offset(8 * kk) * unsigned(a.N) + unsigned(ok ? n : 0)) * 4u;      // past the last column: column 0, not stored
    asm volatile("" : "+v"(lane_off));
    const size_t step = size_t(a.N) * sizeof(float);
    const int M = a.M, K = a.K;

    // where the thread's pieces of a slice of the matrix (4 k of a row; TRANS: 2 k of 4 rows) come from (rows past M: the last
    // one, feeding results that are not stored) and go to
    float4 rw[NP][TRANS ? 2 : 1];
    unsigned w_off[NP], w_at[NP];
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        const int i = min(tid + 256 * j, PIECES - 1);
        if constexpr (TRANS) {
            const int k = 2 * (i / (8 * MT)), m = 4 * (i % (8 * MT));
            w_off[j] = unsigned(k) * unsigned(M) + unsigned(min(m0 + m, M - 4));
            w_at[j] = m * kRow + k;
        } else {
            const int m = i >> 2, k = 4 * (i & 3);
            w_off[j] = unsigned(min(m0 + m, M - 1)) * unsigned(K) + unsigned(k);
            w_at[j] = m * kRow + k;
        }
    }
    auto load_w = [&](const float *W) {
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            rw[j][0] = *reinterpret_cast<const float4 *>(W + w_off[j]);
            if constexpr (TRANS) rw[j][1] = *reinterpret_cast<const float4 *>(W + M + w_off[j]);
        }
    };
    auto store_w = [&](int buf) {
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            if (256 * (j + 1) > PIECES && tid + 256 * j >= PIECES) break;
            __bf16 *d = lds + buf * BUF + w_at[j];
            if constexpr (TRANS) {
                float x[4] = {rw[j][0].x, rw[j][0].y, rw[j][0].z, rw[j][0].w}, y[4] = {rw[j][1].x, rw[j][1].y, rw[j][1].z, rw[j][1].w};
#pragma unroll
                for (int t = 0; t < kTerms; ++t)
#pragma unroll
                    for (int i = 0; i < 4; ++i) *reinterpret_cast<unsigned *>(d + t * TERM + i * kRow) = cut_off(x[i], y[i]);
            } else {
                float x[4] = {rw[j][0].x, rw[j][0].y, rw[j][0].z, rw[j][0].w};
#pragma unroll
                for (int t = 0; t < kTerms; ++t) {
                    const unsigned lo = cut_off(x[0], x[1]), hi = cut_off(x[2], x[3]);
                    *reinterpret_cast<uint2 *>(d + t * TERM) = make_uint2(lo, hi);
                }
            }
        }
    };
    f32x16 acc[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;

    float xa[8], xb[8];
    auto fetch = [&](float (&x)[8], const char *r, size_t d) {
        // a uniform running row pointer plus one 32-bit lane offset, opaque so that no 64-bit address per load is kept;
        // explicitly global: a flat load also counts as an LDS access, and waits for LDS would wait for it.  (The pointer is in scalar
        // registers already where the compiler keeps it there by itself; it does not always.)
        const unsigned long long u = reinterpret_cast<unsigned long long>(r);
        const unsigned lo = __builtin_amdgcn_readfirstlane(unsigned(u)), hi = __builtin_amdgcn_readfirstlane(unsigned(u >> 32));
        r = reinterpret_cast<const char *>((unsigned long long)hi << 32 | lo);
        asm volatile("" : "+s"(r));
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            x[j] = *(const __attribute__((address_space(1))) float *)(r + lane_off);
            r += d;
        }
    };
    int seg = a.nset > 1 ? set : 0, k0 = 0, buf = 0;
    const int end = seg + (a.nset > 1 ? 1 : a.npair);
    const float *W = a.W[seg];
    const char *row = reinterpret_cast<const char *>(a.X[seg] + size_t(b) * K * a.N);
    load_w(W);
    fetch(xa, row, step);
    store_w(0);
    __syncthreads();
    auto advance = [&]() {
        if (k0 + kSlice < K) {
            k0 += kSlice;
            W += TRANS ? size_t(kSlice) * M : kSlice;
            row += kSlice * step;
            return true;
        }
        if (seg + 1 >= end) return false;
        k0 = 0;
        W = a.W[++seg];
        row = reinterpret_cast<const char *>(a.X[seg] + size_t(b) * K * a.N);
        return true;
    };
    // Nothing branches around the requests (the compiler would wait for all of them where the paths meet): behind the
    // last slice they go to one address, for nothing.
    auto slice = [&](float (&cur)[8], float (&nxt)[8]) {
        const bool more = advance();
        load_w(W);
        fetch(nxt, row, more ? step : 0);
        __builtin_amdgcn_sched_barrier(0);          // the requests stay in front of the arithmetic they overlap
        const __bf16 *wl = lds + buf * BUF + col * kRow + 8 * kk;
        bf16x8 x[kTerms];
        cut(cur, x);
        constexpr int order[6][2] = {{2, 0}, {0, 2}, {1, 1}, {1, 0}, {0, 1}, {0, 0}};      // smallest products first
#pragma unroll
        for (int i = 0; i < MT; ++i) {
            bf16x8 w[kTerms];
#pragma unroll
            for (int t = 0; t < kTerms; ++t) w[t] = *reinterpret_cast<const bf16x8 *>(wl + t * TERM + 32 * i * kRow);
#pragma unroll
            for (int p = 0; p < 6; ++p) acc[i] = mma32(w[order[p][0]], x[order[p][1]], acc[i]);
        }
        store_w(buf ^ 1);
        __syncthreads();
        buf ^= 1;
        return more;
    };
    while (slice(xa, xb) && slice(xb, xa)) {}
    const int begin = a.nset > 1 ? set : 0;
    int left = 0;
    if (__any(ok && not_finite(acc))) {
        const size_t xcol = ok ? n : 0;
        unsigned codes[MT] = {};
#pragma unroll 1
        for (int i = 0; i < MT; ++i) {
            f32x16 t = {0};
            const int m = min(m0 + 32 * i + col, M - 1);
#pragma unroll 1
            for (int s = begin; s < end; ++s)
#pragma unroll 1
                for (int k0 = 0; k0 < K; k0 += kSlice) {
                    float w[8], x[8];
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        const int k = k0 + 8 * kk + j;
                        w[j] = TRANS ? a.W[s][size_t(k) * M + m] : a.W[s][size_t(m) * K + k];
                        x[j] = a.X[s][(size_t(b) * K + k) * a.N + xcol];
                    }
                    t = mma32(kinds(w), kinds(x), t);
                }
            const unsigned c = kinds_of(t);
#pragma unroll
            for (int h = 0; h < MT; ++h) codes[h] = h == i ? c : codes[h];
        }
        left = explain(acc, codes);
    }
    if (!ok) return;
    if (left > 0) {
#pragma unroll 1
        for (int m = m0 + 4 * kk; m < min(m0 + MB, M); m = (m & 3) == 3 ? m + 5 : m + 1) {
            float t = 0.f;
            for (int i = begin; i < end; ++i)
                for (int k = 0; k < K; ++k)
                    t = fmaf(TRANS ? a.W[i][size_t(k) * M + m] : a.W[i][size_t(m) * K + k], a.X[i][(size_t(b) * K + k) * a.N + n], t);
            const size_t at = (size_t(b) * M + m) * a.N + n;
            a.C[set][at] = (t + (a.bias[set] ? a.bias[set][m] : 0.f)) + (a.R ? a.R[at] : 0.f);
        }
        return;
    }
    // per half row block all the reads (bias, residual) are issued before the first store, so that they overlap
    const float *bias = a.bias[set];
    float *Cb = a.C[set] + size_t(b) * M * a.N + n;
    const float *Rb = a.R ? a.R + size_t(b) * M * a.N + n : nullptr;
#pragma unroll
    for (int i = 0; i < 2 * MT; ++i) {
        if (m0 + 16 * i >= M) break;
        float add[8], res[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int m = m0 + 16 * i + 8 * (e >> 2) + 4 * kk + (e & 3);
            add[e] = bias ? bias[m] : 0.f;
            res[e] = Rb ? Rb[size_t(m) * a.N] : 0.f;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int m = m0 + 16 * i + 8 * (e >> 2) + 4 * kk + (e & 3);
            Cb[size_t(m) * a.N] = (acc[i >> 1][8 * (i & 1) + e] + add[e]) + res[e];
        }
    }
}

// Strips of the whole rounds of workgroups at MT row blocks, those of the last, partial round cut into single row blocks.
// The workgroups of one strip of X are eight apart: they run on the same die and share its L2.
template <bool TRANS, int MT, bool FAR = false>
__global__ void __launch_bounds__(256, MT == 1 && !FAR ? 8 : 4)
channel_product(S2ChannelProduct a, int strips_per_batch, int nstrips, int mblocks, int whole_groups)
{
    extern __shared__ __attribute__((aligned(16))) __bf16 lds[];
    const int parts = a.nset * mblocks, whole = whole_groups * 8 * parts, lo = blockIdx.x & 7;
    int id = blockIdx.x;
    if (id < whole || MT == 1) {
        id >>= 3;
        const int part = id % parts, strip = (id / parts) * 8 + lo;
        if (strip < nstrips)
            product_strip<TRANS, MT, FAR>(a, strip, strips_per_batch, part / mblocks, (part % mblocks) * 32 * MT, lds);
    } else {
        id = (id - whole) >> 3;
        const int part = id % (parts * MT), strip = (whole_groups + id / (parts * MT)) * 8 + lo, m0 = (part % (mblocks * MT)) * 32;
        if (strip < nstrips && m0 < a.M) product_strip<TRANS, 1>(a, strip, strips_per_batch, part / (mblocks * MT), m0, lds);
    }
}

// ---------------------------------------------------------------------------------------------------------------
// Weight gradients: partial sums over a share of (batch, grid point), added in a fixed order by a second launch, so every
// result is bit-reproducible.  A workgroup of WR x WN wavefronts owns 32 MT WR rows of dY and 32 WN rows of X, a
// wavefront 32 MT rows of dY and 32 of X; slices of 32 grid points (whole 128-byte lines of every row) are cut into three terms on
// their way to LDS: [term][half of the points][row][16 points], rows 48 bytes apart, so that the 16-byte operand reads are
// free of bank conflicts.  The next slice is on its way to the registers meanwhile.  The row sums of dY come from the pieces on
// their way to LDS.
// Bound by the matrix cores (12 MT instructions of 32 cycles per slice and wavefront; 16 fp32 ones of 64 cycles before) and the cutting.
// Rows per workgroup by M, columns by whichever width pads K least.  64 x 576 over 4 x 33024 points: as long as on
// the fp32 matrix cores (109 us; 12 wavefronts cut 256 rows for two of them on a compute unit), three 128 x 128: 135 -> 100 us.
constexpr int kPoints = 32;
constexpr int wgrad_lds(int rows) { return kTerms * 2 * rows * kRow * 2; }       // bytes of LDS

template <int MT, int WR, int WN, bool FAR = false>
__global__ void __launch_bounds__(64 * WR * WN)
channel_wgrad(S2ChannelGrad a, int ktiles, int mblocks, int nsplit, float *__restrict__ part)
{
    constexpr int YR = 32 * MT * WR, ROWS = YR + 32 * WN, NT = 64 * WR * WN, NP = (ROWS * 8 + NT - 1) / NT, NA = (YR * 8 + NT - 1) / NT;
    constexpr int HALF = ROWS * kRow, TERM = 2 * HALF;
    __shared__ __attribute__((aligned(16))) __bf16 lds[kTerms * TERM];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, kk = lane >> 5, M = a.M, K = a.K, N = a.N;
    const int wr = wave % WR, wn = wave / WR;
    // the tiles of one share of the points are eight workgroups apart: same die, same L2
    int id = blockIdx.x;
    const int slo = id & 7;
    id >>= 3;
    const int tiles = ktiles * mblocks * a.nset;
    int tile = id % tiles;
    const int split = (id / tiles) * 8 + slo;
    const int set = tile / (ktiles * mblocks);
    tile -= set * ktiles * mblocks;
    const int m0 = (tile / ktiles) * YR, k0 = (tile % ktiles) * 32 * WN;
    const int per = (N + kPoints - 1) / kPoints;
    const long slices = long(a.batch) * per;
    long s = slices * split / nsplit;
    const long s_end = slices * (split + 1) / nsplit;
    const float *dY = a.dY[set], *X = a.X[set];

    float4 r[NP];
    using Offset = std::conditional_t<FAR, unsigned long long, unsigned>;
    Offset off[NP];            // row inside the tile (rows past the end: the last one, feeding results that are not stored)
    float bsum[NA];
    const int pc = 4 * (tid & 7);
#pragma unroll
    for (int j = 0; j < NP; ++j) {
        const int row = min((tid >> 3) + (NT / 8) * j, ROWS - 1);
        off[j] = Offset(row < YR ? min(row, M - 1 - m0) : min(row - YR, K - 1 - k0)) * unsigned(N) + pc;
    }
#pragma unroll
    for (int j = 0; j < NA; ++j) bsum[j] = 0.f;
    bool in = false;           // is the piece inside the row (the last slice of a row may be half a slice)
    auto load = [&](long c) {
        const int b = int(c / per), n = int(c - long(b) * per) * kPoints;
        const float *y = dY + (size_t(b) * M + m0) * N + n, *x = X + (size_t(b) * K + k0) * N + n;
        in = n + pc < N;
        const int back = in ? 0 : pc;
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const bool isy = (tid >> 3) + (NT / 8) * j < YR;
            r[j] = *reinterpret_cast<const float4 *>((isy ? y : x) + (off[j] - back));
        }
    };
    auto store = [&]() {
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const int row = min((tid >> 3) + (NT / 8) * j, ROWS - 1);
            float4 v = r[j];
            if (!in) v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (j < NA) bsum[j < NA ? j : 0] += (v.x + v.y) + (v.z + v.w);
            __bf16 *d = lds + (pc >> 4) * HALF + row * kRow + (pc & 15);
#pragma unroll
            for (int t = 0; t < kTerms; ++t) {
                const unsigned lo = cut_off(v.x, v.y), hi = cut_off(v.z, v.w);
                *reinterpret_cast<uint2 *>(d + t * TERM) = make_uint2(lo, hi);
            }
        }
    };
    f32x16 acc[MT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
    if (s < s_end) load(s);
    for (; s < s_end; ++s) {
        __syncthreads();                    // everybody is done with the slice before
        store();
        __syncthreads();
        if (s + 1 < s_end) {
            load(s + 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        const __bf16 *sb = lds + col * kRow + 8 * kk, *ya = sb + wr * 32 * MT * kRow, *xa = sb + (YR + 32 * wn) * kRow;
        constexpr int order[6][2] = {{2, 0}, {0, 2}, {1, 1}, {1, 0}, {0, 1}, {0, 0}};      // smallest products first
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            bf16x8 x[kTerms];
#pragma unroll
            for (int t = 0; t < kTerms; ++t) x[t] = *reinterpret_cast<const bf16x8 *>(xa + t * TERM + q * HALF);
#pragma unroll
            for (int i = 0; i < MT; ++i) {
                bf16x8 y[kTerms];
#pragma unroll
                for (int t = 0; t < kTerms; ++t) y[t] = *reinterpret_cast<const bf16x8 *>(ya + t * TERM + q * HALF + 32 * i * kRow);
#pragma unroll
                for (int p = 0; p < 6; ++p) acc[i] = mma32(y[order[p][0]], x[order[p][1]], acc[i]);
            }
        }
    }
    float *P = part + (size_t(set) * nsplit + split) * (size_t(M) * K + M);
    const int k = k0 + 32 * wn + col;
    int left = 0;
    if (__any(k < K && not_finite(acc))) {
        unsigned codes[MT] = {};
#pragma unroll 1
        for (int i = 0; i < MT; ++i) {
            f32x16 t = {0};
            const int m = min(m0 + 32 * (MT * wr + i) + col, M - 1), kc = min(k, K - 1);
#pragma unroll 1
            for (long c = slices * split / nsplit; c < s_end; ++c) {
                const int b = int(c / per), n = int(c - long(b) * per) * kPoints;
                const float *y = dY + (size_t(b) * M + m) * N + 8 * kk, *x = X + (size_t(b) * K + kc) * N + 8 * kk;
#pragma unroll 1
                for (int p = n; p < min(n + kPoints, N); p += 16) {      // (N is a multiple of 16)
                    float yv[8], xv[8];
#pragma unroll
                    for (int j = 0; j < 8; ++j) {
                        yv[j] = y[p + j];
                        xv[j] = x[p + j];
                    }
                    t = mma32(kinds(yv), kinds(xv), t);
                }
            }
            const unsigned c = kinds_of(t);
#pragma unroll
            for (int h = 0; h < MT; ++h) codes[h] = h == i ? c : codes[h];
        }
        left = explain(acc, codes);
    }
    if (k < K && left > 0) {
#pragma unroll 1
        for (int i = 0; i < 16 * MT; ++i) {
            const int m = m0 + 32 * (MT * wr + (i >> 4)) + 8 * (i >> 2 & 3) + 4 * kk + (i & 3);
            if (m >= M) continue;
            float t = 0.f;
            for (long c = slices * split / nsplit; c < s_end; ++c) {
                const int b = int(c / per), n = int(c - long(b) * per) * kPoints;
                const float *y = dY + (size_t(b) * M + m) * N, *x = X + (size_t(b) * K + k) * N;
                for (int p = n; p < min(n + kPoints, N); ++p) t = fmaf(y[p], x[p], t);
            }
            P[size_t(m) * K + k] = t;
        }
    } else if (k < K) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int m = m0 + 32 * (MT * wr + i) + 8 * (e >> 2) + 4 * kk + (e & 3);
                if (m < M) P[size_t(m) * K + k] = acc[i][e];
            }
    }
    if (k0 == 0) {
#pragma unroll
        for (int j = 0; j < NA; ++j) {
            float t = bsum[j];
            t += __shfl_xor(t, 1);
            t += __shfl_xor(t, 2);
            t += __shfl_xor(t, 4);
            const int row = (tid >> 3) + (NT / 8) * j;
            if ((tid & 7) == 0 && row < YR && m0 + row < M) P[size_t(M) * K + m0 + row] = t;
        }
    }
}

// Adds the partials of element i in order.  A workgroup owns 64 elements; thread (q, e) adds the partials q, q + 4,
// q + 8, ... of element e (four chains of loads in flight per element), then the four sums are added.
__global__ void __launch_bounds__(256)
channel_sum_partials(S2ChannelGrad a, int nsplit, const float *__restrict__ part)
{
    __shared__ float red[4][64];
    const int e = threadIdx.x & 63, q = threadIdx.x >> 6, set = blockIdx.y;
    const size_t MK = size_t(a.M) * a.K, count = MK + a.M, i = size_t(blockIdx.x) * 64 + e;
    const float *p0 = part + size_t(set) * nsplit * count + i;
    float s = 0.f;
    if (i < count) {
#pragma unroll 8
        for (int p = q; p < nsplit; p += 4) s += p0[size_t(p) * count];
    }
    red[q][e] = s;
    __syncthreads();
    if (q != 0 || i >= count) return;
    const float t = (red[0][e] + red[1][e]) + (red[2][e] + red[3][e]);
    if (i < MK) {
        if (a.dW[set]) a.dW[set][i] = t;
    } else if (a.dbias[set]) {
        a.dbias[set][i - MK] = t;
    }
}

// 32-row blocks per workgroup: all of M up to 128 rows, else the block size that pads M least (the larger one on a tie)
inline int row_blocks(int M)
{
    if (M <= 128) return (M + 31) / 32;
    int best = 4;
    for (int mt = 3; mt >= 2; --mt)
        if ((M + 32 * mt - 1) / (32 * mt) * mt < (M + 32 * best - 1) / (32 * best) * best) best = mt;
    return best;
}
// Weight gradients: wavefronts per workgroup side by side.  Two row blocks take one each (three pairs, two or one: the
// width that pads K least, the largest on a tie), so that the number of wavefronts is a multiple of four and every SIMD
// gets the same share; otherwise one wavefront takes all the row blocks, four of them side by side.
inline int col_waves(int mt, int K)
{
    if (mt != 2) return 4;
    int best = 6;
    for (int wn = 4; wn >= 2; wn -= 2)
        if ((K + 32 * wn - 1) / (32 * wn) * wn < (K + 32 * best - 1) / (32 * best) * best) best = wn;
    return best;
}
struct GradPlan { int mt, wn, mblocks, ktiles, nsplit; };
// Splits: as many workgroups over all products of the launch as are resident at once (by their LDS), in multiples of eight
// (one per die).
inline GradPlan grad_plan(int M, int K, int nset)
{
    GradPlan p;
    p.mt = row_blocks(M);
    p.wn = col_waves(p.mt, K);
    p.mblocks = (M + 32 * p.mt - 1) / (32 * p.mt);
    p.ktiles = (K + 32 * p.wn - 1) / (32 * p.wn);
    const int lds = wgrad_lds(32 * (p.mt + p.wn)), want = 256 * std::min(4, 160 * 1024 / lds);
    p.nsplit = std::max(8, want / (p.mblocks * p.ktiles * nset) / 8 * 8);
    return p;
}

}  // namespace

void s2_channel_product(bool trans, const S2ChannelProduct &a, hipStream_t st)
{
    const bool far = far_rows(a.N, 9 * sizeof(float));
    const int mt = far ? 1 : row_blocks(a.M), mblocks = (a.M + 32 * mt - 1) / (32 * mt), spb = (a.N + 127) / 128, nstrips = spb * a.batch;
    // Four workgroups per compute unit (eight with one row block), held to by the LDS they ask for: with room for more the
    // dispatcher fills some units with five and leaves others three.
    const int occ = mt == 1 ? 8 : 4, parts = mblocks * a.nset, round = 256 * occ, groups = (nstrips + 7) / 8;
    const int per_round = std::max(1, round / (8 * parts)), rest = groups % per_round;
    const bool split = mt > 1 && rest * 8 * parts * mt <= round;
    const int whole = split ? groups - rest : groups;
    const dim3 grid(unsigned(whole + (groups - whole) * mt) * 8 * parts);
    const size_t lds = mt == 1 ? 19 * 1024 : 38 * 1024;
#define S2_PRODUCT(T, ...) hipLaunchKernelGGL((channel_product<T, __VA_ARGS__>), grid, dim3(256), lds, st, a, spb, nstrips, mblocks, whole)
    switch (far ? trans - 1 : mt + (trans ? 4 : 0)) {
    case -1: S2_PRODUCT(false, 1, true); break;
    case 0: S2_PRODUCT(true, 1, true); break;
    case 1: S2_PRODUCT(false, 1); break;
    case 2: S2_PRODUCT(false, 2); break;
    case 3: S2_PRODUCT(false, 3); break;
    case 4: S2_PRODUCT(false, 4); break;
    case 5: S2_PRODUCT(true, 1); break;
    case 6: S2_PRODUCT(true, 2); break;
    case 7: S2_PRODUCT(true, 3); break;
    default: S2_PRODUCT(true, 4); break;
    }
#undef S2_PRODUCT
}

size_t s2_channel_grad_floats(int M, int K, int nset)
{
    return size_t(nset) * grad_plan(M, K, nset).nsplit * (size_t(M) * K + M);
}

void s2_channel_grad(const S2ChannelGrad &a, float *part, hipStream_t st)
{
    GradPlan p = grad_plan(a.M, a.K, a.nset);
    const bool far = far_rows(a.N, 32 * std::max(p.mt, p.wn));
    if (far) {                                   // (the splits, and with them the partial sums, stay)
        p.mt = 1;
        p.wn = 4;
        p.mblocks = (a.M + 31) / 32;
        p.ktiles = (a.K + 127) / 128;
    }
    const dim3 grid(unsigned(p.ktiles) * p.mblocks * a.nset * p.nsplit);
#define S2_GRAD(MT, WR, WN, ...) \
    hipLaunchKernelGGL((channel_wgrad<MT, WR, WN, ##__VA_ARGS__>), grid, dim3(64 * WR * WN), 0, st, a, p.ktiles, p.mblocks, p.nsplit, part)
    if (far) S2_GRAD(1, 1, 4, true);
    else if (p.mt == 1) S2_GRAD(1, 1, 4);
    else if (p.mt == 2 && p.wn == 2) S2_GRAD(1, 2, 2);
    else if (p.mt == 2 && p.wn == 4) S2_GRAD(1, 2, 4);
    else if (p.mt == 2) S2_GRAD(1, 2, 6);
    else if (p.mt == 3) S2_GRAD(3, 1, 4);
    else S2_GRAD(4, 1, 4);
#undef S2_GRAD
    const size_t count = size_t(a.M) * a.K + a.M;
    hipLaunchKernelGGL(channel_sum_partials, dim3(unsigned((count + 63) / 64), a.nset), dim3(256), 0, st, a, p.nsplit, part);
}
