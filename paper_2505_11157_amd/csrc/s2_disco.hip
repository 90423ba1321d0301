// Discrete-continuous (DISCO) convolution on the sphere (App. B.3, first equation), float32, on the same compact
// form of the indicator as the attention kernels: for output latitude h the disk meets the input latitudes of its
// band in arcs of consecutive longitude offsets, and the filter basis is tabulated per (h, band row, offset):
//     z[b, c, k, h, w] = sum_{h', w'} psi_k[h, h', w'] x[b, c, h', (w' + w pscale) mod nlon_in]
//     y[b, o, h, w]    = sum_{c, k} weight[o, c, k] z[b, c, k, h, w] + bias[o]
// psi_k = hat_k(r) * omega[h'] with K piecewise-linear hats of the geodesic distance r (hat_k(r) = max(0,
// 1 - |r K / theta_cutoff - k|): isotropic filters that vanish on the rim of the disk); the paper leaves the basis
// open.  The contraction with psi is disco_gather below; grids with too many input columns per output column for it take a gather
// per point (lanes on consecutive longitudes, the basis values of a (latitude, offset) uniform over a wavefront).  The channel mixing is a
// channel matrix on the matrix cores.  Backward: psi is applied to dy through the transposed
// neighborhood (the same kernel on the transposed tables, no atomics) and the channel mixing follows,
//     dx[b, c] = sum_{o, k} weight[o, c, k] (psi_k^T dy)[b, o];
// or, where that is cheaper (transposed_first), the channels are mixed first and psi^T gathers dx from the K planes of dz
// (disco_gather_planes).  dweight is the split-K weight-gradient product summed in a fixed order.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <initializer_list>
#include <map>
#include <new>
#include <utility>

#include "s2_nattn_kernels.h"

namespace {

// One direction of the contraction with psi as disco_gather walks it: for every group of kGroup owner latitudes a list of
// chunks, a chunk being some rows (or parts of long ones) that fit into a workgroup's share of LDS and, for each latitude of
// the group, the (row, offset) entries on them, sorted by the interval j <= r K / theta < j + 1 in which only the hats j and
// j + 1 differ from zero.
constexpr int kGroup = 4;
struct GatherPiece {                  // 64 (W + 1) staged columns of a row at most: i0 .. i0 + n - 1 of it
    int lat, left;                    // walked latitude, staged columns in front of the first owner's (may be negative)
    int i0, n;
    int base, sub;                    // the row's LDS position, its columns of one remainder mod P
    int pad[2];
};
struct GatherEntry {
    int plus, minus;                  // LDS byte offsets of the columns +d and -d of owner 0
    float lo, hi;                     // psi_j, psi_{j+1} (halved where +d and -d are the same column)
};
struct GatherTables {
    void *blob = nullptr;
    const int *chunk_of = nullptr;    // [groups + 1]
    const int *chunk = nullptr;       // [chunks][2 + kGroup (K + 1)]: first piece, end piece; per latitude: first entry, end of interval j
    const GatherPiece *piece = nullptr;
    const GatherEntry *entry = nullptr;
    const int *order = nullptr;       // groups, heaviest first
    int lds_bytes = 0, W = 1;         // 0: not available; owners per lane
};

// The same contraction summed over the K planes (disco_gather_planes): per owner latitude a list of terms, padded to whole
// batches for the four wavefronts of a workgroup.
struct PlaneTerm {
    long at;                          // plane j and walked latitude, as an offset into the K planes of one channel
    int plus, minus;                  // walked columns of owner 0, in 0 .. columns - 1
    float w;                          // psi_j (halved where both columns are the same one)
    int pad;
};
struct PlaneTables {
    void *blob = nullptr;
    const int *first = nullptr;       // [owner latitudes + 1]
    const PlaneTerm *term = nullptr;
    const int *order = nullptr;       // owner latitudes, heaviest first
};

}  // namespace

struct s2_disco {
    const s2_grid_t *g;
    int K;
    float *dev_psi = nullptr;     // [entry][KP], KP = K rounded up to a multiple of 4; entry = poff[h * band_max + b] + offset
    int *dev_poff = nullptr;      // [nlat_out * band_max]
    GatherTables fwd, bwd;        // owners = outputs; owners = inputs
    PlaneTables planes;           // owners = inputs
    int compute_units = 256;
};

namespace {

constexpr int kMaxBasis = 16;     // a 4 x 4 planar kernel's worth of basis functions (App. C)

__device__ __forceinline__ int wrapn(int x, int n)
{
    x = x < 0 ? x + n : x;
    return x >= n ? x - n : x;
}

// z[bc][k][h][w]: one lane per output point, block -> (64 longitudes, latitude, bc).  KP: the basis count rounded up to
// a multiple of four; the basis table holds KP values per arc offset (zeros behind the K-th).
template <int KP>
__global__ void __launch_bounds__(64)
disco_z_fwd(S2DeviceTables t, const float *__restrict__ psi, const int *__restrict__ poff, int K,
            const float *__restrict__ x, float *__restrict__ z)
{
    const int w = blockIdx.x * 64 + threadIdx.x, h = blockIdx.y, bc = blockIdx.z;
    if (w >= t.nlon_out) return;
    const size_t si = size_t(t.nlat_in) * t.nlon_in, so = size_t(t.nlat_out) * t.nlon_out;
    float acc[KP];
#pragma unroll
    for (int k = 0; k < KP; ++k) acc[k] = 0.f;
    const int nb = t.band_n[h], hp0 = t.band_lo[h];
    for (int b = 0; b < nb; ++b) {
        const int c = t.cnt[h * t.band_max + b];
        const int first = w * t.pscale + (c == t.nlon_in ? 0 : -((c - 1) >> 1));
        const float *xr = x + size_t(bc) * si + size_t(hp0 + b) * t.nlon_in;
        const float *pr = psi + size_t(poff[h * t.band_max + b]) * KP;
        int col = wrapn(first, t.nlon_in);
        for (int tt = 0; tt < c; ++tt) {
            const float xv = xr[col];
#pragma unroll
            for (int k = 0; k < KP; ++k) acc[k] = fmaf(pr[tt * KP + k], xv, acc[k]);
            col = col + 1 == t.nlon_in ? 0 : col + 1;
        }
    }
#pragma unroll
    for (int k = 0; k < KP; ++k)
        if (k < K) z[(size_t(bc) * K + k) * so + size_t(h) * t.nlon_out + w] = acc[k];
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Contraction with psi: out[ch][k][lat][u] = sum over the entries of owner latitude lat.  At a distance r only two of the K
// hats differ from zero, and the columns +d and -d of a row carry the same values, so two neighbors cost one add and two
// multiply-adds per channel instead of 2 K multiply-adds (a dense contraction with the basis on the matrix cores, 16 rows
// for 9 functions, took 0.62 ms on 129 x 256 with 4 x 64 channels).  Which two accumulators an entry goes to is known at
// compile time: the entries of a chunk are sorted by interval and the loop over the intervals is unrolled.
// One workgroup: 64 W consecutive owners of four neighboring latitudes, one each for its wavefronts, and four channels.
// Neighboring latitudes meet nearly the same rows, so the rows are staged once for the four, and a latitude's entries come in
// one or two chunks, in fewer and longer runs of one interval, than where a wavefront stages for itself.  129 x 256 with 4 x 64
// channels, K = 9: 180 us that way, 171 us in groups, 157 us with the LDS reads of two entries waiting together.  Bound there:
// the 16-byte LDS reads (80 us at 128 bytes a clock and compute unit; two neighbors of four channels each take 32 bytes, whatever
// the order) and behind them, hardly overlapped, the staging (13 us), the results (30 us) and the runs' starts (19 us); the
// polar groups, one workgroup of 55 us, are started first.  More than one quad of channels to a workgroup: 168 us and up.
// Staged position-major with the four channels of a column side by side, so that a neighbor is one 16-byte LDS read per lane at
// consecutive addresses; with P walked columns per owner the columns of one remainder mod P lie together, and where the owner
// grid is the finer one (C owner columns per walked column) the owner latitudes are its classes of every C-th column.  Entries and basis
// values are uniform and come through the scalar cache.
template <int K, int W>
__global__ void __launch_bounds__(64 * kGroup, 3)
disco_gather(GatherTables t, int P, int C, int nlon_own, int nlon_walk, int nlat_own, int nlat_walk, int nch,
             const float *__restrict__ x, float *__restrict__ out)
{
    // 168 registers at three wavefronts a SIMD (what LDS holds): pieces under way, and whether two entries' values fit
    constexpr int kFree = (112 - 4 * K * W) / (4 * (W + 1)), D = kFree < 1 ? 1 : kFree > 4 ? 4 : kFree;
    constexpr bool kTwo = 4 * K * W <= 104;
    extern __shared__ __attribute__((aligned(16))) f32x4 xs[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ntile = (nlon_own + 64 * W - 1) / (64 * W), nquad = (nch + 3) / 4;
    int id = blockIdx.x;
    const int tile = id % ntile; id /= ntile;
    const int quad = id % nquad, grp = t.order[id / nquad], lat = grp * kGroup + wave;
    const int u0 = tile * 64 * W;
    const float inv_walk = 1.f / float(nlon_walk), inv_p = 1.f / float(P);
    const size_t plane_walk = size_t(nlat_walk) * nlon_walk, plane_own = size_t(nlat_own / C) * nlon_own * C;
    const float *xc[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) xc[c] = x + size_t(min(4 * quad + c, nch - 1)) * plane_walk;

    f32x4 acc[K][W];
#pragma unroll
    for (int k = 0; k < K; ++k)
#pragma unroll
        for (int i = 0; i < W; ++i) acc[k][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    // The pieces of a chunk are dealt out to the wavefronts.  (x + 1/2) / n in float32 has the right whole part here: x stays
    // within some thousand columns above the circle's.
    float v[D][W + 1][4];                                // pieces under way from memory
    auto request = [&](int piece, int end) {
#pragma unroll
        for (int s = 0; s < D; ++s) {
            if (piece + s * kGroup >= end) break;
            const GatherPiece m = t.piece[piece + s * kGroup];
            const size_t at = size_t(m.lat) * nlon_walk;
            int first = u0 * P - m.left;                 // in (-nlon, 2 nlon)
            first = (first < 0 ? first + nlon_walk : first) + m.i0;
#pragma unroll
            for (int b = 0; b <= W; ++b) {
                int col = first + min(64 * b + lane, m.n - 1);
                col -= __mul24(int((float(col) + 0.5f) * inv_walk), nlon_walk);
#pragma unroll
                for (int c = 0; c < 4; ++c) v[s][b][c] = xc[c][at + col];
            }
        }
    };
    auto place = [&](int piece, int end) {
#pragma unroll
        for (int s = 0; s < D; ++s) {
            if (piece + s * kGroup >= end) break;
            const GatherPiece m = t.piece[piece + s * kGroup];
#pragma unroll
            for (int b = 0; b <= W; ++b) {
                const int i = m.i0 + 64 * b + lane, q = int((float(i) + 0.5f) * inv_p);
                if (64 * b + lane < m.n) xs[m.base + __mul24(i - __mul24(q, P), m.sub) + q] = f32x4{v[s][b][0], v[s][b][1], v[s][b][2], v[s][b][3]};
            }
        }
    };
    const char *lds = reinterpret_cast<const char *>(xs) + 16 * lane;
    constexpr int kChunk = 2 + kGroup * (K + 1);
    const int c_end = t.chunk_of[grp + 1];
    for (int ci = t.chunk_of[grp]; ci < c_end; ++ci) {
        const int *ch = t.chunk + size_t(ci) * kChunk, p_end = ch[1];
        int p = ch[0] + wave;
        request(p, p_end);
        __syncthreads();                                 // the reads of the previous chunk are done
        place(p, p_end);
        for (p += D * kGroup; p < p_end; p += D * kGroup) {
            request(p, p_end);
            place(p, p_end);
        }
        __syncthreads();
        ch += 2 + wave * (K + 1);
        int e = ch[0];
        GatherEntry n0 = t.entry[e], n1 = t.entry[e + 1];        // two ahead (the table ends with two spare entries)
#pragma unroll
        for (int j = 0; j < K; ++j) {
            const int e_end = ch[1 + j];
            auto add = [&](const GatherEntry &en, const f32x4 &a, const f32x4 &b, int i) {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const float s = a[c] + b[c];
                    acc[j][i][c] = fmaf(en.lo, s, acc[j][i][c]);
                    if (j + 1 < K) acc[j + 1 < K ? j + 1 : 0][i][c] = fmaf(en.hi, s, acc[j + 1 < K ? j + 1 : 0][i][c]);
                }
            };
            auto at = [&](int pos, int i) { return *reinterpret_cast<const f32x4 *>(lds + pos + 1024 * i); };
            for (; kTwo && e + 1 < e_end; e += 2) {              // two at a time: their LDS reads wait together
                const GatherEntry e0 = n0, e1 = n1;
                f32x4 a0[W], b0[W], a1[W], b1[W];
#pragma unroll
                for (int i = 0; i < W; ++i) {
                    a0[i] = at(e0.plus, i);
                    b0[i] = at(e0.minus, i);
                }
#pragma unroll
                for (int i = 0; i < W; ++i) {
                    a1[i] = at(e1.plus, i);
                    b1[i] = at(e1.minus, i);
                }
                n0 = t.entry[e + 2];
                n1 = t.entry[e + 3];
#pragma unroll
                for (int i = 0; i < W; ++i) add(e0, a0[i], b0[i], i);
#pragma unroll
                for (int i = 0; i < W; ++i) add(e1, a1[i], b1[i], i);
            }
            for (; e < e_end; ++e) {
                const GatherEntry en = n0;
                n0 = n1;
                n1 = t.entry[e + 2];
#pragma unroll
                for (int i = 0; i < W; ++i) add(en, at(en.plus, i), at(en.minus, i), i);
            }
        }
    }
    if (lat >= nlat_own) return;
#pragma unroll
    for (int i = 0; i < W; ++i) {
        const int u = u0 + 64 * i + lane;
        if (u >= nlon_own) continue;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            if (4 * quad + c >= nch) continue;
            float *o = out + size_t(4 * quad + c) * K * plane_own + size_t(lat / C) * nlon_own * C + lat % C + size_t(C) * u;
#pragma unroll
            for (int k = 0; k < K; ++k) o[size_t(k) * plane_own] = acc[k][i][c];
        }
    }
}

// dx[ch][lat][u] = sum over the terms of owner latitude lat of w (dz[plane j][plus + u] + dz[plane j][minus + u]): each hat
// reads a plane of its own here, so a neighbor costs up to four loads per channel where disco_gather has two LDS reads, and
// nothing is worth staging (a staged row would serve some two terms per plane).  Loads are coalesced over the owners and hit
// the caches; a workgroup's four wavefronts share 64 owners and four channels and take a quarter of the terms each (a polar
// owner has a thousand), four terms in flight at a time.
template <int CH>
__global__ void __launch_bounds__(256)
disco_gather_planes(PlaneTables t, int C, size_t planes, int nlon_own, int nlon_walk, size_t plane_own, int nch, const float *__restrict__ dz,
                    float *__restrict__ dx)
{
    constexpr int B = 4;
    __shared__ float part[3][CH][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ntile = (nlon_own + 63) / 64, ngrp = (nch + CH - 1) / CH;
    int id = blockIdx.x;
    const int u = (id % ntile) * 64 + lane; id /= ntile;
    const int ch = id % ngrp * CH, lat = t.order[id / ngrp];
    const int uc = u < nlon_own ? u : nlon_own - 1;
    const float *x[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) x[c] = dz + size_t(min(ch + c, nch - 1)) * planes;
    float acc[CH] = {};
    const int first = t.first[lat], quarter = (t.first[lat + 1] - first) / 4;         // a multiple of B
    for (int e = first + wave * quarter, end = e + quarter; e < end; e += B) {
        float v[B][CH];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const PlaneTerm m = t.term[e + b];
            int p = uc + m.plus, q = uc + m.minus;
            p = p >= nlon_walk ? p - nlon_walk : p;
            q = q >= nlon_walk ? q - nlon_walk : q;
#pragma unroll
            for (int c = 0; c < CH; ++c) v[b][c] = x[c][m.at + p] + x[c][m.at + q];
        }
#pragma unroll
        for (int b = 0; b < B; ++b)
#pragma unroll
            for (int c = 0; c < CH; ++c) acc[c] = fmaf(t.term[e + b].w, v[b][c], acc[c]);
    }
    if (wave > 0)
#pragma unroll
        for (int c = 0; c < CH; ++c) part[wave - 1][c][lane] = acc[c];
    __syncthreads();
    if (wave > 0 || u >= nlon_own) return;
#pragma unroll
    for (int c = 0; c < CH; ++c)
        if (ch + c < nch)
            dx[size_t(ch + c) * plane_own + size_t(lat / C) * nlon_own * C + lat % C + size_t(C) * u] =
                acc[c] + part[0][c][lane] + part[1][c][lane] + part[2][c][lane];
}

// weight[o][c][k] -> wt[c][o][k], the channel matrix that follows the transposed contraction
__global__ void __launch_bounds__(256)
disco_weight_transpose(int cout, int cin, int K, const float *__restrict__ w, float *__restrict__ wt)
{
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= cout * cin * K) return;
    const int k = i % K, o = i / K % cout, c = i / K / cout;
    wt[i] = w[(o * cin + c) * K + k];
}

int check(const s2_disco_t *dc, int batch, int cin, int cout, const void *ws, size_t ws_bytes)
{
    if (!dc) return s2_fail(S2_ERR_INVALID_ARG, "disco handle is NULL");
    if (batch < 1 || cin < 1 || cout < 1) return s2_fail(S2_ERR_INVALID_ARG, "batch and channel counts must be >= 1");
    const size_t n_out = size_t(dc->g->nlat_out) * dc->g->nlon_out;
    if ((cin * dc->K) % 16 != 0 || cout % 16 != 0 || n_out % 16 != 0)
        return s2_fail(S2_ERR_UNSUPPORTED, "channels_in * nbasis, channels_out and the number of output points must be multiples of 16");
    if (long(batch) * cin > 65535) return s2_fail(S2_ERR_INVALID_ARG, "batch * channels_in too large");
    if (!ws || reinterpret_cast<uintptr_t>(ws) % 256 != 0 || ws_bytes < s2_disco_workspace_bytes(dc, batch, cin, cout))
        return s2_fail(S2_ERR_WORKSPACE, "workspace missing, not 256-byte aligned or smaller than s2_disco_workspace_bytes()");
    return S2_OK;
}

inline int padded(int K) { return (K + 3) / 4 * 4; }

template <class F>
void by_basis(int K, F f)       // f(KP), KP = the basis count rounded up to a multiple of four
{
    if (K <= 4) f(std::integral_constant<int, 4>());
    else if (K <= 8) f(std::integral_constant<int, 8>());
    else if (K <= 12) f(std::integral_constant<int, 12>());
    else f(std::integral_constant<int, 16>());
}

template <int K = 1, class F>
void by_count(int n, F &&f)       // f(K) for the basis count n = 1 .. kMaxBasis
{
    if (n == K) return f(std::integral_constant<int, K>());
    if constexpr (K < kMaxBasis) by_count<K + 1>(n, f);
}

void launch_gather(const GatherTables &t, int K, int P, int C, int nlon_own, int nlon_walk, int nlat_own, int nlat_walk, int nch,
                   const float *x, float *out, hipStream_t st)
{
    const unsigned blocks = unsigned((nlon_own + 64 * t.W - 1) / (64 * t.W)) * unsigned((nch + 3) / 4) *
                            unsigned((nlat_own + kGroup - 1) / kGroup);
    by_count(K, [&](auto k) {
        constexpr int KK = decltype(k)::value;
        if (t.W == 2)
            hipLaunchKernelGGL((disco_gather<KK, 2>), dim3(blocks), dim3(64 * kGroup), size_t(t.lds_bytes), st, t, P, C, nlon_own, nlon_walk,
                               nlat_own, nlat_walk, nch, x, out);
        else
            hipLaunchKernelGGL((disco_gather<KK, 1>), dim3(blocks), dim3(64 * kGroup), size_t(t.lds_bytes), st, t, P, C, nlon_own, nlon_walk,
                               nlat_own, nlat_walk, nch, x, out);
    });
}

// arrays one behind the other in device memory: array i at off[i]
int upload(void *&blob, size_t *off, std::initializer_list<std::pair<const void *, size_t>> arrays)
{
    size_t n = 0;
    int i = 0;
    for (auto &a : arrays) {
        off[i++] = n;
        n += (a.second + 255) / 256 * 256;
    }
    std::vector<char> host(n, 0);
    i = 0;
    for (auto &a : arrays) {
        if (a.second) std::memcpy(host.data() + off[i], a.first, a.second);
        ++i;
    }
    if (hipMalloc(&blob, std::max<size_t>(n, 1)) != hipSuccess) return S2_ERR_ALLOC;
    return hipMemcpy(blob, host.data(), n, hipMemcpyHostToDevice) == hipSuccess ? 0 : S2_ERR_ALLOC;
}

// psi of one row as pairs of input offsets +d and -d for the owner class sc of C (input offset d leads to walked column
// (sc - d) / C of owner 0, where C divides sc - d): f(first column, second column, psi of +-d, factor, d), only for offsets with a
// hat that is not zero.  A column of its own (d = 0, half a turn on an even circle, one of the two not on the walked grid) is
// both columns, and the factor is one half.
template <class F>
void for_offsets(const float *psi, int cnt, int nlon_in, int K, int KP, int C, int sc, F &&f)
{
    const bool full = cnt == nlon_in;
    const int hw = full ? nlon_in / 2 : (cnt - 1) / 2;
    for (int d = 0; d <= hw; ++d) {
        const float *p = psi + size_t(d) * KP;
        int j = 0;
        while (j < K && p[j] == 0.f) ++j;
        if (j == K) continue;
        const bool once = d == 0 || (full && 2 * d == nlon_in), one = (sc - d) % C == 0, two = !once && (sc + d) % C == 0;
        if (!one && !two) continue;
        const int first = one ? (sc - d) / C : (sc + d) / C, second = two ? (sc + d) / C : first;
        f(first, second, j, p, one && two ? 1.f : 0.5f, d);
    }
}

// A workgroup's share of LDS: three of them on a compute unit.  Longer rows are staged in parts: with a larger share for the
// polar rows the workgroups of every latitude would have it (where a
// wavefront staged for itself, 721 x 1440, 32 channels, K = 4: z 1.33 against 0.77 ms), and a launch of
// their own would run by itself as long as its longest workgroup (361 x 720: z 276 -> 424 us).  From nine walked columns per
// owner on, even a part with a single offset takes more; it may up to what needs no raised limit.
constexpr int kGatherLds = 52 * 1024, kGatherLdsMost = 64 * 1024;

// Tables for owners on `nlat_own` latitudes (classes of latitudes); walked(lat, f) calls f(walked latitude, psi of its input
// offsets 0 .. nlon_in / 2 at [offset * KP + k], offset count of the arc) for every row of owner latitude lat.  P walked columns
// per owner, or C owner columns per walked one: the owner u of class s is input column C u + s, and input offset d leads to
// walked column u + (s - d) / C where C divides s - d.
// 0: built (or a row needs too much LDS: lds_bytes stays 0), else an error code.
template <class Walk>
int build_gather(GatherTables &t, int K, int KP, int P, int C, int nlat_own, int nlon_own, int nlon_walk, Walk &&walked)
{
    // two owners per lane halve the staged columns that are not owners' own; one where a second set would mostly be idle
    t.W = nlon_own % 128 > 0 && nlon_own % 128 <= 64 ? 1 : 2;
    std::vector<int> chunk_of(1, 0), chunk, order;
    std::vector<GatherPiece> pieces;
    std::vector<GatherEntry> entries;
    std::vector<std::pair<long, int>> cost;
    int most = 0;
    struct Pair {
        int first, second, j;
        float lo, hi;
        int d, owner;                                            // offset, latitude of the group
    };
    for (int grp = 0; grp * kGroup < nlat_own; ++grp) {
        const size_t first_entry = entries.size();
        std::vector<std::vector<GatherEntry>> by_interval(kGroup * K);
        int piece0 = int(pieces.size()), base = 0;
        auto flush = [&]() {
            if (int(pieces.size()) == piece0) return;
            chunk.push_back(piece0);
            chunk.push_back(int(pieces.size()));
            for (int i = 0; i < kGroup * K; ++i) {
                if (i % K == 0) chunk.push_back(int(entries.size()));
                entries.insert(entries.end(), by_interval[i].begin(), by_interval[i].end());
                chunk.push_back(int(entries.size()));
                by_interval[i].clear();
            }
            most = std::max(most, base * 16);
            piece0 = int(pieces.size());
            base = 0;
        };
        std::map<int, std::vector<Pair>> rows;                   // by walked latitude
        for (int o = 0; o < kGroup && grp * kGroup + o < nlat_own; ++o) {
            const int lat = grp * kGroup + o;
            walked(lat, [&](int wl, const float *psi, int cnt) {
                for_offsets(psi, cnt, nlon_walk * C, K, KP, C, lat % C, [&](int first, int second, int j, const float *p, float f, int d) {
                    rows[wl].push_back({first, second, j, f * p[j], j + 1 < K ? f * p[j + 1] : 0.f, d, o});
                });
            });
        }
        for (auto &row : rows) {
            const int wl = row.first;
            std::vector<Pair> &pairs = row.second;
            std::stable_sort(pairs.begin(), pairs.end(), [](const Pair &a, const Pair &b) { return a.d < b.d; });
            // Staged columns for the offsets lo .. hi of 64 W owners, owner by owner those of one remainder mod P together.
            struct Window {
                int left, sub;
                Window(int lo, int hi, int P, int owners)
                {
                    left = lo <= 0 ? (-lo + P - 1) / P * P : -(lo / P * P);
                    sub = owners - 1 + (left + hi) / P + 1;
                }
            };
            const int owners = 64 * t.W, room = kGatherLds / 16;
            for (size_t i = 0; i < pairs.size();) {
                // as many pairs as fit: in one window over all their columns, or in one for the first and one for the second ones
                int lo[2] = {pairs[i].first, pairs[i].second}, hi[2] = {lo[0], lo[1]}, size = 0;
                bool one = true;
                size_t end = i;
                for (size_t k = i; k < pairs.size(); ++k) {
                    const int l[2] = {std::min(lo[0], pairs[k].first), std::min(lo[1], pairs[k].second)};
                    const int h[2] = {std::max(hi[0], pairs[k].first), std::max(hi[1], pairs[k].second)};
                    const int whole = P * Window(std::min(l[0], l[1]), std::max(h[0], h[1]), P, owners).sub;
                    const int apart = P * (Window(l[0], h[0], P, owners).sub + Window(l[1], h[1], P, owners).sub);
                    if (k > i && std::min(whole, apart) > room) break;
                    one = whole <= apart;
                    size = std::min(whole, apart);
                    for (int s = 0; s < 2; ++s) {
                        lo[s] = l[s];
                        hi[s] = h[s];
                    }
                    end = k + 1;
                }
                if (base > 0 && base + size > room) flush();
                if (one) {
                    lo[0] = lo[1] = std::min(lo[0], lo[1]);
                    hi[0] = hi[1] = std::max(hi[0], hi[1]);
                }
                int at[2][2];                                    // LDS position and left margin of either column's window
                for (int s = 0; s < (one ? 1 : 2); ++s) {
                    const Window w(lo[s], hi[s], P, owners);
                    for (int i0 = 0, n = w.sub * P, most = 64 * (t.W + 1); i0 < n; i0 += most)
                        pieces.push_back({wl, w.left, i0, std::min(most, n - i0), base, w.sub, {}});
                    at[s][0] = base;
                    at[s][1] = w.left;
                    base += w.sub * P;
                }
                auto place = [&](int s, int off) {
                    const int w = one ? 0 : s, x = at[w][1] + off, sub = Window(lo[w], hi[w], P, owners).sub;
                    return 16 * (at[w][0] + x % P * sub + x / P);
                };
                for (; i < end; ++i) {
                    const Pair &p = pairs[i];
                    by_interval[p.owner * K + p.j].push_back({place(0, p.first), place(1, p.second), p.lo, p.hi});
                }
            }
        }
        flush();
        chunk_of.push_back(int(chunk.size() / (2 + kGroup * (K + 1))));
        cost.push_back({-long(entries.size() - first_entry), grp});
    }
    if (most > kGatherLdsMost) return 0;
    entries.resize(entries.size() + 2, {0, 0, 0.f, 0.f});
    std::stable_sort(cost.begin(), cost.end(), [](const auto &a, const auto &b) { return a.first < b.first; });
    for (auto &c : cost) order.push_back(c.second);
    size_t off[6];
    if (upload(t.blob, off, {{chunk_of.data(), chunk_of.size() * 4}, {chunk.data(), chunk.size() * 4}, {pieces.data(), pieces.size() * sizeof(GatherPiece)},
                             {entries.data(), entries.size() * sizeof(GatherEntry)}, {order.data(), order.size() * 4}}))
        return S2_ERR_ALLOC;
    char *b = static_cast<char *>(t.blob);
    t.chunk_of = reinterpret_cast<const int *>(b);
    t.chunk = reinterpret_cast<const int *>(b + off[1]);
    t.piece = reinterpret_cast<const GatherPiece *>(b + off[2]);
    t.entry = reinterpret_cast<const GatherEntry *>(b + off[3]);
    t.order = reinterpret_cast<const int *>(b + off[4]);
    t.lds_bytes = std::max(most, 16);
    return 0;
}

// Tables of disco_gather_planes; `walked` as for build_gather.
template <class Walk>
int build_planes(PlaneTables &t, int K, int KP, int C, int nlat_own, int nlat_walk, int nlon_walk, Walk &&walked)
{
    constexpr int BATCH = 16;                         // four wavefronts, four terms each
    std::vector<int> first(1, 0), order;
    std::vector<PlaneTerm> terms;
    std::vector<std::pair<long, int>> cost;
    for (int lat = 0; lat < nlat_own; ++lat) {
        walked(lat, [&](int wl, const float *psi, int cnt) {
            for_offsets(psi, cnt, nlon_walk * C, K, KP, C, lat % C, [&](int one, int two, int j, const float *p, float f, int) {
                auto col = [&](int x) { return (x % nlon_walk + nlon_walk) % nlon_walk; };
                for (int k = j; k <= j + 1 && k < K; ++k)
                    if (p[k] != 0.f) terms.push_back({(long(k) * nlat_walk + wl) * nlon_walk, col(one), col(two), f * p[k], 0});
            });
        });
        const int n = int(terms.size()) - first.back();
        if (n > 0)                                    // whole batches: the last term again, without weight
            for (int i = n; i % BATCH; ++i) {
                terms.push_back(terms.back());
                terms.back().w = 0.f;
            }
        first.push_back(int(terms.size()));
        cost.push_back({-long(n), lat});
    }
    std::stable_sort(cost.begin(), cost.end(), [](const auto &a, const auto &b) { return a.first < b.first; });
    for (auto &c : cost) order.push_back(c.second);
    size_t off[3];
    if (upload(t.blob, off, {{first.data(), first.size() * 4}, {terms.data(), terms.size() * sizeof(PlaneTerm)}, {order.data(), order.size() * 4}}))
        return S2_ERR_ALLOC;
    char *b = static_cast<char *>(t.blob);
    t.first = reinterpret_cast<const int *>(b);
    t.term = reinterpret_cast<const PlaneTerm *>(b + off[1]);
    t.order = reinterpret_cast<const int *>(b + off[2]);
    return 0;
}

// Does the backward pass apply psi^T before the channel mixing?  Before it, disco_gather takes cout channels and the mixing runs
// over cout K planes on the input points; after it, disco_gather_planes takes cin channels, which cost it about three times as
// much each on equal grids and less than disco_gather's on 2:1 grids (two classes of owners stage every row), and the mixing
// runs over cin K planes on the output points.  Hence after it from cout = 3 cin on, on 2:1 grids from cout = cin on, and there
// also where disco_gather would not fill the device (twelve wavefronts per compute unit) and takes as long as its longest one.
// Steps with psi^T first / after, us, batch 4: 129 x 256, 16 -> 96 channels, K = 9 625 / 408; 32 -> 96, K = 9 701 / 623;
// 32 -> 64, K = 4 369 / 389; 48 -> 96, K = 9 816 / 908; 64 -> 64, K = 9 691 / 1041; 257 x 512 -> 129 x 256, 16 -> 96, K = 9
// 2154 / 540; 64 -> 64, K = 9 1726 / 1257, K = 4 885 / 928; 64 -> 32, K = 4 576 / 878; 64 x 128, 16 -> 16, K = 9 131 / 117,
// 64 -> 64, K = 9 197 / 240.  The channel matrices take multiples of 16.
bool transposed_first(const s2_disco_t *dc, int batch, int cin, int cout)
{
    const s2_grid_t *g = dc->g;
    if (dc->bwd.lds_bytes == 0 || cin % 16 != 0 || g->nlat_in * g->nlon_in % 16 != 0 || cout >= 3 * cin) return false;
    const int tile = 64 * dc->bwd.W;
    const long waves = long((g->nlon_out + tile - 1) / tile) * ((long(batch) * cout + 3) / 4) * g->nlat_in * g->pscale;
    return cout < cin || (g->pscale == 1 && waves >= 12l * dc->compute_units);
}

}  // namespace

extern "C" int s2_disco_init(const s2_grid_t *g, int nbasis, s2_disco_t **out)
{
    if (!out) return s2_fail(S2_ERR_INVALID_ARG, "out is NULL");
    *out = nullptr;
    if (!g) return s2_fail(S2_ERR_INVALID_ARG, "grid is NULL");
    if (nbasis < 1 || nbasis > kMaxBasis) return s2_fail(S2_ERR_INVALID_ARG, "nbasis must lie in [1, 16]");
    if (g->upscale > 1) return s2_fail(S2_ERR_UNSUPPORTED, "the DISCO convolution covers equal grids and downsampling");
    s2_disco *dc = new (std::nothrow) s2_disco();
    if (!dc) return s2_fail(S2_ERR_ALLOC, "out of host memory");
    dc->g = g;
    dc->K = nbasis;
    // basis values along the arcs of the kernels' tables (zero-weight latitudes are not in them)
    const double kPi = 3.141592653589793238462643383279502884, dr = g->theta / nbasis;
    const int KP = padded(nbasis);      // values per arc offset in the table (zeros behind the last basis function)
    std::vector<int> poff(size_t(g->nlat_out) * g->band_max, 0);
    std::vector<float> psi;
    for (int h = 0; h < g->nlat_out; ++h)
        for (int b = 0; b < g->band_n[h]; ++b) {
            const int hp = g->band_lo[h] + b, c = g->cnt[size_t(h) * g->band_max + b];
            const int lo = c == g->nlon_in ? 0 : -((c - 1) / 2);
            poff[size_t(h) * g->band_max + b] = int(psi.size() / KP);
            for (int tt = 0; tt < c; ++tt) {
                const int wp = ((lo + tt) % g->nlon_in + g->nlon_in) % g->nlon_in;
                const double r = s2_great_circle(g->colat_out[h], g->colat_in[hp], 2.0 * kPi * wp / g->nlon_in);
                for (int k = 0; k < KP; ++k)
                    psi.push_back(k < nbasis ? float(std::max(0.0, 1.0 - std::fabs(r / dr - k)) * g->omega_in[hp]) : 0.f);
            }
        }
    if (g->on_device) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, g->device) == hipSuccess && n > 0) dc->compute_units = n;
        // psi of the offsets 0, 1, ... of an arc (it is symmetric)
        auto arc = [&](int h, int b) -> const float * {
            const int c = g->cnt[size_t(h) * g->band_max + b], mid = c == g->nlon_in ? 0 : (c - 1) / 2;
            return psi.data() + (size_t(poff[size_t(h) * g->band_max + b]) + mid) * KP;
        };
        int rc = build_gather(dc->fwd, nbasis, KP, g->pscale, 1, g->nlat_out, g->nlon_out, g->nlon_in, [&](int h, auto &&f) {
            for (int b = 0; b < g->band_n[h]; ++b) {
                const int c = g->cnt[size_t(h) * g->band_max + b];
                if (c > 0) f(g->band_lo[h] + b, arc(h, b), c);
            }
        });
        auto transposed = [&](int v, auto &&f) {
            const int hp = v / g->pscale;
            for (int i = 0; i < g->tband_n[hp]; ++i) {
                const int h = g->tband_lo[hp] + i, b = hp - g->band_lo[h];
                if (b < 0 || b >= g->band_n[h]) continue;            // a latitude of weight zero is in no band
                const int c = g->cnt[size_t(h) * g->band_max + b];
                if (c > 0) f(h, arc(h, b), c);
            }
        };
        const int classes = g->nlat_in * g->pscale;
        if (!rc) rc = build_gather(dc->bwd, nbasis, KP, 1, g->pscale, classes, g->nlon_out, g->nlon_out, transposed);
        if (!rc) rc = build_planes(dc->planes, nbasis, KP, g->pscale, classes, g->nlat_out, g->nlon_out, transposed);
        if (rc) {
            (void)hipGetLastError();
            s2_disco_destroy(dc);
            return s2_fail(S2_ERR_ALLOC, "set-up of the contraction tables failed");
        }
        // the basis values themselves only for the gather per point
        if (dc->fwd.lds_bytes == 0 &&
            (hipMalloc(&dc->dev_psi, std::max<size_t>(psi.size(), 1) * sizeof(float)) != hipSuccess ||
             hipMalloc(&dc->dev_poff, poff.size() * sizeof(int)) != hipSuccess ||
             hipMemcpy(dc->dev_psi, psi.data(), psi.size() * sizeof(float), hipMemcpyHostToDevice) != hipSuccess ||
             hipMemcpy(dc->dev_poff, poff.data(), poff.size() * sizeof(int), hipMemcpyHostToDevice) != hipSuccess)) {
            (void)hipGetLastError();
            s2_disco_destroy(dc);
            return s2_fail(S2_ERR_ALLOC, "set-up of the basis tables failed");
        }
    }
    *out = dc;
    return S2_OK;
}

extern "C" void s2_disco_destroy(s2_disco_t *dc)
{
    if (!dc) return;
    if (dc->dev_psi) (void)hipFree(dc->dev_psi);
    if (dc->dev_poff) (void)hipFree(dc->dev_poff);
    if (dc->fwd.blob) (void)hipFree(dc->fwd.blob);
    if (dc->bwd.blob) (void)hipFree(dc->bwd.blob);
    if (dc->planes.blob) (void)hipFree(dc->planes.blob);
    delete dc;
}

extern "C" size_t s2_disco_workspace_bytes(const s2_disco_t *dc, int batch, int cin, int cout)
{
    if (!dc || batch < 1 || cin < 1 || cout < 1) return 0;
    const size_t n_out = size_t(dc->g->nlat_out) * dc->g->nlon_out, n_in = size_t(dc->g->nlat_in) * dc->g->nlon_in;
    auto up = [](size_t x) { return (x + 63) / 64 * 64; };
    // z [batch][cin * K][n_out]; psi^T dy [batch][cout * K][n_in] and the transposed weight, or dz like z; partial sums of the
    // weight gradient
    const size_t zs = up(size_t(batch) * cin * dc->K * n_out);
    const size_t mid = transposed_first(dc, batch, cin, cout) ? up(size_t(batch) * cout * dc->K * n_in) + up(size_t(cout) * cin * dc->K)
                                                 : zs;
    return (zs + mid + up(s2_channel_grad_floats(cout, cin * dc->K, 1))) * sizeof(float);
}

extern "C" int s2_disco_fwd(const s2_disco_t *dc, int batch, int cin, int cout, const float *x, const float *weight,
                            const float *bias, float *y, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    int rc = check(dc, batch, cin, cout, workspace, workspace_bytes);
    if (rc) return rc;
    if (!x || !weight || !y) return s2_fail(S2_ERR_INVALID_ARG, "NULL tensor pointer");
    if ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(weight) | reinterpret_cast<uintptr_t>(y)) % 16 != 0)
        return s2_fail(S2_ERR_INVALID_ARG, "tensor pointers must be 16-byte aligned");
    const s2_grid_t *g = dc->g;
    if (!g->on_device) return s2_fail(S2_ERR_DEVICE, "grid handle has no device tables (no HIP device at init)");
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    float *z = static_cast<float *>(workspace);
    const int n_out = g->nlat_out * g->nlon_out, K = dc->K;
    {
        S2TraceScope tr("disco_z_fwd", 0.0, st);
        if (dc->fwd.lds_bytes) {
            launch_gather(dc->fwd, K, g->pscale, 1, g->nlon_out, g->nlon_in, g->nlat_out, g->nlat_in, batch * cin, x, z, st);
        } else {
            const dim3 grid((g->nlon_out + 63) / 64, g->nlat_out, batch * cin);
            by_basis(K, [&](auto KB) {
                hipLaunchKernelGGL((disco_z_fwd<decltype(KB)::value>), grid, dim3(64), 0, st, g->dt, dc->dev_psi, dc->dev_poff, K, x, z);
            });
        }
    }
    S2TraceScope tr("disco_mix", 0.0, st);
    s2_channel_product(false, {cout, n_out, cin * K, batch, 1, 1, {weight}, {z}, {bias}, nullptr, {y}}, st);
    S2_HIP_CHECK(hipGetLastError());
    return S2_OK;
}

extern "C" int s2_disco_bwd(const s2_disco_t *dc, int batch, int cin, int cout, const float *x, const float *weight,
                            const float *dy, float *dx, float *dweight, float *dbias, void *workspace,
                            size_t workspace_bytes, void *hip_stream)
{
    (void)x;       // z = psi * x was kept in the workspace by the forward pass
    int rc = check(dc, batch, cin, cout, workspace, workspace_bytes);
    if (rc) return rc;
    if (!weight || !dy || !dx) return s2_fail(S2_ERR_INVALID_ARG, "NULL tensor pointer");
    if ((reinterpret_cast<uintptr_t>(weight) | reinterpret_cast<uintptr_t>(dy) | reinterpret_cast<uintptr_t>(dx)) % 16 != 0)
        return s2_fail(S2_ERR_INVALID_ARG, "tensor pointers must be 16-byte aligned");
    const s2_grid_t *g = dc->g;
    if (!g->on_device) return s2_fail(S2_ERR_DEVICE, "grid handle has no device tables (no HIP device at init)");
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const int n_out = g->nlat_out * g->nlon_out, K = dc->K;
    auto up = [](size_t v) { return (v + 63) / 64 * 64; };
    float *z = static_cast<float *>(workspace), *mid = z + up(size_t(batch) * cin * K * n_out);
    const bool first = transposed_first(dc, batch, cin, cout);
    const size_t mids = first ? up(size_t(batch) * cout * K * g->nlat_in * g->nlon_in) : up(size_t(batch) * cin * K * n_out);
    float *wt = mid + mids;                   // transposed weight (psi^T first)
    float *part = wt + (first ? up(size_t(cout) * cin * K) : 0);
    {
        S2TraceScope tr("disco_bwd mix", 0.0, st);
        if (dweight || dbias) s2_channel_grad({cout, n_out, cin * K, batch, 1, {dy}, {z}, {dweight}, {dbias}}, part, st);
        if (!first) s2_channel_product(true, {cin * K, n_out, cout, batch, 1, 1, {weight}, {dy}, {nullptr}, nullptr, {mid}}, st);
    }
    if (first) {
        {
            S2TraceScope tr("disco_dx", 0.0, st);
            launch_gather(dc->bwd, K, 1, g->pscale, g->nlon_out, g->nlon_out, g->nlat_in * g->pscale, g->nlat_out, batch * cout, dy, mid, st);
        }
        S2TraceScope tr("disco_dx mix", 0.0, st);
        hipLaunchKernelGGL(disco_weight_transpose, dim3((cout * cin * K + 255) / 256), dim3(256), 0, st, cout, cin, K, weight, wt);
        s2_channel_product(false, {cin, g->nlat_in * g->nlon_in, cout * K, batch, 1, 1, {wt}, {mid}, {nullptr}, nullptr, {dx}}, st);
        S2_HIP_CHECK(hipGetLastError());
        return S2_OK;
    }
    S2TraceScope tr("disco_dx planes", 0.0, st);
    constexpr int CH = 4;
    const unsigned blocks = unsigned((g->nlon_out + 63) / 64) * unsigned((batch * cin + CH - 1) / CH) * unsigned(g->nlat_in * g->pscale);
    hipLaunchKernelGGL(disco_gather_planes<CH>, dim3(blocks), dim3(256), 0, st, dc->planes, g->pscale, size_t(K) * n_out, g->nlon_out,
                       g->nlon_out, size_t(g->nlat_in) * g->nlon_in, batch * cin, mid, dx);
    S2_HIP_CHECK(hipGetLastError());
    return S2_OK;
}
