// Internal definitions shared by the translation units of libs2attn.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>
#include <vector>

#include "s2attn.h"

// Device-resident compact form of the indicator 1[h,h',w'] (App. B.3).
// For output latitude h the disk meets the input latitudes
// band_lo[h] .. band_lo[h]+band_n[h]-1; on input latitude h' it covers `cnt`
// consecutive longitude offsets centred on w' = 0 (cnt odd), or the whole
// circle (cnt == nlon_in).  tband_*/tcnt hold the same numbers indexed by the
// input latitude (input point -> output latitudes), used by the dk/dv gather.
// The same relation as rows of one longitude count, for one kind of owners: outputs (forward, dq) or inputs
// (dk/dv).  Where the longitude counts of the two grids differ, the latitudes of the finer one are cut into interleaved
// classes, so that owner rows and walked rows all have nU = min(nlon_in, nlon_out) columns: owner row v is latitude
// v / c_own, longitudes c_own * u + v % c_own; the same for walked rows with c_walk.
struct S2BandSide {
    const int *blo, *bn;      // [n_own]         first walked row and number of walked rows of an owner row
    const int2 *arc;          // [n_own][bmax]   (first offset, number of offsets); (0, nU): the whole circle; .y may be 0
    int bmax, n_own, nU;
    int c_own, c_walk;
    int nlat_own, nlat_walk;
    // the patch kernels (s2_nattn_patch_impl.h)
    struct Patches {
        const int4 *seg;      // 2 per segment: (first owner row, log2(owner rows), first walked row, walked rows), (chunks, place in row_rec, another part follows, -)
        const int4 *row_rec;  // 2 per walked row of a segment: S2PatchRow
        const int2 *patch;    // workgroups of a slice, heaviest first: segment, first column
        int npatch;
        // walked columns per owner column: 1, the rows are classes; c_walk, they are whole latitudes and offsets count their columns
        int step;
        // for small launches: the same points, those of heavy workgroups in workgroups of two patches and of one, which two and four
        // wavefronts share
        struct Split {
            const int2 *list;     // segment, first column + (log2(wavefronts that share a patch) << 16)
            int n;
            double work;          // of a slice, in workgroups as heavy as the heaviest unsplit one; parts two or three times what they were
        } split[2];
        int heaviest;             // chunks of the heaviest unsplit workgroup
    } patches;
};

// A walked row as the owners of a segment see it.  The columns that any of a workgroup's owners meets on it are cut into chunks
// of four; the chunks of all rows are numbered in order.  Columns are relative to the workgroup's first (times step).
constexpr int kS2PatchWaves = 4;         // wavefronts of a workgroup
constexpr int kS2PatchRows = 128;        // walked rows of a part of a segment
struct S2PatchRow {
    int col;                  // first column of chunk X of the row = col + 4 X
    int uni;                  // union of the owner rows' arcs: first offset (16 bits), length (16 bits)
    int before;               // chunks of the rows before
    float omega;              // the row's relative quadrature weight (owners = inputs: 1)
    unsigned arc[4];          // per owner row: first offset (16 bits), length (16 bits)
};

// Walked rows as 16 owner rows of one column see them, for owners that are the classes of a finer grid: the four wavefronts of a workgroup
// own columns four apart.  A row is walked in pieces that a stage holds, from a column that is counted from the owner's, and stages hold
// whole pieces: every owner's sums run in the order of its own offsets, whatever its column.
constexpr int kS2ColumnRows = 64, kS2ColumnStage = 16;
struct S2ColumnRow {
    int col, uni, before;     // as in S2PatchRow; the piece alone, for the first wavefront
    int row;                  // the walked row
    float omega;
    int unused[3];
    unsigned arc[16];
};

struct S2DeviceTables {
    const float *omega_rel;   // [nlat_in]   omega[h'] / max omega
    const int *band_lo;       // [nlat_out]
    const int *band_n;        // [nlat_out]
    const int *cnt;           // [nlat_out][band_max]
    const int *tband_lo;      // [nlat_in]
    const int *tband_n;       // [nlat_in]
    const int *tcnt;          // [nlat_in][tband_max]
    const int *row_order;     // [nlat_out]  output latitudes, heaviest first
    const int *trow_order;    // [nlat_in]   input latitudes, heaviest first
    int band_max, tband_max;
    int fwd_cls[4];           // output latitudes (in row_order) whose run list is split 8, 4, 2, 1 ways
    int bwd_cls[4];           // same for input latitudes (trow_order)
    double fwd_pairs[4];      // (output, input) pairs per slice handled by each class of output latitudes
    double bwd_pairs[4];      // the same pairs counted per class of input latitudes
    // the same four tables with all class thresholds divided by four: used when there are too few
    // (batch, head) slices for the coarse split to fill the machine
    int fwd_cls_fine[4], bwd_cls_fine[4];
    double fwd_pairs_fine[4], bwd_pairs_fine[4];
    int nlat_in, nlon_in, nlat_out, nlon_out, pscale;
    // streaming kernels for the light latitudes (the last class): contiguous range [st_lo, st_hi) of output
    // latitudes and the number of wavefronts st_nw such that the band of latitude h + st_nw starts no earlier
    // than the last row of the band of h; st_nw = 0 if the light latitudes do not have that structure.
    // tst_*: the same for input latitudes and the transposed bands.
    int st_lo, st_hi, st_nw;
    int tst_lo, tst_hi, tst_nw;
    S2BandSide side_out, side_in;       // owners = output points, owners = input points
    S2BandSide::Patches columns;        // side_out by columns (upsampling grids; else no workgroups)
    // the patch kernels apply: nU < 2^15
    int band_rows_ok;
    unsigned *dev_flags;      // one word in device memory: bit 0 = a bounded wait inside a kernel ran out
    const int *st_cum;        // [st_hi - st_lo + 1]   running cost of the light latitudes (for equal-work segments)
    const int *tst_cum;       // [tst_hi - tst_lo + 1]
    float ln_omega_ref;       // ln(max omega): the stored logsumexp is relative to the true omega
    float omega_ref;          // max omega
    // upsampling (nlon_out = upscale * nlon_in, upscale > 1; pscale is 1 then): output longitude w = upscale*m + s
    // lies between input meridians, so the arc on input latitude band_lo[h] + b depends on the class s:
    // input columns m + ulo .. m + ulo + ucnt - 1 (ucnt may be 0), tables indexed [(h*upscale + s)*band_max + b]
    int upscale;
    const int *ucnt;
    const int *ulo;
};

struct s2_grid {
    int grid_type;
    int nlat_in, nlon_in, nlat_out, nlon_out, pscale;
    double theta;
    std::vector<double> colat_in, omega_in, colat_out;
    // host copies of the compact tables
    std::vector<int> band_lo, band_n, cnt, tband_lo, tband_n, tcnt, row_order, trow_order, st_cum, tst_cum;
    int upscale = 1;
    std::vector<int> ucnt, ulo;      // upsampling only (see S2DeviceTables)
    std::vector<int> vo_lo, vo_n, vi_lo, vi_n;      // S2BandSide tables, owners = outputs / inputs
    std::vector<int2> vo_arc, vi_arc;
    struct Patches {
        std::vector<int4> seg;
        std::vector<S2PatchRow> rows;
        std::vector<int2> list, split[2];
        int step = 1;
        double split_work[2] = {};
        int heaviest = 0;
    } vo_patch, vi_patch;
    struct Columns {
        std::vector<int4> seg;
        std::vector<S2ColumnRow> rows;
        std::vector<int2> list;
    } columns;
    int band_max = 0, tband_max = 0;
    // the band and arc tables exactly as eq. (5) gives them (introspection); the tables above, which the kernels
    // use, leave out input latitudes of weight zero (listed in zero_lat)
    std::vector<int> c_band_lo, c_band_n, c_cnt, c_ucnt, c_ulo, zero_lat;
    int c_band_max = 0;
    // canonical CSR
    std::vector<int64_t> row_ptr;
    std::vector<int32_t> col;
    // device side
    bool on_device = false;
    int device = -1;
    void *dev_blob = nullptr;
    // global attention: omega / max omega per input token, 0 on the padding up to npad_tok (a multiple of 64)
    int npad_tok = 0;
    const float *dev_w_tok = nullptr;
    S2DeviceTables dt{};
};

// Class table for the split vector kernels.  If the coarse split would start so few wavefronts that most SIMDs hold
// fewer than eight, the copy `t` is switched to the fine split.
inline void s2_pick_split(S2DeviceTables &t, bool fwd, int nbh, int nseg)
{
    int *c = fwd ? t.fwd_cls : t.bwd_cls;
    double *p = fwd ? t.fwd_pairs : t.bwd_pairs;
    const long waves = long(nbh) * nseg * (8 * c[0] + 4 * c[1] + 2 * c[2] + c[3]);
    if (waves >= 8192) return;
    const int *cf = fwd ? t.fwd_cls_fine : t.bwd_cls_fine;
    const double *pf = fwd ? t.fwd_pairs_fine : t.bwd_pairs_fine;
    for (int i = 0; i < 4; ++i) {
        c[i] = cf[i];
        p[i] = pf[i];
    }
}

// Optional per-launch timing (s2_trace_* in the C ABI): when enabled, a scope records a HIP event
// before and after the launches it encloses, on the stream they go to.
void s2_trace_begin(const char *name, double pairs, hipStream_t st);
void s2_trace_end(hipStream_t st);
struct S2TraceScope {
    hipStream_t st;
    S2TraceScope(const char *name, double pairs, hipStream_t s) : st(s) { s2_trace_begin(name, pairs, s); }
    ~S2TraceScope() { s2_trace_end(st); }
};

// Test-only switches (bits of s2_debug_control): which kernel families the dispatch may pick, and a forced
// launcher failure.
bool s2_debug_flag(unsigned bit);

// One-time set-up of the kernels of each translation unit on the current device: raises the dynamic LDS limit of
// every kernel that needs more than the default.  Called from s2_grid_init (once per device), so that the attention
// calls themselves only enqueue launches.  0 on success.
int s2_nattn_tiled_configure();
int s2_nattn_bwd_tiled_configure();
int s2_nattn_stream_configure();
int s2_nattn_band_configure();

// great-circle angle between two points given by their colatitudes and their difference in longitude (float64)
double s2_great_circle(double colat_a, double colat_b, double dphi);

// Channel matrices on the matrix cores (s2_channel.hip), all tensors [batch][channels][N] contiguous and 16-byte
// aligned, M, K and N multiples of 16.
//   s2_channel_product: nset products side by side, C[i] = A[i] X[i] + bias[i], or (nset = 1) one over npair pairs,
//                       C[0] = sum_i A[i] X[i] + bias[0] + R;  A = W (M x K) or W^T (trans, W is K x M)
//   s2_channel_grad:    nset times dW[i] (M x K) = sum_{b, n} dY[i] X[i]^T, dbias[i] = sum_{b, n} dY[i] (either may be
//                       NULL); `part`: s2_channel_grad_floats(M, K, nset) floats of scratch
struct S2ChannelProduct {
    int M, N, K, batch, nset, npair;
    const float *W[3], *X[3], *bias[3];
    const float *R;
    float *C[3];
};
struct S2ChannelGrad {
    int M, N, K, batch, nset;
    const float *dY[3], *X[3];
    float *dW[3], *dbias[3];
};
void s2_channel_product(bool trans, const S2ChannelProduct &a, hipStream_t st);
size_t s2_channel_grad_floats(int M, int K, int nset);
void s2_channel_grad(const S2ChannelGrad &a, float *part, hipStream_t st);

void s2_set_error(const std::string &msg);
int s2_fail(int code, const std::string &msg);

#define S2_HIP_CHECK(expr)                                                                   \
    do {                                                                                     \
        hipError_t e_ = (expr);                                                              \
        if (e_ != hipSuccess)                                                                \
            return s2_fail(S2_ERR_DEVICE, std::string(#expr) + ": " + hipGetErrorString(e_)); \
    } while (0)
