// Global quadrature-weighted attention on gfx950: bf16 MFMA (32x32x16), fp32
// softmax and accumulation, flash-style streaming over key tiles (App. B.1
// first equation; App. B.2 writes the quadrature weight as an additive column
// bias ln omega_j on the logits: here it is carried as the equivalent factor
// omega_j / max omega on the exponentials, folded into the transposed operands,
// so that a zero weight needs no special case and the running maximum follows
// the bare logits).
//
// Orientation.  Scores are produced TRANSPOSED, S^T = K Q^T, so that in the
// MFMA result layout a lane owns one query column and 16 keys.  The softmax
// over keys is then a per-lane loop (the two half-wavefronts of a query only
// talk when the running maximum has to move), and the exponentials are fed
// straight back as the B operand of the next MFMA (O^T += V^T P^T) without
// moving data between lanes.  Row r of the K tile is mapped to key
// 16*((r>>2)&1) + 4*(r>>3) + (r&3): with that permutation the 16 keys a lane
// holds are contiguous.
//
// The MFMA "A" operand wants its contraction index contiguous in memory.  V
// (forward) and Q, K, dout (backward) are contracted over tokens, so they are
// transposed once per call into the caller's workspace ([b,h][64][Npad] bf16,
// zero padded to a multiple of 64 tokens).  All streamed operands reach the
// wavefronts through LDS tiles that a workgroup copies once (see below).
//
// Backward (App. B.4 with every token in every neighborhood): D_i = dout_i.out_i,
// p_ij = omega_j exp(s_ij - lse_i), dS_ij = p_ij (dout_i.v_j - D_i);
// one kernel owns 32 keys per wavefront and streams query tiles (dk, dv), one
// owns 32 queries per wavefront and streams key tiles (dq): no atomics.
#include <type_traits>

#include "s2_internal.h"

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef unsigned short bf16raw;

constexpr int kD = 64;            // head dimension of the MFMA path
constexpr float kLog2e = 1.4426950408889634f;

__device__ __forceinline__ bf16x8 ld8(const bf16raw *p)
{
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(p));
}

__device__ __forceinline__ f32x16 mfma(bf16x8 a, bf16x8 b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ bf16x8 pack8(const float *x)
{
    bf16x8 r;
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = (__bf16)x[i];
    return r;
}

// key (or query) index of tile row r under the permutation described above
__device__ __forceinline__ int perm_row(int r) { return 16 * ((r >> 2) & 1) + 4 * (r >> 3) + (r & 3); }

// Preparation pass.  One launch handles up to three operands (blockIdx.z): each is transposed from
// [bh][N][64] to [bh][64][Npad] (zero for tokens >= N), optionally with every token multiplied by its
// weight first (rounded to bf16 once, after the product).  The block that transposes `stat_go` (dout) also
// writes the per-token backward constants, padded to Npad tokens per slice:
// L2[bh][i] = (lse_i - ln max omega) * log2(e) (+inf on the padding: p = exp2(-inf) = 0) and
// D[bh][i] = -(dout_i . out_i) (0 on the padding): the backward kernels start the accumulation of dout.v
// from -D, so that the matrix core delivers dout_i.v_j - D_i directly.
// A block moves 64 tokens: four threads per token read 32 bytes each (coalesced rows), the tile is turned in
// LDS, and four threads per channel write 32 bytes each.
struct PrepOp {
    const bf16raw *in;
    bf16raw *out;
    const float *wtok;      // weights to multiply with, or null
};
struct PrepArgs {
    PrepOp op[3];
    int stat_op;            // index of the operand that is dout (-1: no statistics)
    const bf16raw *o;       // forward output
    const float *lse;
    float *L2, *D;
    float ln_wref;
};

__global__ void __launch_bounds__(256)
prepare_operands(PrepArgs a, int N, int Npad)
{
    constexpr int kP = 72;   // tile pitch in elements: rows start 16-byte aligned, 36 banks apart
    __shared__ __attribute__((aligned(16))) bf16raw tile[kD][kP];
    const PrepOp op = a.op[blockIdx.z];
    const int bh = blockIdx.y, t0 = blockIdx.x * 64;
    const int tid = threadIdx.x, tok = tid >> 2, part = tid & 3;
    const int token = t0 + tok;
    bf16x8 x[2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int u = 0; u < 8; ++u) x[j][u] = (__bf16)0.f;
    if (token < N) {
        const bf16raw *src = op.in + (size_t(bh) * N + token) * kD + 16 * part;
        x[0] = ld8(src);
        x[1] = ld8(src + 8);
    }
    if (int(blockIdx.z) == a.stat_op) {
        float acc = 0.f;
        if (token < N) {
            const bf16raw *po = a.o + (size_t(bh) * N + token) * kD + 16 * part;
            const bf16x8 y0 = ld8(po), y1 = ld8(po + 8);
#pragma unroll
            for (int u = 0; u < 8; ++u) acc = fmaf(float(x[0][u]), float(y0[u]), fmaf(float(x[1][u]), float(y1[u]), acc));
        }
        acc += __shfl_xor(acc, 1);
        acc += __shfl_xor(acc, 2);
        if (part == 0 && token < Npad) {
            a.L2[size_t(bh) * Npad + token] = token < N ? (a.lse[size_t(bh) * N + token] - a.ln_wref) * kLog2e : INFINITY;
            a.D[size_t(bh) * Npad + token] = -acc;
        }
    }
    if (op.wtok && token < N) {
        const float w = op.wtok[token];
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int u = 0; u < 8; ++u) x[j][u] = (__bf16)(float(x[j][u]) * w);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const __bf16 e = x[j][u];      // (a bit_cast applied to the vector element itself reads element 0)
            tile[16 * part + 8 * j + u][tok] = __builtin_bit_cast(bf16raw, e);
        }
    __syncthreads();
    const int ch = tid >> 2;
    if (t0 + 16 * part < Npad) {       // Npad is a multiple of 64: a block's 64 tokens are all inside or all outside
        bf16raw *dst = op.out + (size_t(bh) * kD + ch) * Npad + t0 + 16 * part;
        *reinterpret_cast<uint4 *>(dst) = *reinterpret_cast<const uint4 *>(&tile[ch][16 * part]);
        *reinterpret_cast<uint4 *>(dst + 8) = *reinterpret_cast<const uint4 *>(&tile[ch][16 * part + 8]);
    }
}

// ---------------------------------------------------------------------------------------------
// Staging of streamed operands in LDS.  A workgroup of four wavefronts streams 64-token stages; every
// stage is copied from global memory once per workgroup (coalesced 16-byte pieces, no registers in
// between) into one of two LDS buffers while the other one is being used, and read from there by all
// four wavefronts as MFMA operands.  The two buffers are separate arrays and the stage loop is unrolled
// by two, so every access names its array: the compiler then knows that the reads of one buffer need
// not wait for the copies in flight into the other; the barrier at the end of a stage waits for them.  A staged tile is 64 rows of 128 bytes; the 16-byte
// piece c of row r sits at piece c ^ ((r >> 1) & 7), so that the 16 consecutive lanes a 16-byte LDS read
// serves together (16 consecutive rows, same logical piece) fall on 16 different bank groups, and so do
// the writes of a row.  Token-major tiles ("row tiles": 64 tokens x 64 channels) additionally have the
// rows of each 32-token half permuted so that lane `col` finds the token of MFMA row perm_row(col) in
// LDS row `col`.  Channel-major tiles ("column tiles": 64 channels x 64 tokens) come from the
// token-transposed copies in the workspace.
constexpr int kTileBytes = 64 * 128;

__device__ __forceinline__ int swz(int row, int piece) { return row * 128 + ((piece ^ ((row >> 1) & 7)) << 4); }

// LDS row of token t (0..63) of a stage: inverse of perm_row inside each 32-token half
__device__ __forceinline__ int lds_row_of_token(int t)
{
    const int k = t & 31;
    return (t & 32) | (k & 3) | (((k >> 4) & 1) << 2) | (((k >> 2) & 3) << 3);
}

// Copies go straight from global memory into LDS (global_load_lds_dwordx4: lane i of a wavefront
// deposits its 16 bytes at base + 16 i, i.e. one instruction fills eight consecutive rows), so the
// swizzle and the row permutation are applied on the source side: lane i fetches the piece that belongs
// at physical position i.  Wavefront w of the four copies rows 16 w .. 16 w + 15 of every tile.
typedef __attribute__((address_space(3))) void *lptr_t;

// Copies straight to LDS, 16 or 4 bytes a lane, lane after lane from dst on, written out: the uniform base stays in scalar
// registers and the lane's offset in one vector register.  From the compiler's own form it made the 64-bit address anew for
// each copy and, not seeing which buffer a copy goes to, waited for copies under way within the stage (65 x 128, 32 slices:
// forward 670 -> 628 us, with the backward 2767 -> 2630 us; 46 x 90, four: 63 -> 60 and 196 -> 174 us).  It does not know of
// these copies: landed() waits for the wavefront's copies and LDS reads, then for the other wavefronts of the workgroup.
// (Three buffers in turn, waiting for the older copies only, gained nothing: with small launches the chain of one tile is
// what takes the time, with large ones the LDS of the third buffer costs a workgroup of the compute unit, 643 us.)
__device__ __forceinline__ int lds_at(char *p)
{
    return int(reinterpret_cast<uintptr_t>((lptr_t)p));
}
__device__ __forceinline__ void copy16(const char *base, int off, int dst)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(dst) : "memory", "m0");
}
__device__ __forceinline__ void copy4(const char *base, int off, int dst)
{
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" ::"v"(off), "s"(base), "s"(dst) : "memory", "m0");
}
// An operand loaded the ordinary way is waited for here, not by the compiler behind the copies in the loop that uses it.
template <class T>
__device__ __forceinline__ void arrived(T &x)
{
    asm volatile("" : "+v"(x));
}
__device__ __forceinline__ void landed()
{
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
}
// What a lane fetches of the tiles of a stage: a stage moves the uniform base of a copy, the offsets stay.
struct Copies {
    int wave, lane, token[2], piece[2], col[2], N, Npad;
    __device__ __forceinline__ Copies(int wave, int lane, int N, int Npad) : wave(wave), lane(lane), N(N), Npad(Npad)
    {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int r = 16 * wave + 8 * h + (lane >> 3);
            piece[h] = 16 * ((lane & 7) ^ ((r >> 1) & 7));
            token[h] = (r & 32) | perm_row(r & 31);
            col[h] = (lane >> 3) * Npad * int(sizeof(bf16raw)) + piece[h];
        }
    }
    // token-major tile: LDS row r holds token tok0 + (r & 32) + perm_row(r & 31), clamped to N - 1
    __device__ __forceinline__ void rows(const bf16raw *base, int tok0, char *tile) const
    {
        const char *at = reinterpret_cast<const char *>(base + size_t(tok0) * kD);
#pragma unroll
        for (int h = 0; h < 2; ++h)
            copy16(at, (min(token[h], N - 1 - tok0) << 7) + piece[h], lds_at(tile) + 2048 * wave + 1024 * h);
    }
    // channel-major tile from a transposed operand [64][Npad] (Npad a multiple of 64: always in bounds)
    __device__ __forceinline__ void cols(const bf16raw *base, int tok0, char *tile) const
    {
#pragma unroll
        for (int h = 0; h < 2; ++h)
            copy16(reinterpret_cast<const char *>(base + size_t(16 * wave + 8 * h) * Npad + tok0), col[h],
                   lds_at(tile) + 2048 * wave + 1024 * h);
    }
    // 64 consecutive floats (one wavefront, lane = element)
    __device__ __forceinline__ void floats(const float *src, char *dst) const
    {
        copy4(reinterpret_cast<const char *>(src), 4 * lane, lds_at(dst));
    }
};
__device__ __forceinline__ bf16x8 lds8(const char *p)
{
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4 *>(p));
}
// MFMA operand reads by lane (col, hl).  Row tile, 32-token half `half`, contraction step ks (channels
// 16 ks + 8 hl ..): piece 2 ks + hl of row 32 half + col.  Column tile, channel half `rt`, tokens
// 32 half + 16 hl + 8 j ..: piece 4 half + 2 hl + j of row 32 rt + col.  (32 does not touch the swizzle bits.)
__device__ __forceinline__ bf16x8 row_operand(const char *tile, int col, int hl, int half, int ks)
{
    return lds8(tile + half * 4096 + swz(col, 2 * ks + hl));
}
__device__ __forceinline__ bf16x8 col_operand(const char *tile, int col, int hl, int rt, int half, int j)
{
    return lds8(tile + rt * 4096 + swz(col, 4 * half + 2 * hl + j));
}

// Units of 128 tokens of a slice.  Workgroups are numbered so that each of the eight XCDs (which take consecutive workgroup ids in turn)
// works through one contiguous piece of the (slice, unit) list: the operands of the few slices an XCD
// has in flight then stay in its own L2.  Of its piece an XCD takes the first `whole` units in one workgroup each, the others in two of
// 64 tokens.  halves: units are of 64 tokens, one workgroup each.
struct Units {
    int all, per_slice, per_xcd, whole, tokens;
    bool halves;
};
// f(split, unit of a slice's, slice) for the workgroup's share: split = 1, unit in units of 128 tokens, or 2, of 64
template <class F>
__device__ __forceinline__ void take_unit(const Units &u, F &&f)
{
    const int i = int(blockIdx.x >> 3), j = u.halves ? -1 : i - u.whole, k = j < 0 ? i : u.whole + (j >> 1), unit = int(blockIdx.x & 7) * u.per_xcd + k;
    if (k >= u.per_xcd || unit >= u.all) return;
    const int bh = unit / u.per_slice, q = unit - bh * u.per_slice, half = u.halves ? q : 2 * q + (j & 1);
    if (j < 0 && !u.halves) f(std::integral_constant<int, 1>(), q, bh);
    else if (64 * half < u.tokens) f(std::integral_constant<int, 2>(), half, bh);
}

// Forward.  A workgroup owns 128 queries of one slice (one 32-query MFMA tile per wavefront) and streams
// the keys in stages of 64.  omega enters as a factor, not as a bias: V^T arrives premultiplied by
// w_j = omega_j / max omega (prepare_operands does that), the running sum is l_i = sum_j w_j 2^(x_ij - m_i)
// with x = log2(e) scale q.k, and the reference m_i follows the bare logits of the keys of positive weight (it moves
// only when a logit exceeds it by more than 2^8).  lse_i = ln 2 (m_i + log2 l_i) + ln max omega.
// live: the tokens of positive weight.  Only tiles that hold others too look at the weights one by one (in every tile: 16 comparisons and
// choices more of some 60 vector instructions, and a longer chain where a SIMD has one wavefront: 46 x 90, four heads 58 -> 50 us, 24 heads
// 204 -> 154 of the call).  UNIFORM_W: the longitude count is a multiple of 32, so a 32-key tile never straddles two latitudes.
// SPLIT = 2 is for launches with too few workgroups to fill the chip: the four wavefronts are two pairs, each pair owns
// the same 64 queries and takes every other 32-key tile of a stage, and the pairs' (o, m, l) meet in LDS behind the
// last stage, so a query's serial chain over the keys is half as long and the launch has twice the workgroups
// (46 x 90, four heads: 94 us with SPLIT = 1, 64 us with SPLIT = 2; see split_units for the line).
// common: the launch has units that are not split.  Probabilities are rounded to bf16 relative to the reference, which comes from the first tile
// of live keys; the pair that does not meet that tile takes the reference from it all the same.  With a reference of its own, split units were
// apart from unsplit ones by some 2.5e-3 of their norm (as far from float64 either way), and where a slice lies in a batch decides which it has:
// 65 x 128, 32 slices, against no unit split 3.2e-4 -> 9e-6, 46 x 90, 24 slices, 4.0e-4 -> 1.4e-5, at the same times.
constexpr int kStageFwd = 2 * kTileBytes + 256;      // K row tile, V^T column tile, 64 weights
template <bool UNIFORM_W, int SPLIT>
__device__ __forceinline__ void
forward_unit(char *buf0, char *buf1, int qb, int bh, const bf16raw *__restrict__ q, const bf16raw *__restrict__ k, const bf16raw *__restrict__ vt,
             const float *__restrict__ wtok, bf16raw *__restrict__ out, float *__restrict__ lse, int N, int Npad, int2 live, float c2, float ln_wref, bool common)
{
    static_assert(SPLIT == 1 || SPLIT == 2, "a stage holds two key tiles");
    constexpr int kStage = kStageFwd;
    constexpr int TILES = 4 / SPLIT;                 // query tiles of the workgroup
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, col = lane & 31, hl = lane >> 5;
    const int part = wave / TILES, qi = (qb * TILES + wave % TILES) * 32 + col;
    bf16x8 qop[4];
    {
        const bf16raw *qp = q + (size_t(bh) * N + min(qi, N - 1)) * kD + 8 * hl;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) qop[ks] = ld8(qp + 16 * ks);
    }
    f32x16 o0 = {0}, o1 = {0};
    float m = 0.f, l = 0.f;
    const bf16raw *kb = k + size_t(bh) * N * kD;
    const bf16raw *vb = vt + size_t(bh) * kD * Npad;
    const int nst = Npad >> 6;
    const Copies copies(wave, lane, N, Npad);
    auto request = [&](char *buf, int st) {
        const int t0 = 64 * st;
        copies.rows(kb, t0, buf);
        copies.cols(vb, t0, buf + kTileBytes);
        if (wave == 0) copies.floats(wtok + t0, buf + 2 * kTileBytes);
    };
    bool based = false;        // has the query met a logit above -infinity: only then does m mean anything
    auto stage = [&](const char *cur, char *nxt, int st) {
        if (st + 1 < nst) request(nxt, st + 1);
#pragma unroll
        for (int it = 0; it < 2 / SPLIT; ++it) {
            const int kt = SPLIT == 1 ? it : part;
            // Keys of weight zero (the pole row of the grid of App. A.1, the padding behind the last token) have no
            // term in the sums, so they must not enter the reference maximum either: a tile without a live key is
            // skipped, and in a mixed tile (longitude count not a multiple of 32) their logits are set to -inf.
            const int t0 = 64 * st + 32 * kt;
            if (t0 + 32 <= live.x || t0 >= live.y) continue;
            const bool mixed = !UNIFORM_W && (t0 < live.x || t0 + 32 > live.y);
            const float *wp = reinterpret_cast<const float *>(cur + 2 * kTileBytes) + 32 * kt + 16 * hl;
            float wk[16];
            if (!UNIFORM_W)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const float4 w = *reinterpret_cast<const float4 *>(wp + 4 * g);
                    wk[4 * g + 0] = w.x; wk[4 * g + 1] = w.y; wk[4 * g + 2] = w.z; wk[4 * g + 3] = w.w;
                }
            f32x16 s = {0};
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) s = mfma(row_operand(cur, col, hl, kt, ks), qop[ks], s);
            float x[16], e[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) x[i] = fmaf(s[i], c2, -m);
            if (mixed)
#pragma unroll
                for (int i = 0; i < 16; ++i) x[i] = wk[i] > 0.f ? x[i] : -INFINITY;
            // Fast path: exponentials relative to the current reference; a logit more than 2^8 above it shows in the
            // tile sum (all terms are positive), so the sum is the overflow test and no per-element maximum is taken.
            auto sum = [&]() {
                float p[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    if (UNIFORM_W) p[0] += e[i];
                    else p[i & 3] = fmaf(e[i], wk[i], p[i & 3]);
                }
                return UNIFORM_W ? p[0] : (p[0] + p[1]) + (p[2] + p[3]);
            };
#pragma unroll
            for (int i = 0; i < 16; ++i) e[i] = __builtin_amdgcn_exp2f(x[i]);
            float psum = sum();
            // the two half-wavefronts of a query exchange their maxima only when the reference has to move
            if (!__all(based) || __any(!(psum <= 256.f))) {
                float mx = -INFINITY;
#pragma unroll
                for (int i = 0; i < 16; ++i) mx = fmaxf(mx, x[i]);
                mx = fmaxf(mx, __shfl_xor(mx, 32));
                const float delta = based ? (mx > 8.f ? mx : 0.f) : (mx > -INFINITY ? mx : 0.f);
                const float corr = based ? __builtin_amdgcn_exp2f(-delta) : 1.f;
                based |= mx > -INFINITY;
                m += delta;
                l *= corr;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    o0[i] *= corr;
                    o1[i] *= corr;
                    e[i] = __builtin_amdgcn_exp2f(x[i] - delta);
                }
                psum = sum();
            }
            l = UNIFORM_W ? fmaf(psum, wp[0], l) : l + psum;
#pragma unroll
            for (int i = 0; i < 16; ++i) x[i] = e[i];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const bf16x8 pb = pack8(x + 8 * j);
                o0 = mfma(col_operand(cur + kTileBytes, col, hl, 0, kt, j), pb, o0);
                o1 = mfma(col_operand(cur + kTileBytes, col, hl, 1, kt, j), pb, o1);
            }
        }
        landed();          // everybody is done with `cur`, and the copies into `nxt` have landed
    };
    request(buf0, 0);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) arrived(qop[ks]);
    if (SPLIT == 2 && common && part != (live.x >> 5 & 1)) {
        const int t0 = live.x & ~31;
        const bf16raw *kp = kb + size_t(min(t0 + col, N - 1)) * kD + 8 * hl;
        f32x16 s = {0};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) s = mfma(ld8(kp + 16 * ks), qop[ks], s);
        float mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int key = t0 + 8 * (i >> 2) + 4 * hl + (i & 3);
            if (key >= live.x && key < live.y) mx = fmaxf(mx, s[i] * c2);
        }
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        based = mx > -INFINITY;
        m = based ? mx : 0.f;
    }
    landed();
    for (int st = 0; st < nst; st += 2) {
        stage(buf0, buf1, st);
        if (st + 1 < nst) stage(buf1, buf0, st + 1);
    }
    float lt = l + __shfl_xor(l, 32);
    if constexpr (SPLIT == 2) {
        // every wavefront is past its last stage: the buffers hold the second pair's results, one wavefront each
        constexpr int kSlot = 34 * 64;
        static_assert(kStage >= kSlot * 4, "LDS of the partial results");
        float *slot = reinterpret_cast<float *>(wave & 1 ? buf1 : buf0) + lane;
        if (part == 1) {
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                slot[i * 64] = o0[i];
                slot[(16 + i) * 64] = o1[i];
            }
            slot[32 * 64] = based ? m : -INFINITY;
            slot[33 * 64] = lt;
        }
        __syncthreads();
        if (part == 1) return;
        // A pair without a live key has o = l = 0 and the factor 0; NaN stays NaN through the sums.
        const float other = slot[32 * 64], top = fmaxf(based ? m : -1e30f, other);
        const float f = based ? __builtin_amdgcn_exp2f(m - top) : 1.f, g = __builtin_amdgcn_exp2f(other - top);
        lt = fmaf(slot[33 * 64], g, lt * f);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            o0[i] = fmaf(slot[i * 64], g, o0[i] * f);
            o1[i] = fmaf(slot[(16 + i) * 64], g, o1[i] * f);
        }
        m = top;
    }
    if (qi < N) {
        const float inv = 1.f / lt;
        bf16raw *ob = out + (size_t(bh) * N + qi) * kD + 4 * hl;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            bf16x4 a, b;
#pragma unroll
            for (int u = 0; u < 4; ++u) { a[u] = (__bf16)(o0[4 * g + u] * inv); b[u] = (__bf16)(o1[4 * g + u] * inv); }
            *reinterpret_cast<bf16x4 *>(ob + 8 * g) = a;
            *reinterpret_cast<bf16x4 *>(ob + 32 + 8 * g) = b;
        }
        if (hl == 0) lse[size_t(bh) * N + qi] = (m + log2f(lt)) * 0.6931471805599453f + ln_wref;
    }
}
template <bool UNIFORM_W>
__global__ void __launch_bounds__(256, 3)
global_fwd(const bf16raw *__restrict__ q, const bf16raw *__restrict__ k, const bf16raw *__restrict__ vt, const float *__restrict__ wtok,
           bf16raw *__restrict__ out, float *__restrict__ lse, int N, int Npad, Units units, int2 live, float c2, float ln_wref)
{
    __shared__ __attribute__((aligned(16))) char buf0[kStageFwd];
    __shared__ __attribute__((aligned(16))) char buf1[kStageFwd];
    take_unit(units, [&](auto split, int qb, int bh) {
        forward_unit<UNIFORM_W, decltype(split)::value>(buf0, buf1, qb, bh, q, k, vt, wtok, out, lse, N, Npad, live, c2, ln_wref, !units.halves);
    });
}

// The sums of a workgroup's second pair of wavefronts are added to those of the first, through the stage buffers (one
// for each wavefront of a pair; every wavefront is past its last stage).  True for the second pair, which is done.
template <int TERMS, int BYTES>
__device__ __forceinline__ bool join_pairs(f32x16 *const (&sums)[TERMS], char *buf, int part, int lane)
{
    static_assert(BYTES >= TERMS * 16 * 64 * 4, "LDS of the partial sums");
    float *slot = reinterpret_cast<float *>(buf) + lane;
    if (part == 1) {
#pragma unroll
        for (int t = 0; t < TERMS; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) slot[(16 * t + i) * 64] = (*sums[t])[i];
    }
    __syncthreads();
    if (part == 1) return true;
#pragma unroll
    for (int t = 0; t < TERMS; ++t)
#pragma unroll
        for (int i = 0; i < 16; ++i) (*sums[t])[i] += slot[(16 * t + i) * 64];
    return false;
}

// Backward (App. B.4 with every token in every neighborhood).  With w_j = omega_j / max omega and
// L_i = log2(e) (lse_i - ln max omega):  p_ij = w_j pt_ij,  pt_ij = 2^(log2(e) scale q_i.k_j - L_i),
// dS_ij = p_ij (dout_i.v_j - D_i).  The factor w_j never enters the inner loops: the key-side kernel
// multiplies its finished sums by w_j (the lane's own key), the query-side kernel contracts with
// K^T premultiplied by w_j (prepare_operands).
//
// Key side: a workgroup owns 128 keys (one 32-key tile per wavefront) and streams the queries in stages
// of 64: Q and dout token-major (for S = Q K^T and dP = dout V^T, which land with lane = key,
// registers = 16 queries), Q^T and dout^T channel-major (dV^T += dout^T Pt, dK^T += Q^T dSt), L and D.
// SPLIT = 2: two pairs of wavefronts take every other query tile of the same 64 keys, and their sums meet in LDS.
constexpr int kStageDkdv = 4 * kTileBytes + 512;     // Q, dout row tiles; Q^T, dout^T column tiles; L, D
template <int SPLIT>
__device__ __forceinline__ void
dkdv_unit(char *buf0, char *buf1, int kb, int bh, const bf16raw *__restrict__ q, const bf16raw *__restrict__ k, const bf16raw *__restrict__ v,
          const bf16raw *__restrict__ go, const bf16raw *__restrict__ qt, const bf16raw *__restrict__ got, const float *__restrict__ wtok,
          const float *__restrict__ L2, const float *__restrict__ Dv, bf16raw *__restrict__ dk, bf16raw *__restrict__ dv, int N, int Npad, float c2,
          float scale)
{
    constexpr int kStage = kStageDkdv;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, col = lane & 31, hl = lane >> 5;
    constexpr int TILES = 4 / SPLIT;                 // key tiles of the workgroup
    const int part = wave / TILES, ki = (kb * TILES + wave % TILES) * 32 + col;
    bf16x8 kop[4], vop[4];
    {
        const size_t row = (size_t(bh) * N + min(ki, N - 1)) * kD + 8 * hl;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) { kop[ks] = ld8(k + row + 16 * ks); vop[ks] = ld8(v + row + 16 * ks); }
    }
    f32x16 dk0 = {0}, dk1 = {0}, dv0 = {0}, dv1 = {0};
    const bf16raw *qb = q + size_t(bh) * N * kD, *gb = go + size_t(bh) * N * kD;
    const bf16raw *qtb = qt + size_t(bh) * kD * Npad, *gtb = got + size_t(bh) * kD * Npad;
    const float *Lb = L2 + size_t(bh) * Npad, *Db = Dv + size_t(bh) * Npad;
    const int nst = Npad >> 6;
    const Copies copies(wave, lane, N, Npad);
    auto request = [&](char *buf, int st) {
        const int t0 = 64 * st;
        copies.rows(qb, t0, buf);
        copies.rows(gb, t0, buf + kTileBytes);
        copies.cols(qtb, t0, buf + 2 * kTileBytes);
        copies.cols(gtb, t0, buf + 3 * kTileBytes);
        if (wave == 0) copies.floats(Lb + t0, buf + 4 * kTileBytes);
        if (wave == 1) copies.floats(Db + t0, buf + 4 * kTileBytes + 256);
    };
    auto stage = [&](const char *cur, char *nxt, int st) {
        if (st + 1 < nst) request(nxt, st + 1);
#pragma unroll
        for (int it = 0; it < 2 / SPLIT; ++it) {
            const int h = SPLIT == 1 ? it : part;
            const float *Lp = reinterpret_cast<const float *>(cur + 4 * kTileBytes) + 32 * h + 16 * hl;
            // dP starts from -D_i (the 16 queries this lane's registers stand for)
            f32x16 s = {0}, dp;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float4 Dr = *reinterpret_cast<const float4 *>(Lp + 64 + 4 * g);
                dp[4 * g + 0] = Dr.x; dp[4 * g + 1] = Dr.y; dp[4 * g + 2] = Dr.z; dp[4 * g + 3] = Dr.w;
            }
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                s = mfma(row_operand(cur, col, hl, h, ks), kop[ks], s);
                dp = mfma(row_operand(cur + kTileBytes, col, hl, h, ks), vop[ks], dp);
            }
            float p[16], ds[16];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float4 Lr = *reinterpret_cast<const float4 *>(Lp + 4 * g);
                p[4 * g + 0] = fmaf(s[4 * g + 0], c2, -Lr.x);
                p[4 * g + 1] = fmaf(s[4 * g + 1], c2, -Lr.y);
                p[4 * g + 2] = fmaf(s[4 * g + 2], c2, -Lr.z);
                p[4 * g + 3] = fmaf(s[4 * g + 3], c2, -Lr.w);
            }
            __builtin_amdgcn_sched_barrier(0);          // exponents, exponentials, products in three groups: 1106 -> 1075 us on 65 x 128, 32 slices
#pragma unroll
            for (int i = 0; i < 16; ++i) p[i] = __builtin_amdgcn_exp2f(p[i]);
#pragma unroll
            for (int i = 0; i < 16; ++i) ds[i] = p[i] * dp[i];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const bf16x8 pb = pack8(p + 8 * j), sb = pack8(ds + 8 * j);
                dv0 = mfma(col_operand(cur + 3 * kTileBytes, col, hl, 0, h, j), pb, dv0);
                dv1 = mfma(col_operand(cur + 3 * kTileBytes, col, hl, 1, h, j), pb, dv1);
                dk0 = mfma(col_operand(cur + 2 * kTileBytes, col, hl, 0, h, j), sb, dk0);
                dk1 = mfma(col_operand(cur + 2 * kTileBytes, col, hl, 1, h, j), sb, dk1);
            }
        }
        landed();          // everybody is done with `cur`, and the copies into `nxt` have landed
    };
    request(buf0, 0);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        arrived(kop[ks]);
        arrived(vop[ks]);
    }
    landed();
    for (int st = 0; st < nst; st += 2) {
        stage(buf0, buf1, st);
        if (st + 1 < nst) stage(buf1, buf0, st + 1);
    }
    if constexpr (SPLIT == 2) {
        f32x16 *const sums[4] = {&dk0, &dk1, &dv0, &dv1};
        if (join_pairs<4, kStage>(sums, wave & 1 ? buf1 : buf0, part, lane)) return;
    }
    if (ki < N) {
        const float wk = wtok[ki], wks = wk * scale;
        const bool live = wk > 0.f;
        bf16raw *dkb = dk + (size_t(bh) * N + ki) * kD + 4 * hl, *dvb = dv + (size_t(bh) * N + ki) * kD + 4 * hl;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            bf16x4 a, b, c, d;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                // a key of weight zero gets exactly zero (its unweighted sums may have overflowed: its logits are not
                // bounded by any logsumexp)
                a[u] = (__bf16)(live ? dk0[4 * g + u] * wks : 0.f); b[u] = (__bf16)(live ? dk1[4 * g + u] * wks : 0.f);
                c[u] = (__bf16)(live ? dv0[4 * g + u] * wk : 0.f); d[u] = (__bf16)(live ? dv1[4 * g + u] * wk : 0.f);
            }
            *reinterpret_cast<bf16x4 *>(dkb + 8 * g) = a;
            *reinterpret_cast<bf16x4 *>(dkb + 32 + 8 * g) = b;
            *reinterpret_cast<bf16x4 *>(dvb + 8 * g) = c;
            *reinterpret_cast<bf16x4 *>(dvb + 32 + 8 * g) = d;
        }
    }
}
__global__ void __launch_bounds__(256, 2)
global_bwd_dkdv(const bf16raw *__restrict__ q, const bf16raw *__restrict__ k, const bf16raw *__restrict__ v, const bf16raw *__restrict__ go,
                const bf16raw *__restrict__ qt, const bf16raw *__restrict__ got, const float *__restrict__ wtok, const float *__restrict__ L2,
                const float *__restrict__ Dv, bf16raw *__restrict__ dk, bf16raw *__restrict__ dv, int N, int Npad, Units units, float c2, float scale)
{
    __shared__ __attribute__((aligned(16))) char buf0[kStageDkdv];
    __shared__ __attribute__((aligned(16))) char buf1[kStageDkdv];
    take_unit(units, [&](auto split, int kb, int bh) {
        dkdv_unit<decltype(split)::value>(buf0, buf1, kb, bh, q, k, v, go, qt, got, wtok, L2, Dv, dk, dv, N, Npad, c2, scale);
    });
}

// Query side: a workgroup owns 128 queries and streams the keys in stages of 64: K and V token-major
// (S^T = K Q^T and dP^T = V dout^T land with lane = query, registers = 16 keys) and w K^T channel-major
// (dQ^T += (w K)^T dSt^T).
// Some keys may have weight zero (a pole row of weight zero, padding behind the last token; live: the others).  Their logits are not
// bounded by the logsumexp, so 2^(x - L) may overflow and inf * (w k = 0) would poison dq: in tiles that hold such keys the exponent is
// capped at 100 (a key of positive weight stays below log2(max omega / omega_j), a few tens at most), which keeps the
// factor finite and the product with the zero row exactly zero.  (Exponents first, then exponentials and products, with the cap in a branch:
// 804 -> 765 us on 65 x 128, 32 slices, which needs no cap; 46 x 90, 24 slices, the whole backward 433 -> 403.)
// SPLIT as in the forward.
constexpr int kStageDq = 3 * kTileBytes;             // K, V row tiles; (w K)^T column tile
template <int SPLIT>
__device__ __forceinline__ void
dq_unit(char *buf0, char *buf1, int qb, int bh, const bf16raw *__restrict__ q, const bf16raw *__restrict__ k, const bf16raw *__restrict__ v,
        const bf16raw *__restrict__ go, const bf16raw *__restrict__ ktw, const float *__restrict__ L2, const float *__restrict__ Dv,
        bf16raw *__restrict__ dq, int N, int Npad, int2 live, float c2, float scale)
{
    constexpr int kStage = kStageDq;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63, col = lane & 31, hl = lane >> 5;
    constexpr int TILES = 4 / SPLIT;                 // query tiles of the workgroup
    const int part = wave / TILES, qi = (qb * TILES + wave % TILES) * 32 + col;
    bf16x8 qop[4], gop[4];
    {
        const size_t row = (size_t(bh) * N + min(qi, N - 1)) * kD + 8 * hl;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) { qop[ks] = ld8(q + row + 16 * ks); gop[ks] = ld8(go + row + 16 * ks); }
    }
    float Lq = L2[size_t(bh) * Npad + min(qi, N - 1)];
    const float Dq = Dv[size_t(bh) * Npad + min(qi, N - 1)];
    f32x16 dq0 = {0}, dq1 = {0}, nd;     // nd: -D_q in every register, the start value of dout.v
#pragma unroll
    for (int i = 0; i < 16; ++i) nd[i] = Dq;
    const bf16raw *kb = k + size_t(bh) * N * kD, *vb = v + size_t(bh) * N * kD;
    const bf16raw *ktb = ktw + size_t(bh) * kD * Npad;
    const int nst = Npad >> 6;
    const Copies copies(wave, lane, N, Npad);
    auto request = [&](char *buf, int st) {
        const int t0 = 64 * st;
        copies.rows(kb, t0, buf);
        copies.rows(vb, t0, buf + kTileBytes);
        copies.cols(ktb, t0, buf + 2 * kTileBytes);
    };
    auto stage = [&](const char *cur, char *nxt, int st) {
        if (st + 1 < nst) request(nxt, st + 1);
#pragma unroll
        for (int it = 0; it < 2 / SPLIT; ++it) {
            const int h = SPLIT == 1 ? it : part;
            f32x16 s = {0}, dp = nd;
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) {
                s = mfma(row_operand(cur, col, hl, h, ks), qop[ks], s);
                dp = mfma(row_operand(cur + kTileBytes, col, hl, h, ks), gop[ks], dp);
            }
            float ds[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) ds[i] = fmaf(s[i], c2, -Lq);
            const int t0 = 64 * st + 32 * h;
            if (t0 < live.x || t0 + 32 > live.y)
#pragma unroll
                for (int i = 0; i < 16; ++i) ds[i] = fminf(ds[i], 100.f);
#pragma unroll
            for (int i = 0; i < 16; ++i) ds[i] = __builtin_amdgcn_exp2f(ds[i]) * dp[i];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const bf16x8 sb = pack8(ds + 8 * j);
                dq0 = mfma(col_operand(cur + 2 * kTileBytes, col, hl, 0, h, j), sb, dq0);
                dq1 = mfma(col_operand(cur + 2 * kTileBytes, col, hl, 1, h, j), sb, dq1);
            }
        }
        landed();          // everybody is done with `cur`, and the copies into `nxt` have landed
    };
    request(buf0, 0);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
        arrived(qop[ks]);
        arrived(gop[ks]);
    }
    arrived(Lq);
    arrived(nd);
    landed();
    for (int st = 0; st < nst; st += 2) {
        stage(buf0, buf1, st);
        if (st + 1 < nst) stage(buf1, buf0, st + 1);
    }
    if constexpr (SPLIT == 2) {
        f32x16 *const sums[2] = {&dq0, &dq1};
        if (join_pairs<2, kStage>(sums, wave & 1 ? buf1 : buf0, part, lane)) return;
    }
    if (qi < N) {
        bf16raw *dqb = dq + (size_t(bh) * N + qi) * kD + 4 * hl;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            bf16x4 a, b;
#pragma unroll
            for (int u = 0; u < 4; ++u) { a[u] = (__bf16)(dq0[4 * g + u] * scale); b[u] = (__bf16)(dq1[4 * g + u] * scale); }
            *reinterpret_cast<bf16x4 *>(dqb + 8 * g) = a;
            *reinterpret_cast<bf16x4 *>(dqb + 32 + 8 * g) = b;
        }
    }
}
__global__ void __launch_bounds__(256, 3)
global_bwd_dq(const bf16raw *__restrict__ q, const bf16raw *__restrict__ k, const bf16raw *__restrict__ v, const bf16raw *__restrict__ go,
              const bf16raw *__restrict__ ktw, const float *__restrict__ L2, const float *__restrict__ Dv, bf16raw *__restrict__ dq, int N, int Npad,
              Units units, int2 live, float c2, float scale)
{
    __shared__ __attribute__((aligned(16))) char buf0[kStageDq];
    __shared__ __attribute__((aligned(16))) char buf1[kStageDq];
    take_unit(units, [&](auto split, int qb, int bh) {
        dq_unit<decltype(split)::value>(buf0, buf1, qb, bh, q, k, v, go, ktw, L2, Dv, dq, N, Npad, live, c2, scale);
    });
}

// Whether the wavefronts of a workgroup share the streamed side (SPLIT = 2).  It pays while the launch of workgroups of
// 128 tokens leaves compute units idle or their second wavefront of a SIMD missing; beyond that the second workgroup of
// a compute unit hides the same waits, and the split only halves the reuse of a staged tile.  Times with SPLIT = 1 -> 2,
// in microseconds of the whole call, by the number of workgroups of 128 tokens (46 x 90 unless said):
//     forward        33: 85 -> 50   132: 91 -> 63   264: 108 -> 81   320 (25 x 47): 38 -> 32   396: 116 -> 119
//     query side     33: 224 -> 184   132: 235 -> 209   264: 292 -> 280   320 (25 x 47): 112 -> 110   396: 360 -> 379
//     key side       33: 224 -> 192   132: 235 -> 220   224 (21 x 40): 67 -> 67   260 (65 x 128): 511 -> 529
// Split units are counted by 64 tokens: by twice the units of 128, slices that end within the first half of one had workgroups with nothing to do
// among the others, and compute units two others (12 x 24, 48 slices: 240 workgroups among 288, backward 25.4 us; 21.1).
// (at most two workgroups of the key side fit a compute unit, three of the others: hence two lines).
constexpr long kSplitBlocks = 320, kSplitBlocksKeySide = 256;
// Larger launches: what an XCD's 32 compute units do not share out evenly, where that is at most half a unit for each, goes in halves, so that
// the last compute units end half a unit after the others and not a whole one.  Forward / backward, us: 65 x 128, 32 slices (8.1
// units for a compute unit) 634 / 2059 -> 593 / 1966; 8 slices (2.0) 223 / 667 -> 192 / 576; 46 x 90, 24 (3.1) 204 / 480 -> 178 / 427.
constexpr int kUnitsXcd = 32;
Units split_units(int nbh, int N, long most)
{
    Units u;
    u.tokens = N;
    u.halves = long(nbh) * ((N + 127) / 128) <= most;
    u.per_slice = u.halves ? (N + 63) / 64 : (N + 127) / 128;
    u.all = nbh * u.per_slice;
    u.per_xcd = (u.all + 7) / 8;
    const int rest = u.per_xcd % kUnitsXcd;
    u.whole = !u.halves && 2 * rest <= kUnitsXcd ? u.per_xcd - rest : u.per_xcd;
    return u;
}
dim3 split_grid(const Units &u) { return dim3(8u * unsigned(u.whole + 2 * (u.per_xcd - u.whole))); }

// The tokens of positive weight.  Latitudes of weight zero are poles (that of the grid of App. A.1; no other grid has one), the first or the
// last ones.
int2 live_tokens(const s2_grid_t *g)
{
    const std::vector<int> &z = g->zero_lat;         // in ascending order
    int first = 0, last = g->nlat_in;
    for (size_t i = 0; i < z.size(); ++i) first += z[i] == first;
    for (size_t i = z.size(); i-- > 0 && last > first;) last -= z[i] == last - 1;
    return make_int2(first * g->nlon_in, last * g->nlon_in);
}

int check_global(const s2_grid_t *g, int batch, int heads, int d, int dtype)
{
    if (!g) return s2_fail(S2_ERR_INVALID_ARG, "grid is NULL");
    if (batch < 1 || heads < 1 || d < 1) return s2_fail(S2_ERR_INVALID_ARG, "batch, heads, d must be >= 1");
    if (long(batch) * heads > 65535) return s2_fail(S2_ERR_INVALID_ARG, "batch*heads too large");
    if (g->nlat_in != g->nlat_out || g->nlon_in != g->nlon_out)
        return s2_fail(S2_ERR_INVALID_ARG, "global attention needs identical input and output grids");
    if (dtype != S2_BF16) return s2_fail(S2_ERR_UNSUPPORTED, "global attention supports S2_BF16 only");
    if (d != kD) return s2_fail(S2_ERR_UNSUPPORTED, "global attention supports head dimension 64 only");
    if (!g->on_device) return s2_fail(S2_ERR_DEVICE, "grid handle has no device tables (no HIP device at init)");
    // one workgroup per unit of 128 tokens of a slice, two for units that go in halves: the grid must fit 31 bits
    const long nunits = long(batch) * heads * ((long(g->nlat_in) * g->nlon_in + 127) / 128);
    if (nunits > (1l << 30)) return s2_fail(S2_ERR_INVALID_ARG, "batch*heads*tokens too large for one launch");
    return S2_OK;
}

// the kernels move 16-byte pieces (LDS-direct copies, vector loads and stores)
bool misaligned(const void *p, size_t a = 16) { return reinterpret_cast<uintptr_t>(p) % a != 0; }

size_t transposed_bytes(const s2_grid_t *g, int nbh) { return size_t(nbh) * kD * g->npad_tok * sizeof(bf16raw); }

void launch_prepare(const PrepArgs &a, int nops, int nbh, int N, int Npad, hipStream_t st)
{
    hipLaunchKernelGGL(prepare_operands, dim3(Npad / 64, nbh, nops), dim3(256), 0, st, a, N, Npad);
}

}  // namespace

extern "C" size_t s2_attn_global_fwd_workspace_bytes(const s2_grid_t *g, int batch, int heads, int d, int dtype)
{
    (void)d; (void)dtype;
    if (!g || batch < 1 || heads < 1) return 0;
    return transposed_bytes(g, batch * heads);
}

extern "C" size_t s2_attn_global_bwd_workspace_bytes(const s2_grid_t *g, int batch, int heads, int d, int dtype)
{
    (void)d; (void)dtype;
    if (!g || batch < 1 || heads < 1) return 0;
    const size_t npad = size_t(batch) * heads * g->npad_tok;
    return 3 * transposed_bytes(g, batch * heads) + 2 * ((npad * sizeof(float) + 255) / 256 * 256);
}

extern "C" int s2_attn_global_fwd(const s2_grid_t *g, int batch, int heads, int d, int dtype, float scale,
                                  const void *q, const void *k, const void *v, void *out, float *lse,
                                  void *workspace, size_t workspace_bytes, void *hip_stream)
{
    int rc = check_global(g, batch, heads, d, dtype);
    if (rc) return rc;
    if (!q || !k || !v || !out || !lse) return s2_fail(S2_ERR_INVALID_ARG, "NULL tensor pointer");
    if (misaligned(q) || misaligned(k) || misaligned(v) || misaligned(out))
        return s2_fail(S2_ERR_INVALID_ARG, "tensor pointers must be 16-byte aligned");
    if (!workspace || workspace_bytes < s2_attn_global_fwd_workspace_bytes(g, batch, heads, d, dtype))
        return s2_fail(S2_ERR_WORKSPACE, "workspace missing or smaller than s2_attn_global_fwd_workspace_bytes()");
    if (misaligned(workspace, 256)) return s2_fail(S2_ERR_WORKSPACE, "workspace must be 256-byte aligned");
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const int nbh = batch * heads, N = g->nlat_in * g->nlon_in, Npad = g->npad_tok;
    PrepArgs pa{};
    pa.op[0] = {static_cast<const bf16raw *>(v), static_cast<bf16raw *>(workspace), g->dev_w_tok};
    pa.stat_op = -1;
    launch_prepare(pa, 1, nbh, N, Npad, st);
    S2TraceScope tr("global_fwd", double(nbh) * N * N, st);
    const int2 live = live_tokens(g);
    const Units units = split_units(nbh, N, kSplitBlocks);
    hipLaunchKernelGGL(g->nlon_in % 32 == 0 ? global_fwd<true> : global_fwd<false>, split_grid(units), dim3(256), 0, st,
                       static_cast<const bf16raw *>(q), static_cast<const bf16raw *>(k), static_cast<const bf16raw *>(workspace), g->dev_w_tok,
                       static_cast<bf16raw *>(out), lse, N, Npad, units, live, scale * kLog2e, g->dt.ln_omega_ref);
    S2_HIP_CHECK(hipGetLastError());
    return S2_OK;
}

extern "C" int s2_attn_global_bwd(const s2_grid_t *g, int batch, int heads, int d, int dtype, float scale,
                                  const void *q, const void *k, const void *v, const void *out, const float *lse,
                                  const void *dout, void *dq, void *dk, void *dv, void *workspace,
                                  size_t workspace_bytes, void *hip_stream)
{
    int rc = check_global(g, batch, heads, d, dtype);
    if (rc) return rc;
    if (!q || !k || !v || !out || !lse || !dout || !dq || !dk || !dv)
        return s2_fail(S2_ERR_INVALID_ARG, "NULL tensor pointer");
    if (misaligned(q) || misaligned(k) || misaligned(v) || misaligned(out) || misaligned(dout) || misaligned(dq) ||
        misaligned(dk) || misaligned(dv))
        return s2_fail(S2_ERR_INVALID_ARG, "tensor pointers must be 16-byte aligned");
    if (!workspace || workspace_bytes < s2_attn_global_bwd_workspace_bytes(g, batch, heads, d, dtype))
        return s2_fail(S2_ERR_WORKSPACE, "workspace missing or smaller than s2_attn_global_bwd_workspace_bytes()");
    if (misaligned(workspace, 256)) return s2_fail(S2_ERR_WORKSPACE, "workspace must be 256-byte aligned");
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const int nbh = batch * heads, N = g->nlat_in * g->nlon_in, Npad = g->npad_tok;
    const size_t tb = transposed_bytes(g, nbh);
    const size_t sb = (size_t(nbh) * Npad * sizeof(float) + 255) / 256 * 256;
    char *ws = static_cast<char *>(workspace);
    bf16raw *qt = reinterpret_cast<bf16raw *>(ws), *kt = reinterpret_cast<bf16raw *>(ws + tb),
            *got = reinterpret_cast<bf16raw *>(ws + 2 * tb);
    float *L2 = reinterpret_cast<float *>(ws + 3 * tb), *Dv = reinterpret_cast<float *>(ws + 3 * tb + sb);
    PrepArgs pa{};
    pa.op[0] = {static_cast<const bf16raw *>(q), qt, nullptr};
    pa.op[1] = {static_cast<const bf16raw *>(k), kt, g->dev_w_tok};
    pa.op[2] = {static_cast<const bf16raw *>(dout), got, nullptr};
    pa.stat_op = 2;
    pa.o = static_cast<const bf16raw *>(out);
    pa.lse = lse;
    pa.L2 = L2;
    pa.D = Dv;
    pa.ln_wref = g->dt.ln_omega_ref;
    launch_prepare(pa, 3, nbh, N, Npad, st);
    const float c2 = scale * kLog2e;
    {
        S2TraceScope tr("global_bwd_dkdv", double(nbh) * N * N, st);
        const Units units = split_units(nbh, N, kSplitBlocksKeySide);
        hipLaunchKernelGGL(global_bwd_dkdv, split_grid(units), dim3(256), 0, st, static_cast<const bf16raw *>(q), static_cast<const bf16raw *>(k),
                           static_cast<const bf16raw *>(v), static_cast<const bf16raw *>(dout), qt, got, g->dev_w_tok, L2, Dv,
                           static_cast<bf16raw *>(dk), static_cast<bf16raw *>(dv), N, Npad, units, c2, scale);
    }
    S2TraceScope tr("global_bwd_dq", double(nbh) * N * N, st);
    const Units units = split_units(nbh, N, kSplitBlocks);
    const int2 live = live_tokens(g);
    hipLaunchKernelGGL(global_bwd_dq, split_grid(units), dim3(256), 0, st, static_cast<const bf16raw *>(q),
                       static_cast<const bf16raw *>(k), static_cast<const bf16raw *>(v), static_cast<const bf16raw *>(dout), kt, L2, Dv,
                       static_cast<bf16raw *>(dq), N, Npad, units, live, c2, scale);
    S2_HIP_CHECK(hipGetLastError());
    return S2_OK;
}
