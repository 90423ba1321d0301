// Walks the segments, rows, chunks and patches that s2_grid_init makes for the patch kernels (s2_nattn_patch_impl.h) the way the
// kernels do, on the host (of either list of workgroups, the one for small launches too), and compares what every owner meets with the arc tables: each neighbor once, and nothing else.  Also
// prints how many chunks more than the circle has a wavefront walks at most on a row of which an owner meets all.
// Arguments: grid type, four sizes, theta.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <map>

#include "s2_nattn_kernels.h"

int s2_nattn_tiled_configure() { return 0; }
int s2_nattn_bwd_tiled_configure() { return 0; }
int s2_nattn_stream_configure() { return 0; }
int s2_nattn_band_configure() { return 0; }
int s2_static_scratch_setup(int) { return 0; }

static int check(const s2_grid::Patches &p, const std::vector<int2> &list, const std::vector<int> &blo, const std::vector<int> &bn, const std::vector<int2> &arc, int nU, int c_walk,
                 double &more)
{
    const int n_own = int(blo.size()), bmax = int(arc.size() / blo.size());
    const int S = p.step, nW = S * nU;
    if (S != (c_walk * nU < 1 << 15 ? c_walk : 1)) return 7;      // whole latitudes wherever 16 bits hold their columns, else classes
    std::vector<int> seen(size_t(n_own) * nU, 0);
    for (int2 wg : list) {
        const int share = wg.y >> 16;                 // log2 of the wavefronts that share a patch
        wg.y &= 0xffff;
        const int4 s0 = p.seg[2 * wg.x];
        const int rows = 1 << s0.y, W = 16 >> s0.y;
        for (int wave = 0; wave < kS2PatchWaves >> share; ++wave)
            for (int n = 0; n < 16; ++n) {
                const int own = s0.x + n / W, wc = wg.y + wave * W, u = wc + n % W;
                if (own >= n_own || u >= nU || n / W >= rows) continue;
                ++seen[size_t(own) * nU + u];
                std::map<std::pair<int, int>, int> met;
                for (int part = wg.x;; ++part) {
                const int4 t0 = p.seg[2 * part], t1 = p.seg[2 * part + 1];
                if (t0.x != s0.x || t0.y != s0.y || t0.w > kS2PatchRows) return 1;
                for (int i = 0; i < t0.w; ++i) {
                    const S2PatchRow &r = p.rows[t1.y + i];
                    const int end = i + 1 < t0.w ? p.rows[t1.y + i + 1].before : t1.x;
                    int walked = 0;
                    for (int X = r.before; X < end; ++X) {
                        const int col = r.col + 4 * X + S * wg.y, d = col + 3 - S * wc - int(short(r.uni & 0xffff));
                        if (col < -2 * nW || col + 3 + 2 * nW >= 1 << 22 || col >= 1 << 17 || col < -(1 << 17)) return 2;    // what wrap_col and a list entry hold
                        const unsigned a = r.arc[n / W], rel = unsigned(col - (S * u + int(short(a & 0xffff))));
                        const bool listed = unsigned(d) < (unsigned(r.uni) >> 16) + S * (W - 1) + 3;
                        walked += listed;
                        for (int j = 0; j < 4; ++j)
                            if (rel + j < (a >> 16)) {
                                if (!listed) return 3;
                                const int at = ((col + j) % nW + nW) % nW;
                                ++met[{(t0.z + i) * S + at % S, at / S}];
                            }
                    }
                    if (int(r.arc[n / W] >> 16) >= nW) more = std::max(more, walked - nW / 4.0);
                }
                if (t1.z == 0) break;
                }
                size_t want = 0;
                for (int b = 0; b < bn[own]; ++b) {
                    const int2 x = arc[size_t(own) * bmax + b];
                    for (int c = 0; c < x.y; ++c, ++want) {
                        auto it = met.find({blo[own] + b, ((u + x.x + c) % nU + nU) % nU});
                        if (it == met.end() || it->second != 1) return 4;
                    }
                }
                if (want != met.size()) return 5;
            }
    }
    for (int s : seen)
        if (s != 1) return 6;
    return 0;
}

int main(int argc, char **argv)
{
    s2_grid_t *g = nullptr;
    if (argc != 7 || s2_grid_init(atoi(argv[1]), atoi(argv[2]), atoi(argv[3]), atoi(argv[4]), atoi(argv[5]), atof(argv[6]), &g) != S2_OK) return 100;
    const int nU = g->nlon_in < g->nlon_out ? g->nlon_in : g->nlon_out;
    double more_a = 0.0, more_b = 0.0;
    int a = check(g->vo_patch, g->vo_patch.list, g->vo_lo, g->vo_n, g->vo_arc, nU, g->pscale, more_a),
        b = check(g->vi_patch, g->vi_patch.list, g->vi_lo, g->vi_n, g->vi_arc, nU, g->upscale, more_b);
    for (int i = 0; i < 2; ++i) {
        if (a == 0) a = check(g->vo_patch, g->vo_patch.split[i], g->vo_lo, g->vo_n, g->vo_arc, nU, g->pscale, more_a);
        if (b == 0) b = check(g->vi_patch, g->vi_patch.split[i], g->vi_lo, g->vi_n, g->vi_arc, nU, g->upscale, more_b);
        if (a == 0 && g->vo_patch.split[i].size() <= g->vo_patch.list.size() && nU > 32) a = 8;       // the longest are split
    }
    s2_grid_destroy(g);
    printf("%d %d %g %g\n", a, b, more_a, more_b);
    return a ? a : b ? 10 + b : 0;
}
