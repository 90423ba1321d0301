// Walks the segments, rows, chunks and workgroups that s2_grid_init makes for the forward by columns (S2ColumnRow) the way the kernel
// does, on the host: every owner meets its neighbors, each once, and nothing else, and the owners of a segment's rows meet the same chunks
// in the same stages, counted from their columns, whatever column and wavefront.
// Arguments: grid type, four sizes, theta.  Prints "none" where the grid has no such tables.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <tuple>

#include "s2_nattn_kernels.h"

int s2_nattn_tiled_configure() { return 0; }
int s2_nattn_bwd_tiled_configure() { return 0; }
int s2_nattn_stream_configure() { return 0; }
int s2_nattn_band_configure() { return 0; }
int s2_static_scratch_setup(int) { return 0; }

static int check(const s2_grid &g)
{
    const s2_grid::Columns &p = g.columns;
    const int n_own = int(g.vo_lo.size()), bmax = int(g.vo_arc.size() / g.vo_lo.size()), nU = g.nlon_in;
    std::vector<int> seen(size_t(n_own) * nU, 0);
    std::map<int, std::vector<std::tuple<int, int, int, int>>> order;      // by segment: part, stage, row, column from the owner's
    for (const int2 &wg : p.list)
        for (int wave = 0; wave < kS2PatchWaves; ++wave) {
            const int u = wg.y + 4 * wave;
            if (u >= nU) continue;
            std::vector<std::tuple<int, int, int, int>> chunks;
            std::vector<std::map<std::pair<int, int>, int>> met(16);
            const int first = p.seg[2 * wg.x].x;
            for (int part = wg.x;; ++part) {
                const int4 t0 = p.seg[2 * part], t1 = p.seg[2 * part + 1];
                if (t0.x != first || t0.y != 4 || t0.z != 0 || t0.w > kS2ColumnRows) return 1;
                for (int i = 0; i < t0.w; ++i) {
                    const S2ColumnRow &r = p.rows[t1.y + i];
                    const int end = i + 1 < t0.w ? p.rows[t1.y + i + 1].before : t1.x;
                    for (int X = r.before; X < end; ++X) {
                        const int col = r.col + 4 * X + wg.y, d = col + 3 - u - int(short(r.uni & 0xffff));
                        if (col < -2 * nU || col + 3 + 2 * nU >= 1 << 22 || col >= 1 << 17 || col < -(1 << 17)) return 2;
                        if (unsigned(d) >= (unsigned(r.uni) >> 16) + 3) continue;
                        chunks.push_back({part - wg.x, X / kS2ColumnStage, r.row, col - u});
                        for (int n = 0; n < 16; ++n) {
                            const unsigned rel = unsigned(col - (u + int(short(r.arc[n] & 0xffff))));
                            for (int j = 0; j < 4; ++j)
                                if (rel + j < (r.arc[n] >> 16)) ++met[n][{r.row, ((col + j) % nU + nU) % nU}];
                        }
                    }
                }
                if (t1.z == 0) break;
            }
            auto it = order.emplace(wg.x, chunks).first;
            if (it->second != chunks) return 3;
            for (int n = 0; n < 16 && first + n < n_own; ++n) {
                const int own = first + n;
                ++seen[size_t(own) * nU + u];
                size_t want = 0;
                for (int b = 0; b < g.vo_n[own]; ++b) {
                    const int2 x = g.vo_arc[size_t(own) * bmax + b];
                    for (int c = 0; c < x.y; ++c, ++want) {
                        auto at = met[n].find({g.vo_lo[own] + b, ((u + x.x + c) % nU + nU) % nU});
                        if (at == met[n].end() || at->second != 1) return 4;
                    }
                }
                if (want != met[n].size()) return 5;
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
    if (g->columns.list.empty()) {
        printf("none\n");
        return 0;
    }
    const int rc = check(*g);
    s2_grid_destroy(g);
    printf("%d\n", rc);
    return rc;
}
