// Host check of the coarse tiles' lists (csrc/coarse_tiles.hpp, the functions
// the set-up kernel calls) against lists found by walking the rows of A0: for
// lattices of every kind of axis, each tile's box, rings, corners and columns,
// the strides, and that every entry of the lists is written once.
#include <algorithm>
#include <cstdio>
#include <map>
#include <vector>

#include "../paper_2109_03592_amd/csrc/coarse_tiles.hpp"

using namespace sem;

static int fails = 0;
#define CHECK(cond, ...)                        \
    do {                                        \
        if (!(cond) && fails++ < 10) {          \
            std::printf("FAIL %s: ", #cond);    \
            std::printf(__VA_ARGS__);           \
            std::printf("\n");                  \
        }                                       \
    } while (0)

static void check(const int nel[3], const int per[3], int edge, int depth, bool holes)
{
    TileGeom g{};
    std::vector<int> vd(3);
    for (int a = 0; a < 3; ++a) {
        g.nel[a] = nel[a];
        g.periodic[a] = per[a];
        g.vd[a] = nel[a] + 1 - per[a];
        g.nt[a] = (g.vd[a] + edge - 1) / edge;
    }
    g.depth = depth;
    tile_strides(g);
    const int nv = g.vd[0] * g.vd[1] * g.vd[2], E = nel[0] * nel[1] * nel[2], nt = g.nt[0] * g.nt[1] * g.nt[2];
    // corners and rows from the elements
    std::vector<std::vector<int>> corner(nv), row(nv);
    std::vector<double> d0inv(nv, 1.0);
    if (holes)
        for (int v = 0; v < nv; v += 3) d0inv[v] = 0.0;
    for (int e = 0; e < E; ++e) {
        const int ex = e % nel[0], ey = e / nel[0] % nel[1], ez = e / (nel[0] * nel[1]);
        int vs[8];
        for (int c = 0; c < 8; ++c)
            vs[c] = (ex + (c & 1)) % g.vd[0] + g.vd[0] * ((ey + (c >> 1 & 1)) % g.vd[1] + g.vd[1] * ((ez + (c >> 2)) % g.vd[2]));
        for (int c = 0; c < 8; ++c) {
            corner[vs[c]].push_back(e * 8 + c);
            for (int d = 0; d < 8; ++d) row[vs[c]].push_back(vs[d]);
        }
    }
    for (auto &r : row) {
        std::sort(r.begin(), r.end());
        r.erase(std::unique(r.begin(), r.end()), r.end());
    }
    const int32_t none = -7;
    std::vector<int32_t> vert((size_t)nt * g.verts, none), cn((size_t)nt * g.verts * 8, none);
    std::vector<int16_t> col((size_t)nt * g.rows * 32, none);
    int most[3] = {0, 0, 0};
    for (int t = 0; t < nt; ++t) {
        TileSets s;
        tile_sets(g, t, s);
        for (int i = 0; i < s.count[depth]; ++i) tile_vertex(g, s, t, i, d0inv.data(), vert.data(), cn.data(), col.data());
        for (int lane = 0; lane < 5; ++lane) tile_padding(g, s, t, lane, 5, vert.data(), cn.data(), col.data());
        // the list: the box, then ring by ring through the lattice's rows
        std::vector<int> want;
        std::map<int, int> at;
        const int p[3] = {t % g.nt[0], t / g.nt[0] % g.nt[1], t / (g.nt[0] * g.nt[1])};
        for (int z = p[2] * g.vd[2] / g.nt[2]; z < (p[2] + 1) * g.vd[2] / g.nt[2]; ++z)
            for (int y = p[1] * g.vd[1] / g.nt[1]; y < (p[1] + 1) * g.vd[1] / g.nt[1]; ++y)
                for (int x = p[0] * g.vd[0] / g.nt[0]; x < (p[0] + 1) * g.vd[0] / g.nt[0]; ++x)
                    want.push_back(x + g.vd[0] * (y + g.vd[1] * z));
        for (int v : want) at[v] = 1;
        std::vector<size_t> count{want.size()};
        for (int q = 1; q < kTileRings; ++q) {
            std::vector<int> next;
            if (q <= depth)
                for (int v : want)
                    for (int c : row[v])
                        if (!at.count(c)) {
                            at[c] = 1;
                            next.push_back(c);
                        }
            std::sort(next.begin(), next.end());
            want.insert(want.end(), next.begin(), next.end());
            count.push_back(want.size());
        }
        for (int q = 0; q < kTileRings; ++q) CHECK((int)count[q] == s.count[q], "tile %d ring %d", t, q);
        if (fails) return;
        most[0] = std::max<int>(most[0], count[0]);
        most[1] = std::max<int>(most[1], depth ? count[depth - 1] : 0);
        most[2] = std::max<int>(most[2], count[depth]);
        for (size_t h = 0; h < want.size(); ++h) at[want[h]] = (int)h;
        for (int h = 0; h < g.verts; ++h) {
            const bool listed = h < (int)want.size();
            CHECK(vert[(size_t)t * g.verts + h] == (listed ? want[h] : want[0]), "tile %d vertex %d", t, h);
            for (size_t q = 0; q < 8; ++q) {
                const int w = listed && q < corner[want[h]].size() ? corner[want[h]][q] : -1;
                CHECK(cn[((size_t)t * g.verts + h) * 8 + q] == w, "tile %d corner %d %zu", t, h, q);
            }
        }
        for (int h = 0; h < g.rows; ++h)
            for (size_t x = 0; x < 32; ++x) {
                int w = -1;
                if (h < (int)count[depth - 1] && d0inv[want[h]] > 0.0 && x < row[want[h]].size()) w = at[row[want[h]][x]];
                CHECK(col[((size_t)t * g.rows + h) * 32 + (x & 7) * 4 + (x >> 3)] == w, "tile %d row %d entry %zu", t, h, x);
            }
    }
    CHECK(most[0] == g.core && most[1] == g.rows && most[2] == g.verts, "strides %d %d %d", g.core, g.rows, g.verts);
}

int main()
{
    const int nels[][3] = {{1, 1, 1}, {2, 2, 2}, {1, 2, 3}, {3, 1, 5}, {2, 4, 7}, {6, 6, 6}, {5, 9, 8}, {16, 7, 9}, {17, 3, 1}, {10, 11, 23}};
    for (const auto &nel : nels)
        for (int bits = 0; bits < 8; ++bits)
            for (int edge : {3, 4, 8})
                for (int depth = 0; depth < kTileRings; ++depth)
                    for (bool holes : {false, true}) {
                        const int per[3] = {bits & 1, bits >> 1 & 1, bits >> 2};
                        check(nel, per, edge, depth, holes);
                        if (fails) {
                            std::printf("lattice %d %d %d periodic %d edge %d depth %d\n", nel[0], nel[1], nel[2], bits, edge, depth);
                            return 1;
                        }
                    }
    std::printf("OK\n");
    return 0;
}
