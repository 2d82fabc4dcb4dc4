// coarse_tiles.hpp -- the lists of the coarse term's tiles (coarse.hpp) from
// the vertex lattice alone: which vertices a tile lists, where, and its rows'
// columns.  Host and device share these functions, so the host can check the
// lists that the set-up kernel writes.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace sem {

constexpr int kTileRings = 4;  // a tile's box and the vertices 1 to 3 rows of A0 away

// Coordinates start .. start + len - 1 of an axis of n vertices, modulo n,
// in ascending order: 0 .. wrap - 1, then start ..
struct AxisSet {
    int start, wrap, len;
};

// lo .. hi - 1 and q more at either end, as far as the axis goes
__host__ __device__ inline AxisSet axis_set(int lo, int hi, int q, int n, int periodic)
{
    AxisSet s;
    if (!periodic || hi - lo + 2 * q >= n) {
        s.start = periodic || lo - q < 0 ? 0 : lo - q;
        s.len = (periodic || hi + q > n ? n : hi + q) - s.start;
        s.wrap = 0;
        return s;
    }
    s.len = hi - lo + 2 * q;
    s.start = (lo - q + n) % n;  // n > 2 q
    s.wrap = s.start + s.len > n ? s.start + s.len - n : 0;
    return s;
}
__host__ __device__ inline bool axis_has(const AxisSet &s, int c)
{
    return c < s.wrap || (c >= s.start && c - s.start < s.len - s.wrap);
}
// how many of the set lie below c
__host__ __device__ inline int axis_below(const AxisSet &s, int c)
{
    const int a = c < s.wrap ? c : s.wrap, b = c - s.start, m = s.len - s.wrap;
    return a + (b < 0 ? 0 : (b < m ? b : m));
}
__host__ __device__ inline int axis_at(const AxisSet &s, int i) { return i < s.wrap ? i : s.start + i - s.wrap; }

struct TileGeom {
    int vd[3], nel[3], periodic[3];  // vertices and elements per axis
    int nt[3];                       // tiles per axis
    int depth;                       // rings listed around a box, 0 .. kTileRings - 1
    int verts, rows, core;           // strides of the lists (tile_strides)
};

// one tile's box and rings, and the vertices up to each of them
struct TileSets {
    AxisSet ring[kTileRings][3];
    int count[kTileRings];
};
__host__ __device__ inline void tile_sets(const TileGeom &g, int64_t t, TileSets &s)
{
    const int64_t at[3] = {t % g.nt[0], (t / g.nt[0]) % g.nt[1], t / ((int64_t)g.nt[0] * g.nt[1])};
    for (int q = 0; q < kTileRings; ++q) {
        s.count[q] = 1;
        for (int a = 0; a < 3; ++a) {
            const int lo = (int)(at[a] * g.vd[a] / g.nt[a]), hi = (int)((at[a] + 1) * g.vd[a] / g.nt[a]);
            s.ring[q][a] = axis_set(lo, hi, q < g.depth ? q : g.depth, g.vd[a], g.periodic[a]);
            s.count[q] *= s.ring[q][a].len;
        }
    }
}

// the strides: the most any tile lists (a tile's counts are products over the
// axes, so they are those of the tile that is longest along each)
inline void tile_strides(TileGeom &g)
{
    int most[kTileRings] = {1, 1, 1, 1};
    for (int q = 0; q < kTileRings; ++q)
        for (int a = 0; a < 3; ++a) {
            int len = 0;
            for (int64_t i = 0; i < g.nt[a]; ++i) {
                const int l = axis_set((int)(i * g.vd[a] / g.nt[a]), (int)((i + 1) * g.vd[a] / g.nt[a]),
                                       q < g.depth ? q : g.depth, g.vd[a], g.periodic[a]).len;
                len = l > len ? l : len;
            }
            most[q] *= len;
        }
    g.core = most[0];
    g.rows = g.depth > 0 ? most[g.depth - 1] : 0;
    g.verts = most[g.depth];
}

// place of a listed vertex in its tile's list: the box first, then ring by
// ring, each by ascending vertex
__host__ __device__ inline int tile_place(const TileSets &s, int x, int y, int z, int &ring)
{
    int q = 0;
    while (q < kTileRings - 1 &&
           !(axis_has(s.ring[q][0], x) && axis_has(s.ring[q][1], y) && axis_has(s.ring[q][2], z)))
        ++q;
    ring = q;
    const AxisSet *r = s.ring[q];
    const int place = axis_below(r[0], x) + r[0].len * (axis_below(r[1], y) + r[1].len * axis_below(r[2], z));
    if (q == 0) return place;
    // less those of the smaller rings before it
    const AxisSet *p = s.ring[q - 1];
    int before = axis_below(p[2], z) * p[1].len * p[0].len;
    if (axis_has(p[2], z)) {
        before += axis_below(p[1], y) * p[0].len;
        if (axis_has(p[1], y)) before += axis_below(p[0], x);
    }
    return s.count[q - 1] + place - before;
}

// The list entries of the i-th vertex (ascending) of tile t's largest ring:
// vert, corner and, where a launch takes its row, col, at the strides of
// CoarseTiles.  d0inv: 0 where a vertex's row is empty.
__host__ __device__ inline void tile_vertex(const TileGeom &g, const TileSets &s, int64_t t, int i,
                                            const double *d0inv, int32_t *vert, int32_t *corner, int16_t *col)
{
    const AxisSet *all = s.ring[g.depth];
    const int c[3] = {axis_at(all[0], i % all[0].len), axis_at(all[1], i / all[0].len % all[1].len),
                      axis_at(all[2], i / (all[0].len * all[1].len))};
    const int v = c[0] + g.vd[0] * (c[1] + g.vd[1] * c[2]);
    int ring;
    const int h = tile_place(s, c[0], c[1], c[2], ring);
    vert[t * g.verts + h] = v;
    // its element corners e*8 + corner, ascending
    int32_t *cn = corner + (t * g.verts + h) * 8;
    int n = 0;
    for (int b = 0; b < 8; ++b) {
        int e[3];
        bool there = true;
        for (int a = 0; a < 3; ++a) {
            e[a] = c[a] - ((b >> a) & 1);
            if (e[a] < 0 && g.periodic[a]) e[a] += g.nel[a];
            there = there && e[a] >= 0 && e[a] < g.nel[a];
        }
        if (!there) continue;
        const int32_t entry = (e[0] + g.nel[0] * (e[1] + g.nel[1] * e[2])) * 8 + b;
        int k = n++;
        for (; k > 0 && cn[k - 1] > entry; --k) cn[k] = cn[k - 1];
        cn[k] = entry;
    }
    for (; n < 8; ++n) cn[n] = -1;
    if (ring >= g.depth) return;
    // the row's columns, ascending: entry x at lane x mod 8, x / 8
    int16_t *cl = col + (t * g.rows + h) * 32;
    for (int x = 0; x < 32; ++x) cl[x] = -1;
    if (!(d0inv[v] > 0.0)) return;
    const AxisSet nx = axis_set(c[0], c[0] + 1, 1, g.vd[0], g.periodic[0]),
                  ny = axis_set(c[1], c[1] + 1, 1, g.vd[1], g.periodic[1]),
                  nz = axis_set(c[2], c[2] + 1, 1, g.vd[2], g.periodic[2]);
    int x = 0;
    for (int kz = 0; kz < nz.len; ++kz)
        for (int ky = 0; ky < ny.len; ++ky)
            for (int kx = 0; kx < nx.len; ++kx, ++x) {
                int unused;
                cl[(x & 7) * 4 + (x >> 3)] =
                    (int16_t)tile_place(s, axis_at(nx, kx), axis_at(ny, ky), axis_at(nz, kz), unused);
            }
}

// entries of tile t's lists beyond what it lists
__host__ __device__ inline void tile_padding(const TileGeom &g, const TileSets &s, int64_t t, int lane, int lanes,
                                             int32_t *vert, int32_t *corner, int16_t *col)
{
    const AxisSet *b = s.ring[0];
    const int first = axis_at(b[0], 0) + g.vd[0] * (axis_at(b[1], 0) + g.vd[1] * axis_at(b[2], 0));
    for (int h = s.count[g.depth] + lane; h < g.verts; h += lanes) {
        vert[t * g.verts + h] = first;
        for (int q = 0; q < 8; ++q) corner[(t * g.verts + h) * 8 + q] = -1;
    }
    for (int h = (g.depth > 0 ? s.count[g.depth - 1] : 0) + lane; h < g.rows; h += lanes)
        for (int x = 0; x < 32; ++x) col[(t * g.rows + h) * 32 + x] = -1;
}

}  // namespace sem
