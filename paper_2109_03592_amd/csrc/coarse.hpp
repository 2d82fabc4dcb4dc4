// coarse.hpp -- the coarse term of Eq. 6 (coarse.hip): vertex space, the
// assembled coarse operator and its Chebyshev solve, on the device.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <vector>

#include "sem_internal.hpp"

namespace sem {

// Items [lo, hi) of E of the workgroup's XCD (workgroups go to the 8 XCDs round
// robin) and its place among that XCD's workgroups: each XCD walks one
// contiguous range, so that neighbours' values are met in its own L2.
struct XcdRange {
    int64_t lo, hi, first, step;
};
__device__ inline XcdRange xcd_range(int64_t E)
{
    const int64_t nb = gridDim.x, groups = nb < 8 ? nb : 8;
    const int64_t g = blockIdx.x % groups, kb = blockIdx.x / groups;
    // as many workgroups as an XCD has, so much of the range: with one
    // workgroup an item, none takes two
    const int64_t per = nb / groups, rem = nb % groups, before = g * per + (g < rem ? g : rem);
    XcdRange x;
    x.step = per + (g < rem ? 1 : 0);
    x.lo = E * before / nb;
    x.hi = E * (before + x.step) / nb;
    x.first = x.lo + kb;
    return x;
}

// P z0 at one node: the trilinear combination of the element's corner values
// (ev: its eight vertices, qw: the 1-D hat weights)
__device__ inline double hat_value(const int32_t *__restrict__ ev, const double *__restrict__ z0,
                                   const double *__restrict__ qw, int P, int i, int j, int k)
{
    double s = 0.0;
#pragma unroll
    for (int c = 0; c < 8; ++c) s += qw[(c & 1) * P + i] * qw[((c >> 1) & 1) * P + j] * qw[(c >> 2) * P + k] * z0[ev[c]];
    return s;
}

constexpr int kMaxCoarseDotBlocks = 1024;  // partial pairs of the coarse dot, at most

// The vertex lattice in boxes ("tiles") of up to kTileEdge^3 vertices, each
// with the vertices up to kTileSteps rows of A0 away: one workgroup takes the
// tile through kTileSteps products with A0 on its own, working redundantly on
// the vertices around its box instead of waiting for its neighbours.
constexpr int kTileEdge = 8, kTileSteps = 3;
constexpr int kTileCore = kTileEdge * kTileEdge * kTileEdge;
constexpr int kTileRows = (kTileEdge + 2 * (kTileSteps - 1)) * (kTileEdge + 2 * (kTileSteps - 1)) *
                          (kTileEdge + 2 * (kTileSteps - 1));
constexpr int kTileVerts = (kTileEdge + 2 * kTileSteps) * (kTileEdge + 2 * kTileSteps) * (kTileEdge + 2 * kTileSteps);
constexpr int kTileThreads = 1024;
static_assert(kTileSteps == 3, "a tile's four levels are one 16-byte load");
constexpr size_t kTileLds =
    sizeof(double) * 2 * (kTileVerts + kTileRows + kTileCore) + sizeof(int32_t) * kTileRows;
// Lists of a tile, each tile's at a fixed stride, so that nothing waits for an
// offset to arrive.  A tile lists its box first, then ring by ring.
struct CoarseTiles {
    int n = 0;                          // tiles
    int verts = 0, rows = 0, core = 0;  // strides: listed vertices, those whose rows a launch takes, the box
    const int32_t *level = nullptr;     // [n][4] listed vertices within 0 .. kTileSteps rows of the box
    const int32_t *vert = nullptr;      // [n][verts] the vertices (the padding repeats the first)
    const int32_t *corner = nullptr;    // [n][verts][8] the vertex's element corners e*8 + c, ascending, then -1
    const int16_t *col = nullptr;       // [n][rows][8][4] the row's columns as positions in the tile's list
};

// What the Chebyshev kernels of one coarse term work on (its work vectors are
// the mesh's own or a batched slot's)
struct CoarseChain {
    int k;                                  // steps
    double inv_theta;
    const double *coef, *a_val, *d0inv;     // coef: [k] c1, [k] c2
    const double *partial8;
    double *z0, *res[2], *d[2];             // res, d: of a chain of several launches
    CoarseTiles tiles;
};
// launches of a chain: its k - 1 products, kTileSteps each
__host__ __device__ inline int coarse_launches(int k) { return k <= 2 ? 1 : (k - 2) / kTileSteps + 1; }

struct CoarseSpace {
    int k = 0;               // Chebyshev steps
    double frac = 0.0;       // a = frac * b
    double a = 0.0, b = 0.0; // Chebyshev interval of D0^-1 A0
    double inv_theta = 0.0;
    int64_t nvert = 0;       // element vertices (periodic images merged)
    int64_t n_coarse = 0;    // vertices with a non-zero masked hat function
    int64_t nnz = 0;
    int dot_blocks = 0;      // workgroups of the coarse dot (partial pairs)
    // device
    int32_t *evert = nullptr;   // [E][8] vertex of each element corner
    double *qw = nullptr;       // [2][N+1] 1-D hat weights at the GLL nodes
    // rows of A0, [nvert][8][4]: entry x of a row (at most 27, by ascending
    // column) at lane x mod 8, x / 8; the columns are in the tiles
    double *a_val = nullptr;
    CoarseTiles tiles;
    double *coef = nullptr;     // [2][k] c1, c2
    double *d0inv = nullptr;    // [nvert] 1/diag(A0), 0 where the vertex is not a coarse unknown
    double *partial8 = nullptr; // [E][8] element restriction sums
    double *z0 = nullptr, *res[2] = {nullptr, nullptr}, *d[2] = {nullptr, nullptr};
    std::vector<void *> allocations;
};

// Work vectors of one batched slot's coarse term, carved from one buffer of
// coarse_work_doubles values in this order: element restriction sums [E][8],
// z0, and for a chain of several launches res and d twice [nvert each].  (The mesh's own, for its
// single-mesh solves, are in CoarseSpace.)
struct CoarseWork {
    double *partial8, *z0, *res[2], *d[2];
};
CoarseChain coarse_chain(const CoarseSpace *C, const CoarseWork &W);
int64_t coarse_work_doubles(const CoarseSpace *C, int64_t E);
CoarseWork coarse_work_carve(const CoarseSpace *C, int64_t E, double *base);

// Builds the coarse space of the mesh's current operator (synchronises s).
CoarseSpace *coarse_build(sem_mesh *m, int k, double frac, hipStream_t s);
void coarse_free(CoarseSpace *C);
// CG update (precision T) with the restriction fused in: r -= alpha w,
// partial pairs of <r,r>, <r, inv r> into `partial` (returns their count),
// element restriction sums of the new r.  Skips when st->done.
// with_rz = false: the second entry of each pair is 0 (another local
// preconditioner supplies <r, z>).
template <typename T>
int coarse_update(sem_mesh *m, T *r, const T *w, const T *inv, const PcgState *st, double *partial, bool with_rz,
                  hipStream_t s);
// element restriction sums of r (live nodes: inv > 0)
template <typename T>
void coarse_restrict(sem_mesh *m, const T *r, const T *inv, hipStream_t s);
// from the element sums: r0 = P^T r, z0 = C(A0) r0, and when dot_pairs is
// given the (0, r0.z0) pairs there (returns their count, C->dot_blocks);
// kernels skip when st->done.
int coarse_solve(sem_mesh *m, double *dot_pairs, const PcgState *st, hipStream_t s);
// z = inv r + masked P z0 (z0 from the last coarse_solve)
void coarse_jacobi_prolong(sem_mesh *m, const double *r, double *z, hipStream_t s);
// z = inv r
void launch_jacobi(int64_t n, const double *inv, const double *r, double *z, hipStream_t s);

}  // namespace sem
