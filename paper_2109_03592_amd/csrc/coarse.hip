// coarse.hip -- the coarse term of Eq. 6 on the GPU: a two-level
// preconditioner M^{-1} r = D^{-1} r + P C(A0) P^T r for FP64 CG.
//
//  * P: trilinear hat functions of the element vertices at the GLL nodes (in
//    each element's reference coordinates), zero at Dirichlet nodes.
//  * A0 = P^T A P, assembled on the host from per-element 8x8 blocks
//    P_e^T A_e P_e; each block column is the local operator applied to one
//    masked hat function, tested against the eight hats.
//  * C(A0): k steps of Chebyshev iteration for D0^-1 A0 z = D0^-1 r0 from 0
//    on [frac b, b], b the largest absolute row sum of D0^-1 A0 -- a fixed
//    polynomial, so M stays linear and symmetric positive definite.
//  * Restriction P^T r: per element, eight weighted sums over its nodes
//    (1/mult for unique-node sums), then per vertex the sum of its element
//    corners in a fixed order.  Prolongation: folded into the CG operator's
//    prologue (p = D^-1 r + P z0 + beta p), or added to a vector.
//  * The coarse part of <r, z> is r0 . z0, appended to the CG partials.
// Dirichlet nodes are the nodes whose inverse diagonal is 0.
#include <algorithm>
#include <cmath>
#include <type_traits>
#include <vector>

#include "batch.hpp"
#include "coarse.hpp"
#include "coarse_tiles.hpp"
#include "kernels.hpp"
#include "lattice.hpp"
#include "operator.hpp"

namespace sem {

// ---------------------------------------------------------------------------
// device kernels

// node q of an element: (i, j, k) and the eight hat weights
__device__ inline void hat_weights(const double *__restrict__ qw, int P, int q, double (&phi)[8])
{
    const int i = q % P, j = (q / P) % P, k = q / (P * P);
    const double ai[2] = {qw[i], qw[P + i]}, aj[2] = {qw[j], qw[P + j]}, ak[2] = {qw[k], qw[P + k]};
#pragma unroll
    for (int c = 0; c < 8; ++c) phi[c] = ai[c & 1] * aj[(c >> 1) & 1] * ak[(c >> 2) & 1];
}

// u = masked hat function of corner c on every element (element-local vector)
__global__ __launch_bounds__(256) void hat_kernel(int64_t E, int P, const double *__restrict__ qw, int c,
                                                  const double *__restrict__ inv, double *__restrict__ u)
{
    const int P3 = P * P * P;
    const int64_t n = E * P3;
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += (int64_t)gridDim.x * blockDim.x) {
        double phi[8];
        hat_weights(qw, P, (int)(q % P3), phi);
        u[q] = inv[q] > 0.0 ? phi[c] : 0.0;
    }
}

// Totals of eight values over the wavefront.  Each of the first three steps
// exchanges half of the values a lane still holds, so ten shuffles do the work
// of the 48 of eight full butterflies, with the same pairs added at each
// step (the same bits).  Returns the total of value lane >> 3.
__device__ inline double wave_sum8(const double (&s)[8])
{
    const int lane = threadIdx.x & 63;
    double a[4], b[2];
    const bool h5 = lane & 32, h4 = lane & 16, h3 = lane & 8;
#pragma unroll
    for (int q = 0; q < 4; ++q) a[q] = (h5 ? s[q + 4] : s[q]) + __shfl_xor(h5 ? s[q] : s[q + 4], 32, 64);
#pragma unroll
    for (int q = 0; q < 2; ++q) b[q] = (h4 ? a[q + 2] : a[q]) + __shfl_xor(h4 ? a[q] : a[q + 2], 16, 64);
    double v = (h3 ? b[1] : b[0]) + __shfl_xor(h3 ? b[0] : b[1], 8, 64);
    v += __shfl_xor(v, 4, 64);
    v += __shfl_xor(v, 2, 64);
    v += __shfl_xor(v, 1, 64);
    return v;
}

// E8[e][c'][c] = sum over element e's live nodes of phi_c' * w, w = A_e u_c
__global__ __launch_bounds__(256) void elem_coarse_kernel(int64_t E, int P, const double *__restrict__ w,
                                                          const double *__restrict__ qw,
                                                          const double *__restrict__ inv, int c,
                                                          double *__restrict__ E8)
{
    __shared__ double sqw[2 * (SEM_MAX_ORDER + 1)];
    if (threadIdx.x < 2 * P) sqw[threadIdx.x] = qw[threadIdx.x];
    __syncthreads();
    const int P3 = P * P * P, lane = threadIdx.x & 63;
    for (int64_t e = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); e < E; e += (int64_t)gridDim.x * 4) {
        double s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        for (int q = lane; q < P3; q += 64) {
            const double v = inv[e * P3 + q] > 0.0 ? w[e * P3 + q] : 0.0;
            double phi[8];
            hat_weights(sqw, P, q, phi);
#pragma unroll
            for (int h = 0; h < 8; ++h) s[h] += phi[h] * v;
        }
        const double v = wave_sum8(s);
        if ((lane & 7) == 0) E8[e * 64 + lane + c] = v;
    }
}

// Hat-function sums at compile-time order: node q = i + P j + P^2 k of an
// element adds v phi_c(q) to s[c], phi_c = a[cx][i] a[cy][j] a[cz][k]
// (c = cx + 2 cy + 4 cz, a[side][.] the 1-D weights in LDS).
template <int N>
__device__ inline void hat_add(const double *__restrict__ sqw, int q, double v, double (&s)[8])
{
    constexpr int P = N + 1, P2 = P * P;
    const int i = q % P, j = (q / P) % P, k = q / P2;
    const double ai0 = sqw[i], ai1 = sqw[P + i];
    const double aj0 = sqw[j], aj1 = sqw[P + j], ak0 = sqw[k], ak1 = sqw[P + k];
    const double t00 = aj0 * ak0 * v, t10 = aj1 * ak0 * v, t01 = aj0 * ak1 * v, t11 = aj1 * ak1 * v;
    s[0] += ai0 * t00; s[1] += ai1 * t00; s[2] += ai0 * t10; s[3] += ai1 * t10;
    s[4] += ai0 * t01; s[5] += ai1 * t01; s[6] += ai0 * t11; s[7] += ai1 * t11;
}

// partial8[e*8 + c] = sum over element e's live nodes of phi_c r / mult, by
// one wavefront (sqw: the hat weights in LDS)
template <typename T, int N>
__device__ inline void restrict_element(int64_t e, const T *__restrict__ r, const uint8_t *__restrict__ mult,
                                        const T *__restrict__ inv, const double *sqw, double *__restrict__ partial8)
{
    constexpr int P = N + 1, P3 = P * P * P;
    const int lane = threadIdx.x & 63;
    double s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    const int64_t base = e * P3;
#pragma unroll
    for (int q = lane; q < P3; q += 64) {
        const T iv = ld_stream(inv + base + q);
        const double v = iv > T(0) ? (double)ld_stream(r + base + q) * inv_mult(ld_stream(mult + base + q)) : 0.0;
        hat_add<N>(sqw, q, v, s);
    }
    const double out = wave_sum8(s);
    if ((lane & 7) == 0) partial8[e * 8 + (lane >> 3)] = out;
}

template <typename T, int N>
__global__ __launch_bounds__(256) void restrict_elem_kernel(int64_t E, const T *__restrict__ r,
                                                            const uint8_t *__restrict__ mult,
                                                            const T *__restrict__ inv,
                                                            const double *__restrict__ qw,
                                                            double *__restrict__ partial8)
{
    constexpr int P = N + 1;
    __shared__ double sqw[2 * P];
    if (threadIdx.x < 2 * P) sqw[threadIdx.x] = qw[threadIdx.x];
    __syncthreads();
    for (int64_t e = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); e < E; e += (int64_t)gridDim.x * 4)
        restrict_element<T, N>(e, r, mult, inv, sqw, partial8);
}

// CG update with the coarse restriction fused in: r -= alpha w, the partial
// pairs of <r,r> and <r, invdiag r> per workgroup (FP64 sums, the products
// as in the plain update; the second 0 unless with_rz), and the element
// restriction sums of the new r; one wavefront per element.
template <typename T, int N>
__global__ __launch_bounds__(256) void update_restrict_kernel(int64_t E, const PcgState *__restrict__ st,
                                                              T *__restrict__ r, const T *__restrict__ w,
                                                              const T *__restrict__ inv,
                                                              const uint8_t *__restrict__ mult,
                                                              const double *__restrict__ qw,
                                                              double *__restrict__ partial,
                                                              double *__restrict__ partial8, int with_rz)
{
    constexpr int P = N + 1, P3 = P * P * P;
    if (st->done) return;
    __shared__ double sqw[2 * P];
    if (threadIdx.x < 2 * P) sqw[threadIdx.x] = qw[threadIdx.x];
    __syncthreads();
    const T alpha = (T)st->alpha;
    const int lane = threadIdx.x & 63;
    double rr = 0.0, rz = 0.0;
    for (int64_t e = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); e < E; e += (int64_t)gridDim.x * 4) {
        double s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        const int64_t base = e * P3;
        if constexpr (sizeof(T) == 4 && P3 % 2 == 0) {
            // FP32, N odd: two adjacent nodes of one element row per lane
            // (paired 8-byte loads), in the same per-node arithmetic
            const float2 *r2 = reinterpret_cast<const float2 *>(r + base);
            const float2 *w2 = reinterpret_cast<const float2 *>(w + base);
            const float2 *i2 = reinterpret_cast<const float2 *>(inv + base);
            const uint16_t *m2 = reinterpret_cast<const uint16_t *>(mult + base);
#pragma unroll
            for (int h = lane; h < P3 / 2; h += 64) {
                float2 rv = ld_stream(r2 + h);
                const float2 wv = ld_stream(w2 + h), iv = ld_stream(i2 + h);
                const uint16_t mm = ld_stream(m2 + h);
                rv.x = rv.x - (float)alpha * wv.x;
                rv.y = rv.y - (float)alpha * wv.y;
                st_stream(rv, reinterpret_cast<float2 *>(r + base) + h);
                const double ima = inv_mult((uint8_t)(mm & 0xff)), imb = inv_mult((uint8_t)(mm >> 8));
                const double ra = (double)rv.x, rb = (double)rv.y;
                rr += ra * ra * ima;
                rr += rb * rb * imb;
                if (with_rz) {
                    rz += ra * (double)(iv.x * rv.x) * ima;
                    rz += rb * (double)(iv.y * rv.y) * imb;
                }
                hat_add<N>(sqw, 2 * h, iv.x > 0.0f ? ra * ima : 0.0, s);
                hat_add<N>(sqw, 2 * h + 1, iv.y > 0.0f ? rb * imb : 0.0, s);
            }
        } else {
#pragma unroll
            for (int q = lane; q < P3; q += 64) {
                const int64_t o = base + q;
                const T rv = ld_stream(r + o) - alpha * ld_stream(w + o);
                st_stream(rv, r + o);
                const T iv = ld_stream(inv + o);
                const double im = inv_mult(ld_stream(mult + o));
                const double rd = (double)rv;
                rr += rd * rd * im;
                if (with_rz) rz += rd * (double)(iv * rv) * im;
                hat_add<N>(sqw, q, iv > T(0) ? rd * im : 0.0, s);
            }
        }
        const double out = wave_sum8(s);
        if ((lane & 7) == 0) partial8[e * 8 + (lane >> 3)] = out;
    }
    double v[2] = {rr, rz};
    block_reduce_store<2>(v, partial, 2);
}

// One launch of the Chebyshev solve A0 z = r0, for one tile: up to kTileSteps
// of the steps z += d; res -= A0 d; d = c1 d + c2 D0^-1 res.  The last step
// needs its z only, so the step before it adds that d too and k steps are
// k - 1 products.  The first launch starts from the element sums: r0[v] the sum
// of v's element corners (ascending), z = 0, res = r0, d = D0^-1 r0 / theta.
// Later launches read res and d around the box from buffers their own results
// do not go to.  A row's entries are taken by eight lanes and summed by a
// fixed pattern.  Returns this lane's part of sum r0 z at the end.
//
// On a mesh of a few thousand elements each step as a launch of its own costs
// the 4.5 us of any small kernel and does next to nothing.  A tile's launch is
// bound by its lookups (listed vertices' corners, rows around the box), which
// is why it repeats work on small boxes rather than less on few large ones.
// 16x16x16 pipe, 4 steps (216 tiles): 24 us in five launches -> 12 us in one;
// 24x24x48, 192 tiles of a larger edge: 30 -> 23 us; the 12 boxes of a batch
// (up to 1024 elements): 19 -> 7 us.  Rows kept in registers from step to step
// were no faster, and shuffles through the LDS instead of sum8 0.5 us slower.
__device__ inline double coarse_tile(const CoarseChain &C, int t, int launch, double *sm)
{
    const CoarseTiles &T = C.tiles;
    double *da = sm, *db = da + kTileVerts, *res = db + kTileVerts, *dinv = res + kTileRows, *z = dinv + kTileRows;
    double *r0 = z + kTileCore;
    int32_t *verts = reinterpret_cast<int32_t *>(r0 + kTileCore);
    const int j0 = launch * kTileSteps;
    const int left = C.k - 1 - j0, steps = left < kTileSteps ? left : kTileSteps;
    const bool first = launch == 0, last = left <= kTileSteps;
    const int tid = threadIdx.x, sub = tid & 7;
    const int64_t vbase = (int64_t)t * T.verts, rbase = (int64_t)t * T.rows;
    const int4 lv = reinterpret_cast<const int4 *>(T.level)[t];
    const int level[kTileSteps + 1] = {lv.x, lv.y, lv.z, lv.w};
    double c1[kTileSteps], c2[kTileSteps];
#pragma unroll
    for (int q = 0; q < kTileSteps; ++q) {
        c1[q] = q < steps ? C.coef[j0 + q] : 0.0;
        c2[q] = q < steps ? C.coef[C.k + j0 + q] : 0.0;
    }
    const double *din = C.d[launch & 1], *rin = C.res[launch & 1];
    for (int h = tid; h < T.verts; h += kTileThreads) {
        const int v = T.vert[vbase + h];
        const double di = C.d0inv[v];
        double d, r = 0.0, sum = 0.0;
        if (first || (last && h < T.core)) {
            int32_t idx[8];
            double y[8];
            const int4 *cn = reinterpret_cast<const int4 *>(T.corner + (vbase + h) * 8);
            const int4 ca = cn[0], cb = cn[1];
            idx[0] = ca.x; idx[1] = ca.y; idx[2] = ca.z; idx[3] = ca.w;
            idx[4] = cb.x; idx[5] = cb.y; idx[6] = cb.z; idx[7] = cb.w;
#pragma unroll
            for (int c = 0; c < 8; ++c) y[c] = idx[c] >= 0 ? C.partial8[idx[c]] : 0.0;
#pragma unroll
            for (int c = 0; c < 8; ++c)
                if (idx[c] >= 0) sum += y[c];
        }
        if (first) {
            r = sum;
            d = sum * di * C.inv_theta;
        } else {
            d = din[v];
            if (h < T.rows) r = rin[v];
        }
        da[h] = d;
        if (h < T.rows) {
            res[h] = r;
            dinv[h] = di;
            verts[h] = v;
        }
        if (h < T.core) {
            z[h] = first ? 0.0 : C.z0[v];
            r0[h] = sum;
        }
    }
    __syncthreads();
    const int nc = level[0];
    for (int q = 0; q < steps; ++q) {
        const bool end = last && q == steps - 1;
        const int left_rows = steps - 1 - q;
        const int n = left_rows == 2 ? level[2] : (left_rows == 1 ? level[1] : level[0]);
        const double e1 = q == 0 ? c1[0] : (q == 1 ? c1[1] : c1[2]), e2 = q == 0 ? c2[0] : (q == 1 ? c2[1] : c2[2]);
        // wave-uniform trip count: the sums run on full wavefronts
#pragma unroll 2
        for (int h0 = (tid >> 6) * 8; h0 < n; h0 += kTileThreads / 8) {
            const int h = h0 + ((tid & 63) >> 3);
            double s = 0.0;
            if (h < n) {
                const double2 *val = reinterpret_cast<const double2 *>(C.a_val + ((int64_t)verts[h] * 8 + sub) * 4);
                const double2 va = val[0], vb = val[1];
                const short4 c = reinterpret_cast<const short4 *>(T.col)[(rbase + h) * 8 + sub];
                if (c.x >= 0) s += va.x * da[c.x];
                if (c.y >= 0) s += va.y * da[c.y];
                if (c.z >= 0) s += vb.x * da[c.z];
                if (c.w >= 0) s += vb.y * da[c.w];
            }
            s = sum8(s);
            if (h < n && sub == 0) {
                const double dv = da[h], rv = res[h] - s, dn = e1 * dv + e2 * rv * dinv[h];
                res[h] = rv;
                db[h] = dn;
                if (h < nc) {
                    const double zv = z[h] + dv;
                    z[h] = end ? zv + dn : zv;
                }
            }
        }
        __syncthreads();
        double *x = da;
        da = db;
        db = x;
    }
    double dot = 0.0;
    for (int h = tid; h < nc; h += kTileThreads) {
        const int v = T.vert[vbase + h];
        const double zv = steps == 0 ? z[h] + da[h] : z[h];
        C.z0[v] = zv;
        if (last) {
            dot += r0[h] * zv;
        } else {
            C.d[(launch + 1) & 1][v] = da[h];
            C.res[(launch + 1) & 1][v] = res[h];
        }
    }
    __syncthreads();  // the next tile rewrites the LDS
    return dot;
}

// Chebyshev launch `launch` of a mesh; in the last one the (0, sum r0 z) pair
// of each workgroup goes into `partial` when given.
__global__ __launch_bounds__(kTileThreads) void coarse_tile_kernel(CoarseChain C, int launch,
                                                                   double *__restrict__ partial,
                                                                   const PcgState *__restrict__ st)
{
    if (st && st->done) return;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    double p[2] = {0.0, 0.0};
    // the workgroups of one XCD take neighbouring tiles, whose rows overlap
    const XcdRange X = xcd_range(C.tiles.n);
    for (int64_t t = X.first; t < X.hi; t += X.step)
        p[1] += coarse_tile(C, (int)t, launch, reinterpret_cast<double *>(smem_raw));
    if (partial) block_reduce_store<2>(p, partial, 2);
}

// z = masked P z0, or with r z = inv r + masked P z0 (the whole
// preconditioner with the Jacobi local part), rounded to the precision of z;
// masked nodes (inv 0) get 0.  One lane per (i, j) column of an element, the
// workgroup kPrElems elements: the eight corner values and the bilinear forms
// of the column are taken once, a node costs two multiply-adds, and the pass
// is bound by its 16 (24 with r) bytes per node.
template <int N>
constexpr int kPrElems = 256 / ((N + 1) * (N + 1)) > 0 ? 256 / ((N + 1) * (N + 1)) : 1;

template <int N, bool JACOBI, typename TZ>
__device__ inline void prolong_column(int64_t e, int ij, const int32_t *__restrict__ evert,
                                      const double *__restrict__ z0, const double *__restrict__ qw,
                                      const double *__restrict__ inv, const double *__restrict__ r,
                                      TZ *__restrict__ z)
{
    constexpr int P = N + 1, P2 = P * P, P3 = P2 * P;
    const int i = ij % P, j = ij / P;
    const int64_t o = e * P3 + ij;
    double iv[P], rv[P];
#pragma unroll
    for (int k = 0; k < P; ++k) {
        iv[k] = ld_stream(inv + o + k * P2);
        if (JACOBI) rv[k] = ld_stream(r + o + k * P2);
    }
    double zc[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) zc[c] = z0[evert[e * 8 + c]];
    const double ai0 = qw[i], ai1 = qw[P + i], aj0 = qw[j], aj1 = qw[P + j];
    const double cs0 = aj0 * (ai0 * zc[0] + ai1 * zc[1]) + aj1 * (ai0 * zc[2] + ai1 * zc[3]);
    const double cs1 = aj0 * (ai0 * zc[4] + ai1 * zc[5]) + aj1 * (ai0 * zc[6] + ai1 * zc[7]);
#pragma unroll
    for (int k = 0; k < P; ++k) {
        double v = iv[k] > 0.0 ? qw[k] * cs0 + qw[P + k] * cs1 : 0.0;
        if (JACOBI) v += iv[k] * rv[k];
        st_stream((TZ)v, z + o + k * P2);
    }
}

// z = inv r + masked P z0
template <int N>
__global__ __launch_bounds__(256) void prolong_kernel(int64_t E, const int32_t *__restrict__ evert,
                                                      const double *__restrict__ z0, const double *__restrict__ qw,
                                                      const double *__restrict__ inv, const double *__restrict__ r,
                                                      double *__restrict__ z)
{
    constexpr int P2 = (N + 1) * (N + 1);
    const int el = threadIdx.x / P2, ij = threadIdx.x - el * P2;
    const int64_t e = (int64_t)blockIdx.x * kPrElems<N> + el;
    if (el >= kPrElems<N> || e >= E) return;
    prolong_column<N, true, double>(e, ij, evert, z0, qw, inv, r, z);
}

__global__ void jacobi_kernel(int64_t n, const double *__restrict__ inv, const double *__restrict__ r,
                              double *__restrict__ z)
{
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += (int64_t)gridDim.x * blockDim.x)
        z[q] = inv[q] * r[q];
}

// ---------------------------------------------------------------------------
// host side

static int cgrid(int64_t n, int cap) { return (int)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, cap)); }

template <typename X>
static X *cmalloc(CoarseSpace *C, size_t count)
{
    void *p = nullptr;
    SEM_HIP(hipMalloc(&p, std::max<size_t>(count * sizeof(X), 16)));
    C->allocations.push_back(p);
    return static_cast<X *>(p);
}

void coarse_free(CoarseSpace *C)
{
    if (!C) return;
    for (void *p : C->allocations) (void)hipFree(p);
    delete C;
}

// The lists of the tiles, one workgroup each.  They follow from the lattice, so
// nothing is searched or sent: on the 48x48x96 pipe (588 tiles) this launch and
// its allocations take 0.2 ms where a walk of the host over the rows of A0 and
// the copy of its 110 MB of lists took 50.
__global__ __launch_bounds__(256) void tile_lists_kernel(TileGeom g, const double *__restrict__ d0inv,
                                                         int32_t *__restrict__ level, int32_t *__restrict__ vert,
                                                         int32_t *__restrict__ corner, int16_t *__restrict__ col)
{
    __shared__ TileSets s;
    const int64_t t = blockIdx.x;
    const int tid = threadIdx.x;
    if (tid == 0) tile_sets(g, t, s);
    __syncthreads();
    if (tid < kTileRings) level[t * kTileRings + tid] = s.count[tid];
    for (int i = tid; i < s.count[g.depth]; i += 256) tile_vertex(g, s, t, i, d0inv, vert, corner, col);
    tile_padding(g, s, t, tid, 256, vert, corner, col);
}

// The tiles of the vertex lattice (extents vd).  The box edge is the smallest
// from 3 on that gives at most a workgroup per compute unit: a smaller box
// lists fewer vertices, which is what a workgroup's time goes by, a larger one
// repeats less (3: 27 listed vertices per vertex, 8: 5.4).  Preconditioner of
// 16^3 elements with edge 2, 3 and 4: 31.0, 31.0 and 32.8 us.
static void build_tiles(CoarseSpace *C, const HostMesh &h, const int vd[3], hipStream_t s)
{
    static_assert(kTileRings == kTileSteps + 1, "a ring for each product of a launch");
    TileGeom g{};
    for (int a = 0; a < 3; ++a) {
        g.vd[a] = vd[a];
        g.nel[a] = h.nel[a];
        g.periodic[a] = h.periodic[a] ? 1 : 0;
    }
    for (int edge = 3; edge <= kTileEdge; ++edge) {
        for (int a = 0; a < 3; ++a) g.nt[a] = (vd[a] + edge - 1) / edge;
        if ((int64_t)g.nt[0] * g.nt[1] * g.nt[2] <= 256) break;
    }
    const int64_t n = (int64_t)g.nt[0] * g.nt[1] * g.nt[2];
    g.depth = std::min(kTileSteps, C->k - 1);
    tile_strides(g);
    if (g.core > kTileCore || g.rows > kTileRows || g.verts > kTileVerts)
        fail(SEM_EINVAL, "sem_set_coarse: a tile exceeds its bounds");
    CoarseTiles &T = C->tiles;
    T.n = (int)n;
    T.verts = g.verts;
    T.rows = g.rows;
    T.core = g.core;
    int32_t *level = cmalloc<int32_t>(C, (size_t)n * kTileRings), *vert = cmalloc<int32_t>(C, (size_t)n * T.verts),
            *corner = cmalloc<int32_t>(C, (size_t)n * T.verts * 8);
    int16_t *col = cmalloc<int16_t>(C, (size_t)n * T.rows * 32);
    hipLaunchKernelGGL(tile_lists_kernel, dim3((unsigned)n), dim3(256), 0, s, g, C->d0inv, level, vert, corner, col);
    SEM_HIP(hipGetLastError());
    T.level = level;
    T.vert = vert;
    T.corner = corner;
    T.col = col;
}

CoarseSpace *coarse_build(sem_mesh *m, int k, double frac, hipStream_t s)
{
    const HostMesh &h = m->h;
    const int N = h.N, P = N + 1;
    const int64_t E = h.E, P3 = (int64_t)P * P * P, nL = h.nL;
    if (k < 1 || k > 1000) fail(SEM_EINVAL, "sem_set_coarse: chebyshev_steps must be 1..1000");
    if (!(frac > 0.0 && frac < 1.0)) fail(SEM_EINVAL, "sem_set_coarse: fraction must be in (0, 1)");
    if (E * 8 >= INT32_MAX) fail(SEM_EUNSUPPORTED, "sem_set_coarse: too many elements");
    CoarseSpace *C = new CoarseSpace();
    try {
        C->k = k;
        C->frac = frac;
        const int nx = h.nel[0], ny = h.nel[1], nz = h.nel[2];
        const int vd[3] = {nx + 1 - h.periodic[0], ny + 1 - h.periodic[1], nz + 1 - h.periodic[2]};
        C->nvert = (int64_t)vd[0] * vd[1] * vd[2];
        // element corners -> vertices
        std::vector<int32_t> evert((size_t)E * 8);
        for (int64_t e = 0; e < E; ++e) {
            const int64_t ex = e % nx, ey = (e / nx) % ny, ez = e / ((int64_t)nx * ny);
            for (int c = 0; c < 8; ++c) {
                const int64_t a = (ex + (c & 1)) % vd[0], b = (ey + ((c >> 1) & 1)) % vd[1],
                              cc = (ez + ((c >> 2) & 1)) % vd[2];
                evert[e * 8 + c] = (int32_t)(a + vd[0] * (b + (int64_t)vd[1] * cc));
            }
        }
        // vertex -> (element, corner) entries, ascending
        std::vector<int32_t> v_off((size_t)C->nvert + 1, 0), v_idx((size_t)E * 8);
        for (int64_t q = 0; q < E * 8; ++q) v_off[evert[q] + 1]++;
        for (int64_t v = 0; v < C->nvert; ++v) v_off[v + 1] += v_off[v];
        {
            std::vector<int32_t> cur(v_off.begin(), v_off.end() - 1);
            for (int64_t q = 0; q < E * 8; ++q) v_idx[cur[evert[q]]++] = (int32_t)q;
        }
        // 1-D hat weights at the GLL nodes
        std::vector<double> qw(2 * P);
        for (int i = 0; i < P; ++i) {
            qw[i] = 0.5 * (1.0 - h.xi[i]);
            qw[P + i] = 0.5 * (1.0 + h.xi[i]);
        }
        C->evert = cmalloc<int32_t>(C, evert.size());
        C->qw = cmalloc<double>(C, qw.size());
        SEM_HIP(hipMemcpyAsync(C->evert, evert.data(), sizeof(int32_t) * evert.size(), hipMemcpyHostToDevice, s));
        SEM_HIP(hipMemcpyAsync(C->qw, qw.data(), sizeof(double) * qw.size(), hipMemcpyHostToDevice, s));
        // element blocks P_e^T A_e P_e with the mesh's current operator
        std::vector<double> E8((size_t)E * 64);
        {
            double *u = nullptr, *w = nullptr, *dE8 = nullptr;
            SEM_HIP(hipMalloc(&u, sizeof(double) * nL));
            SEM_HIP(hipMalloc(&w, sizeof(double) * nL));
            SEM_HIP(hipMalloc(&dE8, sizeof(double) * E * 64));
            try {
                for (int c = 0; c < 8; ++c) {
                    hipLaunchKernelGGL(hat_kernel, dim3(vec_blocks(nL)), dim3(256), 0, s, E, P, C->qw, c, m->inv64, u);
                    SEM_HIP(hipGetLastError());
                    const sem_status st = sem_ax(m, SEM_FP64, u, w, nullptr, s);
                    if (st != SEM_OK) fail(st, "sem_set_coarse: operator apply failed");
                    hipLaunchKernelGGL(elem_coarse_kernel, dim3(cgrid(E * 64, 8192)), dim3(256), 0, s, E, P, w,
                                       C->qw, m->inv64, c, dE8);
                    SEM_HIP(hipGetLastError());
                }
                SEM_HIP(hipMemcpyAsync(E8.data(), dE8, sizeof(double) * E * 64, hipMemcpyDeviceToHost, s));
                SEM_HIP(hipStreamSynchronize(s));
            } catch (...) {
                hipFree(u);
                hipFree(w);
                hipFree(dE8);
                throw;
            }
            SEM_HIP(hipFree(u));
            SEM_HIP(hipFree(w));
            SEM_HIP(hipFree(dE8));
        }
        // A0 rows: sum of the element blocks of the vertex's corners, ascending,
        // at the places of the row's columns (ascending; the lattice gives them)
        std::vector<double> rows((size_t)C->nvert * 32, 0.0), diag((size_t)C->nvert, 0.0);
        auto entry = [&](int64_t v, int x) -> double & { return rows[(size_t)v * 32 + (x & 7) * 4 + (x >> 3)]; };
        auto columns = [&](int64_t v, AxisSet (&set)[3], int (&at)[3]) {
            at[0] = (int)(v % vd[0]);
            at[1] = (int)(v / vd[0] % vd[1]);
            at[2] = (int)(v / ((int64_t)vd[0] * vd[1]));
            for (int a = 0; a < 3; ++a) set[a] = axis_set(at[a], at[a] + 1, 1, vd[a], h.periodic[a]);
        };
        C->n_coarse = C->nnz = 0;
        for (int64_t v = 0; v < C->nvert; ++v) {
            AxisSet set[3];
            int at[3], place[3][3];  // place of the neighbour one down, of the vertex itself, of the one up
            columns(v, set, at);
            for (int a = 0; a < 3; ++a)
                for (int d = 0; d < 3; ++d) place[a][d] = axis_below(set[a], (at[a] + d - 1 + vd[a]) % vd[a]);
            const int len = set[0].len * set[1].len * set[2].len;
            double row[27] = {0.0};
            for (int32_t q = v_off[v]; q < v_off[v + 1]; ++q) {
                const int cr = v_idx[q] % 8;
                const double *block = &E8[(size_t)v_idx[q] * 8];
                for (int c = 0; c < 8; ++c) {
                    const int x = place[0][(c & 1) - (cr & 1) + 1],
                              y = place[1][((c >> 1) & 1) - ((cr >> 1) & 1) + 1], z = place[2][(c >> 2) - (cr >> 2) + 1];
                    row[x + set[0].len * (y + set[1].len * z)] += block[c];
                }
            }
            diag[v] = row[place[0][1] + set[0].len * (place[1][1] + set[1].len * place[2][1])];
            if (!(diag[v] > 0.0)) continue;  // not a coarse unknown: empty row
            for (int x = 0; x < len; ++x) entry(v, x) = row[x];
            C->n_coarse++;
            C->nnz += len;
        }
        // vertices whose masked hat is zero are not coarse unknowns: drop their columns
        std::vector<double> d0inv((size_t)C->nvert, 0.0);
        for (int64_t v = 0; v < C->nvert; ++v)
            if (diag[v] > 0.0) d0inv[v] = 1.0 / diag[v];
        double bmax = 0.0;
        for (int64_t v = 0; v < C->nvert; ++v) {
            if (!(diag[v] > 0.0)) continue;
            AxisSet set[3];
            int at[3];
            columns(v, set, at);
            const int len = set[0].len * set[1].len * set[2].len;
            double sabs = 0.0;
            for (int x = 0; x < len; ++x) {
                double &a = entry(v, x);
                if (C->n_coarse < C->nvert) {
                    const int64_t u = axis_at(set[0], x % set[0].len) +
                                      vd[0] * (axis_at(set[1], x / set[0].len % set[1].len) +
                                               (int64_t)vd[1] * axis_at(set[2], x / (set[0].len * set[1].len)));
                    if (!(diag[u] > 0.0)) a = 0.0;
                }
                sabs += std::fabs(a);
            }
            bmax = std::max(bmax, sabs * d0inv[v]);
        }
        if (!(bmax > 0.0)) fail(SEM_EINVAL, "sem_set_coarse: the coarse operator is zero");
        C->b = bmax;
        C->a = frac * bmax;
        C->a_val = cmalloc<double>(C, rows.size());
        C->d0inv = cmalloc<double>(C, d0inv.size());
        SEM_HIP(hipMemcpyAsync(C->a_val, rows.data(), sizeof(double) * rows.size(), hipMemcpyHostToDevice, s));
        SEM_HIP(hipMemcpyAsync(C->d0inv, d0inv.data(), sizeof(double) * d0inv.size(), hipMemcpyHostToDevice, s));
        // Chebyshev coefficients
        const double theta = 0.5 * (C->b + C->a), delta = 0.5 * (C->b - C->a), sigma = theta / delta;
        C->inv_theta = 1.0 / theta;
        double rho = 1.0 / sigma;
        std::vector<double> coef(2 * (size_t)k);
        for (int j = 0; j < k; ++j) {
            const double rho_new = 1.0 / (2.0 * sigma - rho);
            coef[j] = rho_new * rho;
            coef[k + j] = 2.0 * rho_new / delta;
            rho = rho_new;
        }
        C->coef = cmalloc<double>(C, coef.size());
        SEM_HIP(hipMemcpyAsync(C->coef, coef.data(), sizeof(double) * coef.size(), hipMemcpyHostToDevice, s));
        C->z0 = cmalloc<double>(C, C->nvert);
        for (int q = 0; q < 2 && coarse_launches(k) > 1; ++q) {
            C->res[q] = cmalloc<double>(C, C->nvert);
            C->d[q] = cmalloc<double>(C, C->nvert);
        }
        C->partial8 = cmalloc<double>(C, (size_t)E * 8);
        build_tiles(C, h, vd, s);
        C->dot_blocks = std::min(C->tiles.n, kMaxCoarseDotBlocks);
        SEM_HIP(hipMemsetAsync(C->z0, 0, sizeof(double) * C->nvert, s));
        SEM_HIP(hipStreamSynchronize(s));
    } catch (...) {
        coarse_free(C);
        throw;
    }
    return C;
}

// launches F<N> for the mesh's order
#define SEM_COARSE_ORDER_SWITCH(N, CALL)                                                                  \
    switch (N) {                                                                                       \
    case 1: CALL(1); break;  case 2: CALL(2); break;   case 3: CALL(3); break;   case 4: CALL(4); break;  \
    case 5: CALL(5); break;  case 6: CALL(6); break;   case 7: CALL(7); break;   case 8: CALL(8); break;  \
    case 9: CALL(9); break;  case 10: CALL(10); break; case 11: CALL(11); break; case 12: CALL(12); break; \
    default: fail(SEM_EUNSUPPORTED, "coarse term: order out of range");                               \
    }

static int elem_blocks(int64_t E) { return (int)std::max<int64_t>(1, std::min<int64_t>((E + 3) / 4, 8192)); }

template <typename T>
int coarse_update(sem_mesh *m, T *r, const T *w, const T *inv, const PcgState *st, double *partial, bool with_rz,
                  hipStream_t s)
{
    CoarseSpace *C = m->coarse;
    const int64_t E = m->h.E;
    const int blocks = elem_blocks(E);
    const int rz = with_rz ? 1 : 0;
#define SEM_UPD(n)                                                                                              \
    hipLaunchKernelGGL((update_restrict_kernel<T, n>), dim3(blocks), dim3(256), 0, s, E, st, r, w, inv, m->mult, \
                       C->qw, partial, C->partial8, rz)
    SEM_COARSE_ORDER_SWITCH(m->h.N, SEM_UPD)
#undef SEM_UPD
    SEM_HIP(hipGetLastError());
    return blocks;
}
template int coarse_update<double>(sem_mesh *, double *, const double *, const double *, const PcgState *, double *,
                                   bool, hipStream_t);
template int coarse_update<float>(sem_mesh *, float *, const float *, const float *, const PcgState *, double *,
                                  bool, hipStream_t);

static int64_t round32(int64_t n) { return (n + 31) / 32 * 32; }

int64_t coarse_work_doubles(const CoarseSpace *C, int64_t E)
{
    return round32(E * 8) + (coarse_launches(C->k) > 1 ? 5 : 1) * round32(C->nvert);
}

CoarseWork coarse_work_carve(const CoarseSpace *C, int64_t E, double *base)
{
    CoarseWork W;
    double *q = base;
    auto take = [&](int64_t n) {
        double *r = q;
        q += round32(n);
        return r;
    };
    W.partial8 = take(E * 8);
    W.z0 = take(C->nvert);
    for (int q = 0; q < 2; ++q) {
        const bool more = coarse_launches(C->k) > 1;
        W.res[q] = more ? take(C->nvert) : nullptr;
        W.d[q] = more ? take(C->nvert) : nullptr;
    }
    return W;
}

template <typename T>
void coarse_restrict(sem_mesh *m, const T *r, const T *inv, hipStream_t s)
{
    CoarseSpace *C = m->coarse;
    const int64_t E = m->h.E;
#define SEM_RES(n)                                                                                                  \
    hipLaunchKernelGGL((restrict_elem_kernel<T, n>), dim3(elem_blocks(E)), dim3(256), 0, s, E, r, m->mult, inv, \
                       C->qw, C->partial8)
    SEM_COARSE_ORDER_SWITCH(m->h.N, SEM_RES)
#undef SEM_RES
    SEM_HIP(hipGetLastError());
}
template void coarse_restrict<double>(sem_mesh *, const double *, const double *, hipStream_t);
template void coarse_restrict<float>(sem_mesh *, const float *, const float *, hipStream_t);

CoarseChain coarse_chain(const CoarseSpace *C, const CoarseWork &W)
{
    CoarseChain c;
    c.k = C->k;
    c.inv_theta = C->inv_theta;
    c.coef = C->coef;
    c.a_val = C->a_val;
    c.d0inv = C->d0inv;
    c.partial8 = W.partial8;
    c.z0 = W.z0;
    for (int q = 0; q < 2; ++q) {
        c.res[q] = W.res[q];
        c.d[q] = W.d[q];
    }
    c.tiles = C->tiles;
    return c;
}

int coarse_solve(sem_mesh *m, double *dot_pairs, const PcgState *st, hipStream_t s)
{
    CoarseSpace *C = m->coarse;
    const CoarseChain chain =
        coarse_chain(C, {C->partial8, C->z0, {C->res[0], C->res[1]}, {C->d[0], C->d[1]}});
    const int launches = coarse_launches(C->k);
    for (int q = 0; q < launches; ++q)
        hipLaunchKernelGGL(coarse_tile_kernel, dim3(C->dot_blocks), dim3(kTileThreads), kTileLds, s, chain, q,
                           q == launches - 1 ? dot_pairs : nullptr, st);
    SEM_HIP(hipGetLastError());
    return C->dot_blocks;
}

void coarse_jacobi_prolong(sem_mesh *m, const double *r, double *z, hipStream_t s)
{
    CoarseSpace *C = m->coarse;
    const int64_t E = m->h.E;
#define SEM_PROLONG(n)                                                                                     \
    hipLaunchKernelGGL(prolong_kernel<n>, dim3((unsigned)((E + kPrElems<n> - 1) / kPrElems<n>)), dim3(256), 0, s, E, \
                       C->evert, C->z0, C->qw, m->inv64, r, z)
    SEM_COARSE_ORDER_SWITCH(m->h.N, SEM_PROLONG)
#undef SEM_PROLONG
    SEM_HIP(hipGetLastError());
}

// ---------------------------------------------------------------------------
// The coarse term of a batch's slots.  Each phase is one launch over the work
// items of all slots that take part, whatever their orders and sizes (slot by
// slot, the eight small launches of a slot took about 80 us an iteration).

#define SEM_BATCH_COARSE_ORDERS(X) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10)

template <typename T>
__device__ inline bool coarse_skips(const SlotDesc &sd, int at_start)
{
    return !at_start && sd.st[sizeof(T) == 8 ? 0 : 1].done;
}

// element sums of the items' elements, one wavefront per element
template <typename T>
__global__ __launch_bounds__(256) void batch_restrict_kernel(const SlotDesc *__restrict__ slots,
                                                             const CoarseDesc *__restrict__ cd, GroupDev g,
                                                             int at_start)
{
    constexpr int prec = sizeof(T) == 8 ? 0 : 1;
    __shared__ double sqw[2 * (SEM_MAX_ORDER + 1)];
    const int64_t n = g.counts[kCountCoarse];
    for (int64_t it = blockIdx.x; it < n; it += gridDim.x) {
        const Item item = g.ce_items[it];
        const SlotDesc &sd = slots[item.slot];
        const CoarseDesc &C = cd[item.slot];
        if (coarse_skips<T>(sd, at_start)) continue;  // uniform over the workgroup
        __syncthreads();
        if ((int)threadIdx.x < 2 * (C.N + 1)) sqw[threadIdx.x] = C.qw[threadIdx.x];
        __syncthreads();
        const T *r = static_cast<const T *>(sd.r[prec]), *inv = static_cast<const T *>(sd.inv[prec]);
        const int64_t e0 = (int64_t)item.local * kCoarseElems;
        const int64_t e1 = e0 + kCoarseElems < C.E ? e0 + kCoarseElems : C.E;
        for (int64_t e = e0 + (threadIdx.x >> 6); e < e1; e += 4) {
            switch (C.N) {
#define SEM_BRC(nn) \
            case nn: restrict_element<T, nn>(e, r, sd.mult, inv, sqw, C.partial8); break;
                SEM_BATCH_COARSE_ORDERS(SEM_BRC)
#undef SEM_BRC
            }
        }
    }
}

// zc = masked P z0 on the items' elements
template <typename T>
__global__ __launch_bounds__(256) void batch_prolong_kernel(const SlotDesc *__restrict__ slots,
                                                            const CoarseDesc *__restrict__ cd, GroupDev g,
                                                            int at_start)
{
    const int64_t n = g.counts[kCountCoarse];
    for (int64_t it = blockIdx.x; it < n; it += gridDim.x) {
        const Item item = g.ce_items[it];
        const SlotDesc &sd = slots[item.slot];
        const CoarseDesc &C = cd[item.slot];
        if (coarse_skips<T>(sd, at_start)) continue;
        T *zc = static_cast<T *>(const_cast<void *>(sd.zc));
        const int P2 = (C.N + 1) * (C.N + 1);
        const int64_t e0 = (int64_t)item.local * kCoarseElems;
        const int64_t ne = e0 + kCoarseElems < C.E ? kCoarseElems : C.E - e0;
        for (int q = threadIdx.x; q < ne * P2; q += 256) {
            switch (C.N) {
#define SEM_BPC(nn)                                                                                          \
            case nn:                                                                                         \
                prolong_column<nn, false, T>(e0 + q / ((nn + 1) * (nn + 1)), q % ((nn + 1) * (nn + 1)), C.evert, \
                                             C.z0, C.qw, C.inv64, nullptr, zc);                              \
                break;
                SEM_BATCH_COARSE_ORDERS(SEM_BPC)
#undef SEM_BPC
            }
        }
    }
}

// Chebyshev launch `launch` of the slots that have one (coarse_tile)
template <typename T>
__global__ __launch_bounds__(kTileThreads) void batch_tile_kernel(const SlotDesc *__restrict__ slots,
                                                                  const CoarseDesc *__restrict__ cd, GroupDev g,
                                                                  int launch, int at_start)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int64_t n = g.counts[kCountCoarse + 1];
    for (int64_t it = blockIdx.x; it < n; it += gridDim.x) {
        const Item item = g.cv_items[it];
        const CoarseDesc &C = cd[item.slot];
        const int launches = coarse_launches(C.chain.k);
        if (launch >= launches || coarse_skips<T>(slots[item.slot], at_start)) continue;
        double p[1] = {coarse_tile(C.chain, item.local, launch, reinterpret_cast<double *>(smem_raw))};
        if (launch == launches - 1) {
            block_reduce_store<1>(p, g.cv_partial + it, 0);
            __syncthreads();
        }
    }
}

template <typename T>
static hipError_t batch_coarse_t(bool at_start, int steps, const SlotDesc *slots, const CoarseDesc *cdesc,
                                 const GroupDev &g, const BatchLaunch &L, hipStream_t s)
{
    const int st = at_start ? 1 : 0;
    const dim3 grid(L.vec_grid), block(256);
    hipLaunchKernelGGL(batch_restrict_kernel<T>, grid, block, 0, s, slots, cdesc, g, st);
    // a workgroup takes 87 KB of LDS, so a compute unit holds one, and the second
    // half starts where the first is done (256, with more items each: the same
    // 49.7 ms for 12 boxes of up to 1024 elements)
    const dim3 tile_grid(std::min(L.vec_grid, 512));
    for (int q = 0; q < coarse_launches(steps); ++q)
        hipLaunchKernelGGL(batch_tile_kernel<T>, tile_grid, dim3(kTileThreads), kTileLds, s, slots, cdesc, g, q, st);
    hipLaunchKernelGGL(batch_prolong_kernel<T>, grid, block, 0, s, slots, cdesc, g, st);
    return hipGetLastError();
}

hipError_t batch_coarse(int prec, bool at_start, int steps, const SlotDesc *slots, const CoarseDesc *cdesc,
                        const GroupDev &g, const BatchLaunch &L, hipStream_t s)
{
    return prec == 0 ? batch_coarse_t<double>(at_start, steps, slots, cdesc, g, L, s)
                     : batch_coarse_t<float>(at_start, steps, slots, cdesc, g, L, s);
}

void launch_jacobi(int64_t n, const double *inv, const double *r, double *z, hipStream_t s)
{
    hipLaunchKernelGGL(jacobi_kernel, dim3(vec_blocks(n)), dim3(256), 0, s, n, inv, r, z);
    SEM_HIP(hipGetLastError());
}

}  // namespace sem
