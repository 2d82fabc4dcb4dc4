// schwarz.hip -- the sum over overlapping local subdomains of Eq. 6 on the
// GPU:  z = sum_k R_k^T A_k^{-1} R_k r.
//
//  * Subdomain k is element k extended by one node layer into each
//    neighbour that exists (also across periodic faces); nodes on Dirichlet
//    faces are not unknowns.  Its extended index range per direction is
//    lo .. lo+count-1 within -1 .. N+1.
//  * A_k is separable (the fast-diagonalisation form): with the 1-D GLL
//    stiffness A_d and lumped mass B_d of the element's mean edge length in
//    direction d, assembled on the element and its existing neighbours (same
//    length) and restricted to the kept indices,
//        A_k = B_t x B_s x A_r + B_t x A_s x B_r + A_t x B_s x B_r.
//    With S_d^T B_d S_d = I and S_d^T A_d S_d = diag(lam_d),
//        A_k^{-1} = (S_t x S_s x S_r) diag(1/(lam_r + lam_s + lam_t)) (S_t x S_s x S_r)^T,
//    six 1-D contractions per element (fdm_kernel, one workgroup per
//    element, the element in LDS).  The 1-D factors are computed on the host
//    and shared by all elements with the same (length, side kinds).
//  * The local solutions are summed into every node they cover
//    (assemble_kernel): a node receives the contributions of all extended
//    elements that hold it, added in ascending (unwrapped) element order per
//    direction, so every copy of a shared node gets the same bits.
//  * <r, z> for CG is taken inside fdm_kernel as sum_k (R_k r) . y_k, i.e. the
//    sum over modes of yhat^2 / (lam_r + lam_s + lam_t), yhat = S^T R_k r.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>
#include <tuple>
#include <vector>

#include "coarse.hpp"
#include "kernels.hpp"
#include "operator.hpp"
#include "schwarz.hpp"

namespace sem {

struct Lattice {
    int nel[3];
    int periodic[3];
    int dirichlet;  // bit 2d (2d+1): Dirichlet on the low (high) face of axis d
};

__host__ __device__ inline bool has_left(const Lattice &L, int d, int pos) { return pos > 0 || L.periodic[d]; }
__host__ __device__ inline bool has_right(const Lattice &L, int d, int pos)
{
    return pos < L.nel[d] - 1 || L.periodic[d];
}
// ---------------------------------------------------------------------------
// device kernels

// Kept range of the extended positions (extended index + 1, 0..N+2) of an
// element at pos along axis d: every position of an existing neighbour, none
// beyond a free face, none on a Dirichlet face.
__host__ __device__ inline int kept_lo(const Lattice &L, int d, int pos)
{
    return has_left(L, d, pos) ? 0 : (((L.dirichlet >> (2 * d)) & 1) ? 2 : 1);
}
__host__ __device__ inline int kept_hi(const Lattice &L, int d, int pos, int n)
{
    return has_right(L, d, pos) ? n - 1 : (((L.dirichlet >> (2 * d + 1)) & 1) ? n - 3 : n - 2);
}

// workgroup of the local solves: the (N+3)^2 lines rounded up to wavefronts
template <int N>
constexpr int kFdmThreads = ((N + 3) * (N + 3) + 63) / 64 * 64;

// put(b, sum_a M[b][a] x[a]) for every row b of the 1-D factors M
// (workgroup-uniform: scalar loads).  The next row is loaded while the
// present one is worked on; unrolled further, the rows of a whole matrix are
// hoisted and spill the scalar registers.
template <int n, typename Put>
__device__ inline void fdm_line(const double *__restrict__ M, const double (&x)[n], const Put &put)
{
    double s[n];
#pragma unroll
    for (int a = 0; a < n; ++a) s[a] = M[a];
#pragma unroll 2
    for (int b = 0; b < n; ++b) {
        const double *next = M + (b + 1 < n ? b + 1 : b) * n;
        double t[n];
#pragma unroll
        for (int a = 0; a < n; ++a) t[a] = next[a];
        double v = 0.0;
#pragma unroll
        for (int a = 0; a < n; ++a) v += s[a] * x[a];
        put(b, v);
#pragma unroll
        for (int a = 0; a < n; ++a) s[a] = t[a];
    }
}

// One workgroup per element (persistent walk); lane (l0, l1) < n^2 owns one
// line of the extended element in every contraction.  The element's lines are
// gathered along t straight into registers (the x and y neighbours of a lane
// do not change along its line), contracted there, and pass through one
// element of LDS: a lane alone reads and rewrites its line of a direction, so
// each direction works in place and needs one barrier.  Order t, s, r, scale,
// r, s, t: the two r contractions and the scaling stay in registers and the
// last t contraction goes straight to memory.  An odd row pitch keeps lines
// along r free of bank conflicts.
// <R_k r, y_k> equals sum over modes of yhat^2 / (lam_r + lam_s + lam_t),
// yhat = S^T R_k r, and is taken where the scaling is applied.
// With partial8, the element's eight hat-weighted sums of its own nodes
// (coarse restriction, weights cq) are taken from the gathered lines: a node's
// multiplicity and mask follow from the sides of the element.
// Bound by FP64 vector issue (12 (N+3)^4 flops an element, 100 of 128 lanes
// at N = 7; the vector unit is busy about 80% of the time).  On the 24x24x48
// pipe (N = 7, 27,648 elements) 168 us with the restriction, where the form
// with every stage through LDS and a lane per gathered node took 217 us and
// the separate restriction 102 us.  Not kept: whole matrices unrolled (264 us:
// 301 spilled scalar registers).
template <int N>
__global__ __launch_bounds__(256) void fdm_kernel(int64_t E, Lattice L, const double *__restrict__ r,
                                                  const int32_t *__restrict__ tidx,
                                                  const double *__restrict__ table, double *__restrict__ zext,
                                                  double *__restrict__ partial, const double *__restrict__ cq,
                                                  double *__restrict__ partial8, const PcgState *__restrict__ st)
{
    constexpr int P = N + 1, P2 = P * P, P3 = P2 * P;
    constexpr int n = N + 3, n2 = n * n, n3 = n2 * n, TE = 2 * n2 + n;
    constexpr int pr = n | 1, pp = n * pr;  // row and plane pitch in LDS
    if (st && st->done) return;
    __shared__ double U[n * pp];
    __shared__ double T[2 * n2], Q[4 * n], sq[2 * P];
    const int tid = threadIdx.x;
    if (partial8) {
        if (tid < 2 * P) sq[tid] = cq[tid];
        __syncthreads();
    }
    const bool line = tid < n2;
    const int l0 = tid % n, l1 = line ? tid / n : 0;
    double dot = 0.0;
    const XcdRange X = xcd_range(E);
    for (int64_t e = X.first; e < X.hi; e += X.step) {
        const int ei = (int)e;
        const int pos[3] = {ei % L.nel[0], (ei / L.nel[0]) % L.nel[1], ei / (L.nel[0] * L.nel[1])};
        // the element's 1-D factors S, S^T, lam: workgroup-uniform addresses (scalar loads)
        const double *S[3];
#pragma unroll
        for (int d = 0; d < 3; ++d) S[d] = table + (int64_t)tidx[e * 3 + d] * TE;
        double x[n];
        // R_k r along t: the column (l0, l1) lies in the element or in an x, y
        // or diagonal neighbour (r is continuous: any copy of a node holds its
        // value); 0 beyond the kept range
        {
            int pe[2], lc[2];
            bool ok = line;
#pragma unroll
            for (int d = 0; d < 2; ++d) {
                const int a = d == 0 ? l0 : l1;
                int p = pos[d], c = a - 1;
                if (a == 0) { p -= 1; c = N - 1; }
                if (a == n - 1) { p += 1; c = 1; }
                if (p < 0) p += L.nel[d];
                if (p >= L.nel[d]) p -= L.nel[d];
                ok = ok && a >= kept_lo(L, d, pos[d]) && a <= kept_hi(L, d, pos[d], n);
                pe[d] = p;
                lc[d] = c;
            }
            const int lo2 = kept_lo(L, 2, pos[2]), hi2 = kept_hi(L, 2, pos[2], n);
            const int zdn = pos[2] > 0 ? pos[2] - 1 : L.nel[2] - 1, zup = pos[2] + 1 < L.nel[2] ? pos[2] + 1 : 0;
            const int64_t exy = pe[0] + (int64_t)L.nel[0] * pe[1], nxy = (int64_t)L.nel[0] * L.nel[1];
            const double *col = r + exy * P3 + lc[0] + P * lc[1];
            const double *own = col + pos[2] * nxy * P3;
#pragma unroll
            for (int c = 0; c < n; ++c) {
                const double *src = c == 0 ? col + zdn * nxy * P3 + (N - 1) * P2
                                           : (c == n - 1 ? col + zup * nxy * P3 + P2 : own + (c - 1) * P2);
                double v = 0.0;
                if (ok && c >= lo2 && c <= hi2) v = *src;
                x[c] = v;
            }
        }
        if (partial8 && line) {
            // two t-sums of the column, weighted by 1/mult of its nodes
            const bool mine = l0 >= 1 && l0 <= n - 2 && l1 >= 1 && l1 <= n - 2;
            double w = mine ? 1.0 : 0.0;
#pragma unroll
            for (int d = 0; d < 2; ++d) {
                const int a = d == 0 ? l0 : l1;
                if ((a == 1 && has_left(L, d, pos[d])) || (a == n - 2 && has_right(L, d, pos[d]))) w *= 0.5;
            }
            double t0 = 0.0, t1 = 0.0;
#pragma unroll
            for (int c = 1; c <= n - 2; ++c) {
                double v = x[c];
                if (c == 1 && has_left(L, 2, pos[2])) v *= 0.5;
                if (c == n - 2 && has_right(L, 2, pos[2])) v *= 0.5;
                t0 += sq[c - 1] * v;
                t1 += sq[P + c - 1] * v;
            }
            T[tid] = w * t0;
            T[n2 + tid] = w * t1;
        }
        // S_t^T; the lane's line of U was read by this lane alone (the last
        // stage of the previous element)
        if (line) {
            double *u = U + l1 * pr + l0;
            fdm_line<n>(S[2] + n2, x, [&](int c, double v) { u[c * pp] = v; });
        }
        __syncthreads();
        // S_s^T on the line (r = l0, t = l1)
        if (line) {
            double *u = U + l1 * pp + l0;
#pragma unroll
            for (int b = 0; b < n; ++b) x[b] = u[b * pr];
            fdm_line<n>(S[1] + n2, x, [&](int b, double v) { u[b * pr] = v; });
        }
        if (partial8 && tid < 4 * n) {
            const int cx = tid & 1, ct = (tid >> 1) & 1, b = tid >> 2;
            double s = 0.0;
#pragma unroll
            for (int a = 1; a <= n - 2; ++a) s += sq[cx * P + a - 1] * T[ct * n2 + b * n + a];
            Q[tid] = s;
        }
        __syncthreads();
        // S_r^T, the scaling and S_r on the line (s = l0, t = l1)
        if (line) {
            double *u = U + l1 * pp + l0 * pr;
#pragma unroll
            for (int a = 0; a < n; ++a) x[a] = u[a];
            const double lst = S[1][2 * n2 + l0] + S[2][2 * n2 + l1];
            fdm_line<n>(S[0] + n2, x, [&](int b, double v) {
                const double den = S[0][2 * n2 + b] + lst;
                const double q = den > 0.0 ? v / den : 0.0;
                dot += v * q;
                u[b] = q;
            });
#pragma unroll
            for (int b = 0; b < n; ++b) x[b] = u[b];
            fdm_line<n>(S[0], x, [&](int a, double v) { u[a] = v; });
        }
        if (partial8 && tid < 8) {
            const int cx = tid & 1, cy = (tid >> 1) & 1, ct = tid >> 2;
            double s = 0.0;
#pragma unroll
            for (int b = 1; b <= n - 2; ++b) s += sq[cy * P + b - 1] * Q[b * 4 + ct * 2 + cx];
            partial8[e * 8 + tid] = s;
        }
        __syncthreads();
        // S_s
        if (line) {
            double *u = U + l1 * pp + l0;
#pragma unroll
            for (int b = 0; b < n; ++b) x[b] = u[b * pr];
            fdm_line<n>(S[1], x, [&](int b, double v) { u[b * pr] = v; });
        }
        __syncthreads();
        // S_t on the line (r = l0, s = l1), to the extended solution
        if (line) {
#pragma unroll
            for (int c = 0; c < n; ++c) x[c] = U[c * pp + l1 * pr + l0];
            double *out = zext + e * n3 + tid;
            fdm_line<n>(S[2], x, [&](int c, double v) { st_stream(v, out + c * n2); });
        }
    }
    if (partial) {
        __syncthreads();
        double p[2] = {0.0, dot};
        block_reduce_store<2>(p, partial, 2);
    }
}

// elements per workgroup of the column kernels (one lane per (i, j) column)
template <int N>
constexpr int kColElems = 256 / ((N + 1) * (N + 1)) > 0 ? 256 / ((N + 1) * (N + 1)) : 1;

// z at every local node: the sum of the extended solutions that hold it, 0 at
// Dirichlet nodes, plus (COARSE) the trilinear coarse correction.  Per
// direction a node of index idx is held by its element and, when idx <= 1 or
// idx >= N-1, by the neighbour on that side if it exists (N >= 3: at most two
// holders per direction, added in ascending offset).  One lane per (i, j)
// column: the x and y holders are found once per column, the z holders are
// the same for a whole plane, and an address is formed by one addition per
// load; a load past the holders is not issued.  On the 24x24x48 pipe (N = 7,
// 27,648 elements) 105 us with the coarse term, where the lane-per-node form
// with its separate prolongation pass took 144 + 167 us; it moves 345 MB (56 us
// at a copy's rate) and is bound by its partly filled loads.  Not kept: more
// loads in flight per lane (half a column 111 us, a whole one 116 us; the
// waves that fit fell from 8 to 5 and 3 per SIMD).
// COLUMN false: one lane per node, plane blockIdx.y.  On a mesh whose columns
// leave compute units idle, a lane's planes are a chain of memory latencies:
// 64 elements of N = 7 3.8 us instead of 6.7, M^-1 r 11.9 instead of 15.0.
template <int N, bool COARSE, bool COLUMN>
__global__ __launch_bounds__(256) void assemble_kernel(int64_t E, Lattice L, const double *__restrict__ zext,
                                                       const int32_t *__restrict__ evert,
                                                       const double *__restrict__ z0, const double *__restrict__ cq,
                                                       double *__restrict__ z, const PcgState *__restrict__ st)
{
    static_assert(N >= 3, "two holders per direction");
    constexpr int P = N + 1, P2 = P * P, P3 = P2 * P;
    constexpr int n = N + 3, n2 = n * n, n3 = n2 * n;
    constexpr int EB = kColElems<N>;
    if (st && st->done) return;
    const int el = threadIdx.x / P2, ij = threadIdx.x - el * P2;
    const int i = ij % P, j = ij / P;
    // one contiguous range of workgroups per XCD (as xcd_range)
    const unsigned nb = gridDim.x, per = nb / 8, rem = nb % 8, xcd = blockIdx.x % 8, kb = blockIdx.x / 8;
    const unsigned lb = (xcd < rem ? xcd * (per + 1) : rem * (per + 1) + (xcd - rem) * per) + kb;
    const int64_t e = (int64_t)lb * EB + el;
    if (el >= EB || e >= E) return;
    const int ei = (int)e;
    const int pos[3] = {ei % L.nel[0], (ei / L.nel[0]) % L.nel[1], ei / (L.nel[0] * L.nel[1])};
    double cs0 = 0.0, cs1 = 0.0;
    if (COARSE) {
        double zc[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) zc[c] = z0[evert[e * 8 + c]];
        const double ai0 = cq[i], ai1 = cq[P + i], aj0 = cq[j], aj1 = cq[P + j];
        cs0 = aj0 * (ai0 * zc[0] + ai1 * zc[1]) + aj1 * (ai0 * zc[2] + ai1 * zc[3]);
        cs1 = aj0 * (ai0 * zc[4] + ai1 * zc[5]) + aj1 * (ai0 * zc[6] + ai1 * zc[7]);
    }
    // per direction: offset to the holders' values (ascending element offset)
    // relative to this element's own, whether each exists, and the masks
    const int64_t estep[3] = {n3, (int64_t)L.nel[0] * n3, (int64_t)L.nel[0] * L.nel[1] * n3};
    auto wrap_lo = [&](int d) -> int64_t { return (pos[d] > 0 ? -1 : L.nel[d] - 1) * estep[d]; };
    auto wrap_hi = [&](int d) -> int64_t { return (pos[d] + 1 < L.nel[d] ? 1 : 1 - L.nel[d]) * estep[d]; };
    auto walled = [&](int d, int idx) {
        return (idx == 0 && !has_left(L, d, pos[d]) && ((L.dirichlet >> (2 * d)) & 1)) ||
               (idx == N && !has_right(L, d, pos[d]) && ((L.dirichlet >> (2 * d + 1)) & 1));
    };
    bool ok[2][2];
    int64_t off[2][2];
#pragma unroll
    for (int d = 0; d < 2; ++d) {
        const int idx = d == 0 ? i : j, step = d == 0 ? 1 : n;
        const bool lo_side = idx <= 1, hi_side = idx >= N - 1;
        const int64_t own = (idx + 1) * step;
        ok[d][0] = lo_side ? has_left(L, d, pos[d]) : true;
        off[d][0] = lo_side ? wrap_lo(d) + (idx + N + 1) * step : own;
        ok[d][1] = lo_side ? true : (hi_side && has_right(L, d, pos[d]));
        off[d][1] = lo_side ? own : wrap_hi(d) + (idx - N + 1) * step;
    }
    const bool wall_ij = walled(0, i) || walled(1, j);
    const double *base = zext + e * n3;
    const double *src[4];
    bool good[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        src[c] = base + off[0][c & 1] + off[1][c >> 1];
        good[c] = ok[0][c & 1] && ok[1][c >> 1];
    }
    const bool zl = has_left(L, 2, pos[2]), zr = has_right(L, 2, pos[2]);
    const int64_t zlo = wrap_lo(2), zhi = wrap_hi(2);
#pragma unroll
    for (int kk = 0; kk < (COLUMN ? P : 1); ++kk) {
        const int k = COLUMN ? kk : (int)blockIdx.y;
        double val[8];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            // holder h along z of plane k, ascending offset; absent holders add 0
            const bool lo_side = k <= 1, hi_side = k >= N - 1;
            const bool okz = lo_side ? (h == 1 || zl) : (h == 0 || (hi_side && zr));
            const int64_t oz = lo_side ? (h == 0 ? zlo + (k + N + 1) * n2 : (int64_t)(k + 1) * n2)
                                       : (h == 0 ? (int64_t)(k + 1) * n2 : zhi + (k - N + 1) * n2);
            if (!lo_side && !hi_side && h == 1) break;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                val[h * 4 + c] = 0.0;
                if (okz && good[c]) val[h * 4 + c] = src[c][oz];
            }
        }
        double s = 0.0;
#pragma unroll
        for (int c = 0; c < 8; ++c)
            if (c < 4 || k <= 1 || k >= N - 1) s += val[c];
        if (COARSE) s += cq[k] * cs0 + cq[P + k] * cs1;
        st_stream(wall_ij || walled(2, k) ? 0.0 : s, z + e * P3 + k * P2 + ij);
    }
}

// The same at N = 2, where a node of index 1 is held by both neighbours: up
// to three holders per direction, one lane per node.
template <bool COARSE>
__global__ __launch_bounds__(256) void assemble2_kernel(int64_t E, Lattice L, const double *__restrict__ zext,
                                                        const int32_t *__restrict__ evert,
                                                        const double *__restrict__ z0, const double *__restrict__ cq,
                                                        const double *__restrict__ inv, double *__restrict__ z,
                                                        const PcgState *__restrict__ st)
{
    constexpr int N = 2, P = N + 1, P2 = P * P, P3 = P2 * P;
    constexpr int n = N + 3, n2 = n * n, n3 = n2 * n;
    if (st && st->done) return;
    const int64_t nL = E * P3;
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < nL; q += (int64_t)gridDim.x * blockDim.x) {
        const int ei = (int)(q / P3);
        const int rem = (int)(q - (int64_t)ei * P3);
        const int idx[3] = {rem % P, (rem / P) % P, rem / P2};
        const int pos[3] = {ei % L.nel[0], (ei / L.nel[0]) % L.nel[1], ei / (L.nel[0] * L.nel[1])};
        double s = 0.0;
        bool ok[3][3];
        int el[3][3], ps[3][3];
#pragma unroll
        for (int d = 0; d < 3; ++d) {
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                const int delta = t - 1;
                const int at = idx[d] - delta * N + 1;
                int p2 = pos[d] + delta;
                bool v = at >= 0 && at < n;
                if (p2 < 0) { v = v && L.periodic[d]; p2 += L.nel[d]; }
                if (p2 >= L.nel[d]) { v = v && L.periodic[d]; p2 -= L.nel[d]; }
                ok[d][t] = v && at >= kept_lo(L, d, p2) && at <= kept_hi(L, d, p2, n);
                el[d][t] = p2;
                ps[d][t] = at;
            }
        }
#pragma unroll
        for (int tz = 0; tz < 3; ++tz)
#pragma unroll
            for (int ty = 0; ty < 3; ++ty)
#pragma unroll
                for (int tx = 0; tx < 3; ++tx) {
                    if (!(ok[0][tx] && ok[1][ty] && ok[2][tz])) continue;
                    const int e2 = el[0][tx] + L.nel[0] * (el[1][ty] + L.nel[1] * el[2][tz]);
                    s += zext[(int64_t)e2 * n3 + ps[0][tx] + n * ps[1][ty] + n2 * ps[2][tz]];
                }
        if (COARSE) s += hat_value(evert + (int64_t)ei * 8, z0, cq, P, idx[0], idx[1], idx[2]);
        z[q] = ld_stream(inv + q) > 0.0 ? s : 0.0;
    }
}

// ---------------------------------------------------------------------------
// host: 1-D factors

// Eigen-decomposition of a symmetric n x n matrix (row-major) by cyclic
// Jacobi rotations: a = v diag(d) v^T, eigenvectors in the columns of v.
static void symmetric_eigen(std::vector<double> a, int n, std::vector<double> &v, std::vector<double> &d)
{
    v.assign((size_t)n * n, 0.0);
    for (int i = 0; i < n; ++i) v[(size_t)i * n + i] = 1.0;
    for (int sweep = 0; sweep < 100; ++sweep) {
        double off = 0.0, tot = 0.0;
        for (int p = 0; p < n; ++p)
            for (int q = 0; q < n; ++q) {
                const double x = a[(size_t)p * n + q] * a[(size_t)p * n + q];
                tot += x;
                if (p != q) off += x;
            }
        if (off <= 1e-32 * tot || off == 0.0) break;
        for (int p = 0; p < n - 1; ++p)
            for (int q = p + 1; q < n; ++q) {
                const double apq = a[(size_t)p * n + q];
                if (std::fabs(apq) < 1e-300) continue;
                const double theta = (a[(size_t)q * n + q] - a[(size_t)p * n + p]) / (2.0 * apq);
                const double t = (theta >= 0.0 ? 1.0 : -1.0) / (std::fabs(theta) + std::sqrt(theta * theta + 1.0));
                const double c = 1.0 / std::sqrt(t * t + 1.0), s = t * c;
                for (int k = 0; k < n; ++k) {  // columns p, q
                    const double akp = a[(size_t)k * n + p], akq = a[(size_t)k * n + q];
                    a[(size_t)k * n + p] = c * akp - s * akq;
                    a[(size_t)k * n + q] = s * akp + c * akq;
                }
                for (int k = 0; k < n; ++k) {  // rows p, q
                    const double apk = a[(size_t)p * n + k], aqk = a[(size_t)q * n + k];
                    a[(size_t)p * n + k] = c * apk - s * aqk;
                    a[(size_t)q * n + k] = s * apk + c * aqk;
                }
                for (int k = 0; k < n; ++k) {
                    const double vkp = v[(size_t)k * n + p], vkq = v[(size_t)k * n + q];
                    v[(size_t)k * n + p] = c * vkp - s * vkq;
                    v[(size_t)k * n + q] = s * vkp + c * vkq;
                }
            }
    }
    d.resize(n);
    for (int i = 0; i < n; ++i) d[i] = a[(size_t)i * n + i];
}

void fdm_1d(int N, const std::vector<double> &xi, const std::vector<double> &w, const std::vector<double> &D,
            double ell, int left, int right, std::vector<double> &S, std::vector<double> &lam, int &lo, int &count)
{
    (void)xi;
    const int P = N + 1, M = 3 * N + 1;
    std::vector<double> Ke((size_t)P * P), K((size_t)M * M, 0.0), B(M, 0.0);
    for (int a = 0; a < P; ++a)
        for (int b = 0; b < P; ++b) {
            double s = 0.0;
            for (int q = 0; q < P; ++q) s += D[(size_t)q * P + a] * w[q] * D[(size_t)q * P + b];
            Ke[(size_t)a * P + b] = (2.0 / ell) * s;
        }
    const int parts[3] = {left == kSideInterior ? 0 : -1, 1, right == kSideInterior ? 2 : -1};
    for (int p : parts) {
        if (p < 0) continue;
        for (int a = 0; a < P; ++a) {
            for (int b = 0; b < P; ++b) K[(size_t)(p * N + a) * M + p * N + b] += Ke[(size_t)a * P + b];
            B[p * N + a] += 0.5 * ell * w[a];
        }
    }
    lo = left == kSideInterior ? -1 : (left == kSideNeumann ? 0 : 1);
    const int hi = right == kSideInterior ? N + 1 : (right == kSideNeumann ? N : N - 1);
    count = hi - lo + 1;
    const int n = count;
    std::vector<double> C((size_t)n * n), sb(n);
    for (int a = 0; a < n; ++a) sb[a] = 1.0 / std::sqrt(B[N + lo + a]);
    for (int a = 0; a < n; ++a)
        for (int b = 0; b < n; ++b) C[(size_t)a * n + b] = K[(size_t)(N + lo + a) * M + N + lo + b] * sb[a] * sb[b];
    std::vector<double> Q;
    symmetric_eigen(C, n, Q, lam);
    S.assign((size_t)n * n, 0.0);
    for (int a = 0; a < n; ++a)
        for (int b = 0; b < n; ++b) S[(size_t)a * n + b] = Q[(size_t)a * n + b] * sb[a];
}

// ---------------------------------------------------------------------------
// host: set-up and launches

template <typename X>
static X *smalloc(SchwarzSpace *Z, size_t count)
{
    void *p = nullptr;
    SEM_HIP(hipMalloc(&p, std::max<size_t>(count * sizeof(X), 16)));
    Z->allocations.push_back(p);
    return static_cast<X *>(p);
}

void schwarz_free(SchwarzSpace *Z)
{
    if (!Z) return;
    for (void *p : Z->allocations) (void)hipFree(p);
    delete Z;
}

static Lattice lattice_of(const sem_mesh *m, int dirichlet)
{
    Lattice L{};
    for (int d = 0; d < 3; ++d) {
        L.nel[d] = m->h.nel[d];
        L.periodic[d] = m->h.periodic[d];
    }
    L.dirichlet = dirichlet;
    return L;
}

SchwarzSpace *schwarz_build(sem_mesh *m, hipStream_t s)
{
    const HostMesh &h = m->h;
    const int N = h.N, P = N + 1, n = N + 3;
    const int64_t E = h.E, P3 = (int64_t)P * P * P;
    if (E >= INT32_MAX) fail(SEM_EUNSUPPORTED, "sem_set_schwarz: too many elements");
    SchwarzSpace *Z = new SchwarzSpace();
    try {
        Z->n = n;
        int faces = h.desc.dirichlet_faces;
        if (faces < 0) {
            faces = 0;
            for (int d = 0; d < 3; ++d)
                if (!h.periodic[d]) faces |= 3 << (2 * d);
        }
        for (int d = 0; d < 3; ++d)
            if (h.periodic[d]) faces &= ~(3 << (2 * d));
        Z->dirichlet = faces;
        const Lattice L = lattice_of(m, faces);
        // element corner coordinates -> mean edge lengths
        HostMesh ch;
        sem_mesh_desc d = h.desc;
        d.vertices = h.vertices.empty() ? nullptr : h.vertices.data();
        build_host_coords(d, ch);
        const int64_t nL = ch.nL;
        auto X = [&](int64_t e, int i, int j, int k, int c) {
            return ch.xyz[(size_t)c * nL + e * P3 + i + P * (j + (int64_t)P * k)];
        };
        auto dist = [&](int64_t e, int i0, int j0, int k0, int i1, int j1, int k1) {
            const double dx = X(e, i1, j1, k1, 0) - X(e, i0, j0, k0, 0);
            const double dy = X(e, i1, j1, k1, 1) - X(e, i0, j0, k0, 1);
            const double dz = X(e, i1, j1, k1, 2) - X(e, i0, j0, k0, 2);
            return std::sqrt(dx * dx + dy * dy + dz * dz);
        };
        const int TE = 2 * n * n + n;
        std::map<std::tuple<double, int, int>, int32_t> index;
        std::vector<double> table;
        std::vector<int32_t> tidx((size_t)E * 3);
        std::vector<double> S1, lam;
        for (int64_t e = 0; e < E; ++e) {
            const int pos[3] = {(int)(e % h.nel[0]), (int)((e / h.nel[0]) % h.nel[1]),
                                (int)(e / ((int64_t)h.nel[0] * h.nel[1]))};
            const int c[2] = {0, N};
            double ell[3] = {0.0, 0.0, 0.0};
            for (int a : c)
                for (int b : c) {
                    ell[0] += dist(e, 0, a, b, N, a, b);  // r-edges at (j, k) = (a, b)
                    ell[1] += dist(e, a, 0, b, a, N, b);
                    ell[2] += dist(e, a, b, 0, a, b, N);
                }
            for (int dd = 0; dd < 3; ++dd) {
                const double len = ell[dd] / 4.0;
                const int left = has_left(L, dd, pos[dd]) ? kSideInterior
                                 : ((faces >> (2 * dd)) & 1) ? kSideDirichlet : kSideNeumann;
                const int right = has_right(L, dd, pos[dd]) ? kSideInterior
                                  : ((faces >> (2 * dd + 1)) & 1) ? kSideDirichlet : kSideNeumann;
                const auto key = std::make_tuple(len, left, right);
                auto it = index.find(key);
                if (it == index.end()) {
                    if (!(len > 0.0)) fail(SEM_EINVAL, "sem_set_schwarz: degenerate element edge");
                    int lo = 0, count = 0;
                    fdm_1d(N, h.xi, h.w, h.D, len, left, right, S1, lam, lo, count);
                    const size_t base = table.size();
                    table.resize(base + TE, 0.0);
                    // rows at the extended positions lo + 1 ..; absent positions and
                    // modes are zero rows and columns
                    for (int a = 0; a < count; ++a)
                        for (int b = 0; b < count; ++b) {
                            const double v = S1[(size_t)a * count + b];
                            table[base + (size_t)(lo + 1 + a) * n + b] = v;
                            table[base + (size_t)n * n + (size_t)b * n + lo + 1 + a] = v;
                        }
                    for (int b = 0; b < n; ++b) table[base + (size_t)2 * n * n + b] = b < count ? lam[b] : 1.0;
                    it = index.emplace(key, (int32_t)(table.size() / TE - 1)).first;
                }
                tidx[(size_t)e * 3 + dd] = it->second;
            }
        }
        Z->n_table = (int64_t)table.size() / TE;
        Z->tidx = smalloc<int32_t>(Z, tidx.size());
        Z->table = smalloc<double>(Z, table.size());
        Z->zext = smalloc<double>(Z, (size_t)E * n * n * n);
        Z->zs = smalloc<double>(Z, (size_t)h.nL);
        SEM_HIP(hipMemcpyAsync(Z->tidx, tidx.data(), sizeof(int32_t) * tidx.size(), hipMemcpyHostToDevice, s));
        SEM_HIP(hipMemcpyAsync(Z->table, table.data(), sizeof(double) * table.size(), hipMemcpyHostToDevice, s));
        SEM_HIP(hipStreamSynchronize(s));
    } catch (...) {
        schwarz_free(Z);
        throw;
    }
    return Z;
}

static int fdm_blocks(int64_t E) { return (int)std::max<int64_t>(1, std::min<int64_t>(E, kMaxSchwarzPairs)); }

// orders of the local solves
#define SEM_SCHWARZ_ORDER_SWITCH(N, CALL)                                                     \
    switch (N) {                                                                           \
    case 3: CALL(3); break;   case 4: CALL(4); break;   case 5: CALL(5); break;               \
    case 6: CALL(6); break;   case 7: CALL(7); break;   case 8: CALL(8); break;               \
    case 9: CALL(9); break;   case 10: CALL(10); break; case 11: CALL(11); break;             \
    case 12: CALL(12); break;                                                                 \
    default: fail(SEM_EUNSUPPORTED, "Schwarz: order out of range (2..12)");                   \
    }

int schwarz_solves(sem_mesh *m, const double *r, double *pairs, bool restrict_r, const PcgState *st, hipStream_t s)
{
    SchwarzSpace *Z = m->schwarz;
    const Lattice L = lattice_of(m, Z->dirichlet);
    const int64_t E = m->h.E;
    const int fb = fdm_blocks(E);
    const double *cq = restrict_r ? m->coarse->qw : nullptr;
    double *p8 = restrict_r ? m->coarse->partial8 : nullptr;
#define SEM_FDM(n)                                                                                                  \
    hipLaunchKernelGGL(fdm_kernel<n>, dim3(fb), dim3(kFdmThreads<n>), 0, s, E, L, r, Z->tidx, Z->table, Z->zext,     \
                       pairs, cq, p8, st)
    if (m->h.N == 2) SEM_FDM(2);
    else SEM_SCHWARZ_ORDER_SWITCH(m->h.N, SEM_FDM)
#undef SEM_FDM
    SEM_HIP(hipGetLastError());
    return fb;
}

void schwarz_assemble(sem_mesh *m, double *z, bool add_coarse, const PcgState *st, hipStream_t s)
{
    SchwarzSpace *Z = m->schwarz;
    const Lattice L = lattice_of(m, Z->dirichlet);
    const int64_t E = m->h.E;
    const int32_t *ev = add_coarse ? m->coarse->evert : nullptr;
    const double *z0 = add_coarse ? m->coarse->z0 : nullptr, *cq = add_coarse ? m->coarse->qw : nullptr;
    if (m->h.N == 2) {
        const dim3 grid(vec_blocks(m->h.nL));
        if (add_coarse)
            hipLaunchKernelGGL(assemble2_kernel<true>, grid, dim3(256), 0, s, E, L, Z->zext, ev, z0, cq, m->inv64, z, st);
        else
            hipLaunchKernelGGL(assemble2_kernel<false>, grid, dim3(256), 0, s, E, L, Z->zext, ev, z0, cq, m->inv64, z, st);
        SEM_HIP(hipGetLastError());
        return;
    }
    // a lane per node up to where its workgroups (N + 1 times those of the
    // columns) fill the device and repeat the columns' work for nothing: M^-1 r,
    // us per node and per column, N = 7 with 183 workgroups of columns 16.7 and
    // 17.9, with 250 18.2 and 17.3; N = 11 216 21.2 and 23.8, 512 26.1 and 23.9;
    // N = 3 108 11.3 and 12.3, 172 13.5 and 13.3
    const unsigned per_node = m->h.N <= 4 ? 128 : 208;
#define SEM_ASM_RUN(n, coarse, column, grid)                                                                        \
    hipLaunchKernelGGL((assemble_kernel<n, coarse, column>), grid, dim3(256), 0, s, E, L, Z->zext, ev, z0, cq, z, st)
#define SEM_ASM(n)                                                                                                 \
    do {                                                                                                           \
        const unsigned wgs = (unsigned)((E + kColElems<n> - 1) / kColElems<n>);                                    \
        if (wgs <= per_node) {                                                                                     \
            if (add_coarse) SEM_ASM_RUN(n, true, false, dim3(wgs, n + 1));                                         \
            else SEM_ASM_RUN(n, false, false, dim3(wgs, n + 1));                                                   \
        } else {                                                                                                   \
            if (add_coarse) SEM_ASM_RUN(n, true, true, dim3(wgs));                                                 \
            else SEM_ASM_RUN(n, false, true, dim3(wgs));                                                           \
        }                                                                                                          \
    } while (0)
    SEM_SCHWARZ_ORDER_SWITCH(m->h.N, SEM_ASM)
#undef SEM_ASM
#undef SEM_ASM_RUN
    SEM_HIP(hipGetLastError());
}

int schwarz_apply(sem_mesh *m, const double *r, double *z, double *pairs, const PcgState *st, hipStream_t s)
{
    const int n = schwarz_solves(m, r, pairs, false, st, s);
    schwarz_assemble(m, z, false, st, s);
    return n;
}

}  // namespace sem

extern "C" sem_status sem_host_fdm_1d(int N, double ell, int left, int right, double *S, double *lam, int *lo,
                                      int *count)
{
    using namespace sem;
    try {
        if (N < 1 || N > SEM_MAX_ORDER) fail(SEM_EINVAL, "sem_host_fdm_1d: N out of range");
        if (!(ell > 0.0)) fail(SEM_EINVAL, "sem_host_fdm_1d: ell must be positive");
        if (left < 0 || left > 2 || right < 0 || right > 2) fail(SEM_EINVAL, "sem_host_fdm_1d: unknown side kind");
        if (!S || !lam || !lo || !count) fail(SEM_EINVAL, "sem_host_fdm_1d: null argument");
        std::vector<double> xi, w, D, S1, l1;
        gll_rule(N, xi, w);
        lagrange_derivative(xi, D);
        int l = 0, c = 0;
        fdm_1d(N, xi, w, D, ell, left, right, S1, l1, l, c);
        std::memcpy(S, S1.data(), sizeof(double) * S1.size());
        std::memcpy(lam, l1.data(), sizeof(double) * l1.size());
        *lo = l;
        *count = c;
        return SEM_OK;
    } catch (const Failure &f) {
        return f.status;
    } catch (const std::bad_alloc &) {
        set_error("sem_host_fdm_1d: out of memory");
        return SEM_ENOMEM;
    }
}
