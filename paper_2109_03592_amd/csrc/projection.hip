// projection.hip -- projection onto previous solutions (section 2 of the
// paper accelerates successive solves this way, after Fischer).
//
// A basis x_1..x_l of earlier solutions is kept A-orthonormal together with
// A x_i.  For a new right-hand side the guess xbar = sum_i (x_i . b) x_i is
// the element of the span closest to the solution in the A-norm; PCG then
// starts from it.  A solution joins the basis after two passes of
// Gram-Schmidt in the A-inner product (x_i^T A v = x_i . (A v), unique-dof
// inner products) and A-normalisation; a remainder whose A-norm fell below
// drop_tol times the vector's own is dropped; a full basis restarts.
//
// Every step is bound by the passes over the basis (56.6 MB per vector on the
// 24x24x24 pipe at N = 7), so a solution joins in three of them:
//   1. X_i . A x of all i and x . A x in one;
//   2. the removal of those parts, which also takes the second pass's inner
//      products while X_i is in registers, and writes v, A v;
//   3. the second removal, which also takes v . A v.
// A vector is kept as step 3 left it and its 1 / |v|_A goes into the
// coefficients, instead of a pass that scales it; step 2 scales by the power
// of two next to |x|_A, so no product leaves the range the unit vectors had.
// The six additions and the projection of that pipe move 15.6 GB -> 11.7 GB
// this way, 4.07 -> 2.25 ms.  The kernels are compiled per count of vectors, up
// to kProjPass a launch: with the count a runtime bound the loads of one point
// wait for each other (five inner products, 340 MB, took 90 us; these take 65
// with x . A x among them, 400 MB).  A basis outgrows the
// caches, so its vectors are read past them (2.46 -> 2.25 ms; a basis of 8
// vectors of 22 MB would fit and loses 5%), and four workgroups per compute unit
// keep enough loads in flight (eight: 2.30 ms).
#include <algorithm>
#include <cmath>
#include <type_traits>
#include <vector>

#include "kernels.hpp"
#include "operator.hpp"
#include "sem_internal.hpp"

namespace sem {

constexpr int kMaxProj = 32;

constexpr int kProjPass = 8;       // vectors a launch takes
constexpr int kProjBlocks = 1024;  // four workgroups per compute unit

struct ProjPtrs {
    const double *v[kProjPass];
};
struct ProjScales {
    double s[kMaxProj];
};
// coef: the coefficients of a pass, x . A x, v . A v
constexpr int kCoefN0 = kMaxProj, kCoefN2 = kMaxProj + 1, kCoefSize = kMaxProj + 2;

// power of two next to 1 / |x|_A (1 where x has no norm: it will be dropped)
__host__ __device__ inline double unit_scale(double n0)
{
    if (!(n0 > 0.0) || !(n0 <= 1.7976931348623157e308)) return 1.0;
    int ex;
    frexp(n0, &ex);
    return ldexp(1.0, -(ex >> 1));
}

// partial[b * nv + i] = sum over this workgroup's points of V_i y / mult;
// NORM: [b * nv + L] the same of x
template <int L, bool NORM>
__global__ __launch_bounds__(256) void proj_dots_kernel(int64_t n, ProjPtrs V, const double *__restrict__ y,
                                                        const double *__restrict__ x,
                                                        const uint8_t *__restrict__ mult,
                                                        double *__restrict__ partial)
{
    constexpr int NV = L + (NORM ? 1 : 0);
    double acc[NV];
#pragma unroll
    for (int i = 0; i < NV; ++i) acc[i] = 0.0;
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += (int64_t)gridDim.x * blockDim.x) {
        const double yq = y[q] * inv_mult(mult[q]);
#pragma unroll
        for (int i = 0; i < L; ++i) acc[i] += ld_stream(V.v[i] + q) * yq;
        if (NORM) acc[L] += x[q] * yq;
    }
    block_reduce_store<NV>(acc, partial, NV);
}

// Workgroup i: the sum of partial[b * nv + i] over b in a fixed order; a
// coefficient is that times 1 / |V_i|_A^2, the others stand as they are
__global__ __launch_bounds__(256) void proj_reduce_kernel(const double *__restrict__ partial, int64_t blocks, int nv,
                                                          int L, int first, int extra, ProjScales sc,
                                                          double *__restrict__ coef)
{
    __shared__ double red[256];
    const int i = blockIdx.x;
    double s = 0.0;
    for (int64_t b = threadIdx.x; b < blocks; b += blockDim.x) s += partial[b * nv + i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int h = blockDim.x / 2; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) coef[i < L ? first + i : extra] = i < L ? red[0] * sc.s[first + i] * sc.s[first + i] : red[0];
}

// out = sum_i c_i V_i, ADD: on top of what out holds
template <int L, bool ADD>
__global__ __launch_bounds__(256) void proj_combine_kernel(int64_t n, ProjPtrs V, const double *__restrict__ c,
                                                           double *__restrict__ out)
{
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += (int64_t)gridDim.x * blockDim.x) {
        double s = ADD ? out[q] : 0.0;
#pragma unroll
        for (int i = 0; i < L; ++i) s += c[i] * ld_stream(V.v[i] + q);
        out[q] = s;
    }
}

// v = in - sum_i c_i X_i, Av -= sum_i c_i AX_i.
// SCALE: in, Av and the coefficients times unit_scale(n0); SCALE 2: the
// coefficients only (in and Av are scaled already).
// DOTS: partials of X_i . Av; NORM: of v . Av.
template <int L, int SCALE, bool DOTS, bool NORM>
__global__ __launch_bounds__(256) void proj_remove_kernel(int64_t n, ProjPtrs X, ProjPtrs AX,
                                                          const double *__restrict__ c, const double *n0,
                                                          const double *in, double *v, double *__restrict__ Av,
                                                          const uint8_t *__restrict__ mult,
                                                          double *__restrict__ partial)
{
    constexpr int NV = (DOTS ? L : 0) + (NORM ? 1 : 0);
    double acc[NV > 0 ? NV : 1];
#pragma unroll
    for (int i = 0; i < NV; ++i) acc[i] = 0.0;
    const double us = SCALE ? unit_scale(*n0) : 1.0;
    double cs[L > 0 ? L : 1];
#pragma unroll
    for (int i = 0; i < L; ++i) cs[i] = c[i] * us;
    for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < n; q += (int64_t)gridDim.x * blockDim.x) {
        double a = in[q], b = Av[q], xv[L > 0 ? L : 1];
        if (SCALE == 1) {
            a *= us;
            b *= us;
        }
#pragma unroll
        for (int i = 0; i < L; ++i) {
            xv[i] = ld_stream(X.v[i] + q);
            a -= cs[i] * xv[i];
            b -= cs[i] * ld_stream(AX.v[i] + q);
        }
        v[q] = a;
        Av[q] = b;
        if (NV > 0) {
            const double bm = b * inv_mult(mult[q]);
            if (DOTS) {
#pragma unroll
                for (int i = 0; i < L; ++i) acc[i] += xv[i] * bm;
            }
            if (NORM) acc[NV - 1] += a * bm;
        }
    }
    if constexpr (NV > 0) block_reduce_store<NV>(acc, partial, NV);
}

template <typename F>
static sem_status pguard(F &&f)
{
    try {
        return f();
    } catch (const Failure &x) {
        return x.status;
    } catch (const std::bad_alloc &) {
        set_error("host allocation failed");
        return SEM_ENOMEM;
    } catch (const std::exception &x) {
        set_error(x.what());
        return SEM_EINVAL;
    } catch (...) {
        set_error("unknown internal error");
        return SEM_EINVAL;
    }
}

}  // namespace sem

struct sem_proj {
    sem_mesh *mesh = nullptr;
    int max_vectors = 0;
    int l = 0;                  // basis vectors held
    int op_version = 0;         // operator the basis was built for
    double drop_tol = 1e-8;
    std::vector<double *> X, AX;  // of any length; the unit vectors are scale[i] X_i
    double scale[sem::kMaxProj];  // 1 / |X_i|_A
    double *coef = nullptr;       // [kCoefSize]
    double *partial = nullptr;    // [blocks * (kProjPass + 1)]
    int64_t blocks = 0;
};

namespace sem {

static ProjPtrs ptrs(const std::vector<double *> &v, int first, int count)
{
    ProjPtrs p{};
    for (int i = 0; i < count; ++i) p.v[i] = v[first + i];
    return p;
}

// f(std::integral_constant<int, L>) for the count L of a launch
template <typename F>
static void with_count(int L, F &&f)
{
    switch (L) {
    case 0: return f(std::integral_constant<int, 0>());
    case 1: return f(std::integral_constant<int, 1>());
    case 2: return f(std::integral_constant<int, 2>());
    case 3: return f(std::integral_constant<int, 3>());
    case 4: return f(std::integral_constant<int, 4>());
    case 5: return f(std::integral_constant<int, 5>());
    case 6: return f(std::integral_constant<int, 6>());
    case 7: return f(std::integral_constant<int, 7>());
    default: return f(std::integral_constant<int, kProjPass>());
    }
}

static void sync_version(sem_proj *P)
{
    if (P->op_version != P->mesh->op_version) {
        P->l = 0;
        P->op_version = P->mesh->op_version;
    }
}

static void reduce(sem_proj *P, int nv, int L, int first, int extra, hipStream_t s)
{
    ProjScales sc{};
    for (int i = 0; i < P->l; ++i) sc.s[i] = P->scale[i];
    hipLaunchKernelGGL(proj_reduce_kernel, dim3(nv), dim3(256), 0, s, P->partial, P->blocks, nv, L, first, extra, sc,
                       P->coef);
    SEM_HIP(hipGetLastError());
}

// coefficients of all vectors for y; x: also coef[kCoefN0] = x . y
static void dots(sem_proj *P, const double *y, const double *x, hipStream_t s)
{
    const int64_t n = P->mesh->h.nL;
    for (int first = 0; first < P->l || (first == 0 && x); first += kProjPass) {
        const int L = std::min(P->l - first, kProjPass);
        const bool norm = first == 0 && x;
        with_count(L, [&](auto count) {
            constexpr int K = decltype(count)::value;
            if (norm)
                hipLaunchKernelGGL((proj_dots_kernel<K, true>), dim3((unsigned)P->blocks), dim3(256), 0, s, n,
                                   ptrs(P->X, first, L), y, x, P->mesh->mult, P->partial);
            else if constexpr (K > 0)
                hipLaunchKernelGGL((proj_dots_kernel<K, false>), dim3((unsigned)P->blocks), dim3(256), 0, s, n,
                                   ptrs(P->X, first, L), y, x, P->mesh->mult, P->partial);
        });
        SEM_HIP(hipGetLastError());
        reduce(P, L + (norm ? 1 : 0), L, first, kCoefN0, s);
    }
}

static void project(sem_proj *P, const double *b, double *x, hipStream_t s)
{
    const int64_t n = P->mesh->h.nL;
    if (P->l == 0) {
        SEM_HIP(hipMemsetAsync(x, 0, sizeof(double) * n, s));
        return;
    }
    dots(P, b, nullptr, s);
    for (int first = 0; first < P->l; first += kProjPass) {
        const int L = std::min(P->l - first, kProjPass);
        with_count(L, [&](auto count) {
            constexpr int K = decltype(count)::value;
            if (first == 0)
                hipLaunchKernelGGL((proj_combine_kernel<K, false>), dim3(vec_blocks(n)), dim3(256), 0, s, n,
                                   ptrs(P->X, first, L), P->coef + first, x);
            else
                hipLaunchKernelGGL((proj_combine_kernel<K, true>), dim3(vec_blocks(n)), dim3(256), 0, s, n,
                                   ptrs(P->X, first, L), P->coef + first, x);
        });
        SEM_HIP(hipGetLastError());
    }
}

template <int SCALE, bool DOTS, bool NORM>
static void remove_pass(sem_proj *P, int first, int L, const double *in, double *v, double *Av, hipStream_t s)
{
    with_count(L, [&](auto count) {
        constexpr int K = decltype(count)::value;
        hipLaunchKernelGGL((proj_remove_kernel<K, SCALE, DOTS, NORM>), dim3((unsigned)P->blocks), dim3(256), 0, s,
                           P->mesh->h.nL, ptrs(P->X, first, L), ptrs(P->AX, first, L), P->coef + first,
                           P->coef + kCoefN0, in, v, Av, P->mesh->mult, P->partial);
    });
    SEM_HIP(hipGetLastError());
}

// returns 1 when x joined the basis, 0 when it was dropped
static int add(sem_proj *P, const double *x, hipStream_t s)
{
    sem_mesh *m = P->mesh;
    if (P->l >= P->max_vectors) P->l = 0;
    const int l = P->l;
    double *v = P->X[l], *Av = P->AX[l];
    const sem_status st = sem_axgs(m, SEM_FP64, x, Av, s);
    if (st != SEM_OK) fail(st, "sem_proj_add: operator apply failed");
    dots(P, Av, x, s);
    if (l <= kProjPass) {
        if (l == 0) {
            remove_pass<1, false, false>(P, 0, 0, x, v, Av, s);
        } else {
            remove_pass<1, true, false>(P, 0, l, x, v, Av, s);
            reduce(P, l, l, 0, 0, s);
            remove_pass<0, false, true>(P, 0, l, v, v, Av, s);
            reduce(P, 1, 0, 0, kCoefN2, s);
        }
    } else {
        remove_pass<1, false, false>(P, 0, kProjPass, x, v, Av, s);
        for (int first = kProjPass; first < l; first += kProjPass)
            remove_pass<2, false, false>(P, first, std::min(l - first, kProjPass), v, v, Av, s);
        dots(P, Av, nullptr, s);
        int first = 0;
        for (; first + kProjPass < l; first += kProjPass) remove_pass<0, false, false>(P, first, kProjPass, v, v, Av, s);
        remove_pass<0, false, true>(P, first, l - first, v, v, Av, s);
        reduce(P, 1, 0, 0, kCoefN2, s);
    }
    double nn[2];  // x . A x, v . A v
    SEM_HIP(hipMemcpyAsync(nn, P->coef + kCoefN0, sizeof(nn), hipMemcpyDeviceToHost, s));
    SEM_HIP(hipStreamSynchronize(s));
    if (!(nn[0] > 0.0) || !std::isfinite(nn[0])) return 0;
    const double us = unit_scale(nn[0]), n0 = nn[0] * us * us, n2 = l == 0 ? n0 : nn[1];
    if (!(n2 > P->drop_tol * P->drop_tol * n0)) return 0;
    P->scale[l] = 1.0 / std::sqrt(n2);
    P->l = l + 1;
    return 1;
}

}  // namespace sem

using namespace sem;

extern "C" {

sem_status sem_proj_create(sem_mesh *mesh, int max_vectors, sem_proj **out)
{
    return pguard([&]() -> sem_status {
        if (!mesh || !out) fail(SEM_EINVAL, "sem_proj_create: null argument");
        if (max_vectors < 1 || max_vectors > kMaxProj) fail(SEM_EINVAL, "sem_proj_create: max_vectors must be 1..32");
        *out = nullptr;
        sem_proj *P = new sem_proj();
        P->mesh = mesh;
        P->max_vectors = max_vectors;
        P->op_version = mesh->op_version;
        const int64_t n = mesh->h.nL;
        P->blocks = std::min(vec_blocks(n), kProjBlocks);
        auto alloc = [&](size_t bytes) {
            void *p = nullptr;
            if (hipMalloc(&p, std::max<size_t>(bytes, 16)) != hipSuccess) {
                (void)hipGetLastError();
                return (double *)nullptr;
            }
            return (double *)p;
        };
        bool ok = true;
        for (int i = 0; i < max_vectors && ok; ++i) {
            double *a = alloc(sizeof(double) * n), *b = alloc(sizeof(double) * n);
            if (a) P->X.push_back(a);
            if (b) P->AX.push_back(b);
            ok = a && b;
        }
        if (ok) ok = (P->coef = alloc(sizeof(double) * kCoefSize)) != nullptr;
        if (ok) ok = (P->partial = alloc(sizeof(double) * (size_t)P->blocks * (kProjPass + 1))) != nullptr;
        if (!ok) {
            sem_proj_free(P);
            fail(SEM_ENOMEM, "sem_proj_create: device allocation failed");
        }
        *out = P;
        return SEM_OK;
    });
}

sem_status sem_proj_free(sem_proj *P)
{
    if (!P) return SEM_OK;
    for (double *p : P->X) hipFree(p);
    for (double *p : P->AX) hipFree(p);
    if (P->coef) hipFree(P->coef);
    if (P->partial) hipFree(P->partial);
    delete P;
    return SEM_OK;
}

sem_status sem_proj_reset(sem_proj *P)
{
    return pguard([&]() -> sem_status {
        if (!P) fail(SEM_EINVAL, "sem_proj_reset: null handle");
        P->l = 0;
        return SEM_OK;
    });
}

sem_status sem_proj_size(sem_proj *P, int *n)
{
    return pguard([&]() -> sem_status {
        if (!P || !n) fail(SEM_EINVAL, "sem_proj_size: null argument");
        sync_version(P);
        *n = P->l;
        return SEM_OK;
    });
}

sem_status sem_proj_project(sem_proj *P, const double *b, double *x, void *stream)
{
    return pguard([&]() -> sem_status {
        if (!P || !b || !x) fail(SEM_EINVAL, "sem_proj_project: null argument");
        sync_version(P);
        project(P, b, x, (hipStream_t)stream);
        return SEM_OK;
    });
}

sem_status sem_proj_add(sem_proj *P, const double *x, int *added, void *stream)
{
    return pguard([&]() -> sem_status {
        if (!P || !x) fail(SEM_EINVAL, "sem_proj_add: null argument");
        sync_version(P);
        const int a = add(P, x, (hipStream_t)stream);
        if (added) *added = a;
        return SEM_OK;
    });
}

sem_status sem_proj_solve(sem_proj *P, const double *b, double *x, const sem_solve_opts *opts, sem_solve_stats *stats,
                          void *stream)
{
    return pguard([&]() -> sem_status {
        if (!P || !b || !x) fail(SEM_EINVAL, "sem_proj_solve: null argument");
        hipStream_t s = (hipStream_t)stream;
        sync_version(P);
        sem_solve_opts o;
        sem_solve_opts_default(&o);
        if (opts) o = *opts;
        o.x0_given = 1;
        project(P, b, x, s);
        const sem_status st = sem_pcg_solve(P->mesh, b, x, &o, stats, stream);
        if (st == SEM_OK) add(P, x, s);
        return st;
    });
}

}  // extern "C"
