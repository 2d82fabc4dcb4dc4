// resident.hip -- Jacobi-PCG of a small mesh in one launch.
//
// A mesh of a few hundred elements moves so little per iteration that its CG
// is bound by launches and by the latency of the memory chains in each
// kernel: four launches and about 33 us an iteration for 64 elements of order
// 7.  Here one workgroup per compute unit owns a few elements for the whole
// run: factors in LDS where they fit, r, p and the Jacobi diagonal in registers,
// x in scratch memory, and per iteration only the face values of w = A p and
// three scalars travel between workgroups.
//
//  * The two reductions of an iteration are also its grid barriers.  A
//    workgroup publishes its partial sum as words that carry the iteration's
//    tag beside 32 bits of payload each; everyone polls the words of every
//    workgroup and, once all tags match, holds all the partials, which it sums
//    in a fixed order (the same bits everywhere).  No atomics on shared
//    counters, one trip to memory per reduction.
//  * w is stored before <p, A p> is published, and read after all the words
//    have arrived, with device-scope accesses (the L2 caches of the XCDs are
//    not coherent with each other otherwise).
//  * The arithmetic of a node is that of the operator tile and of the update
//    with the gather-scatter folded in (copies summed from 0 in ascending
//    local index), so only the order of the dot products' partial sums differs.
//  * Every wait is bounded by a clock: if the workgroups do not meet (other
//    work holds the compute units), the run is called off and nothing is
//    written; whether it stands is decided by one compare-and-swap.
#include "resident.hpp"

#include "kernels.hpp"
#include "operator.hpp"

namespace sem {

template <typename T>
__device__ inline T ld_dev(const T *p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T>
__device__ inline void st_dev(T *p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

__device__ inline double read_lane(double s, int lane)
{
    const long long b = __double_as_longlong(s);
    const int lo = __builtin_amdgcn_readlane((int)b, lane), hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
// Sum over the wavefront, the same bits in every lane.  Within rows of 16
// lanes through DPP moves and across the rows through scalar reads: a fifth of
// the latency of six cross-lane shuffles through LDS, and it is paid four
// times per iteration.
__device__ inline double wave_total(double s)
{
    s = dpp_add<0x140>(sum8(s));  // row_mirror
    return (read_lane(s, 0) + read_lane(s, 16)) + (read_lane(s, 32) + read_lane(s, 48));
}

// Partial sums v of this workgroup in, their totals over all workgroups out;
// the device-scope stores of every lane are visible to all before anyone
// returns.  False when the run is called off.  words: 2 NV per workgroup.
template <int NV>
__device__ inline bool exchange(double (&v)[NV], uint64_t *words, int nwg, uint32_t tag, uint64_t wait_ticks,
                                PcgState *st)
{
    __shared__ double red[NV][16], total[NV];
    __shared__ int meet;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwave = (blockDim.x + 63) >> 6;
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        const double s = wave_total(v[q]);
        if (lane == 0) red[q][wave] = s;
    }
    // this wave's stores of w have reached memory before its workgroup
    // publishes (everything that travels does so with device-scope accesses, so
    // no cache has to be written back or invalidated)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (wave == 0) {
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            double s = 0.0;
            for (int w = 0; w < nwave; ++w) s += red[q][w];
            const uint64_t b = (uint64_t)__double_as_longlong(s), t = (uint64_t)tag << 32;
            if (lane < 2) st_dev(words + ((size_t)blockIdx.x * NV + q) * 2 + lane, t | (lane ? b >> 32 : b & 0xffffffffu));
        }
        // lane's workgroups: lane, lane + 64, ... (all their words in flight together)
        constexpr int K = kResidentMaxWg / 64;
        uint64_t got[K][NV][2];
        const uint64_t t0 = wall_clock64();
        int ok = 1;
        for (;;) {
            bool all = true;
#pragma unroll
            for (int k = 0; k < K; ++k)
                if (lane + 64 * k < nwg)
#pragma unroll
                    for (int q = 0; q < NV; ++q)
#pragma unroll
                        for (int h = 0; h < 2; ++h)
                            got[k][q][h] = ld_dev(words + ((size_t)(lane + 64 * k) * NV + q) * 2 + h);
#pragma unroll
            for (int k = 0; k < K; ++k)
                if (lane + 64 * k < nwg)
#pragma unroll
                    for (int q = 0; q < NV; ++q)
                        all = all && (uint32_t)(got[k][q][0] >> 32) == tag && (uint32_t)(got[k][q][1] >> 32) == tag;
            if (__all(all)) break;
            if (wall_clock64() - t0 > wait_ticks) {
                // call the run off, unless some workgroup has completed it (then
                // all have published and the words are on their way)
                int was = 0;
                if (lane == 0) was = atomicCAS(&st->pad, 0, 2);
                if (__shfl(was, 0, 64) != 1) {
                    ok = 0;
                    break;
                }
            }
            __builtin_amdgcn_s_sleep(1);
        }
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            double s = 0.0;
#pragma unroll
            for (int k = 0; k < K; ++k)
                if (lane + 64 * k < nwg && ok)
                    s += __longlong_as_double((long long)((got[k][q][1] << 32) | (got[k][q][0] & 0xffffffffu)));
            s = wave_total(s);
            if (lane == 0) total[q] = s;
        }
        if (lane == 0) meet = ok;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NV; ++q) v[q] = total[q];
    return meet != 0;
}

// Keeps the compiler from carrying what follows from v through the iteration
// loop: hoisted, the addresses, masks and matrix entries of a column would
// take several hundred registers.
template <typename X>
__device__ inline X fresh_v(X v)
{
    asm volatile("" : "+v"(v));
    return v;
}
__device__ inline int fresh_s(int v)
{
    asm volatile("" : "+s"(v));
    return v;
}

// lanes of a workgroup, at most: 256 keep the whole register file of a SIMD
// for one wave where the columns are long
template <typename T>
constexpr int resident_threads(int N) { return (N + 1) * (int)sizeof(T) >= 64 ? 256 : 512; }

// GL: the factors stay in LDS; else they are read from the caches every
// iteration, one plane ahead (twice the elements per compute unit).
template <typename T, int N, bool GL>
__global__ __launch_bounds__(GL ? resident_threads<T>(N) : 512) void resident_kernel(ResidentParams<T> a)
{
    constexpr int P = N + 1, P2 = P * P, P3 = P2 * P;
    // planes whose loads may be moved ahead of each other's products (more of
    // them spill registers)
    constexpr int kAhead = P * sizeof(T) <= 64 ? 2 : 1;
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ T sD[P2];
    __shared__ int stands;
    if (a.st->done) {
        if (blockIdx.x == 0 && threadIdx.x == 0) a.st->pad = 1;
        return;
    }
    const int tid = threadIdx.x;
    const int el = tid / P2, ij = tid - el * P2;
    const int i = ij % P, j = ij / P;
    const bool inblk = el < a.epw;
    const int slot = inblk ? el : a.epw - 1;  // padding lanes read a valid slot
    const int64_t e = (int64_t)blockIdx.x * a.epw + el;
    const bool active = inblk && e < a.E;
    const int lanes = a.epw * P2;
    T *su = reinterpret_cast<T *>(smem_raw) + (size_t)slot * 3 * P3;
    T *sr = su + P3, *ss = sr + P3;
    T *sG = reinterpret_cast<T *>(smem_raw) + (size_t)a.epw * 3 * P3 + (inblk ? tid : 0);  // [6 P][lanes], lane's own
    for (int q = tid; q < P2; q += blockDim.x) sD[q] = dtable<T>(N)[q];

    // this lane's column: r, p and the diagonal in registers, x in scratch
    // (read and written by this lane alone, copied out when the run stands)
    const int o = active ? (int)(e * P3) + ij : 0;
    T r[P], p[P], iv[P], x[P], w[P];
    uint32_t mlog[(P + 9) / 10];  // log2 of the multiplicities, three bits each
#pragma unroll
    for (int q = 0; q < (P + 9) / 10; ++q) mlog[q] = 0;
#pragma unroll
    for (int k = 0; k < P; ++k) {  // an inactive lane reads the first column and works on its own slot
        r[k] = a.r[o + k * P2];
        p[k] = a.p[o + k * P2];
        x[k] = a.x[o + k * P2];
        iv[k] = a.inv[o + k * P2];
        mlog[k / 10] |= (uint32_t)__builtin_ctz(a.mult[o + k * P2]) << (3 * (k % 10));
    }
    const T *g = a.G + (active ? e : 0) * 6 * P3 + ij;
    if (GL && inblk) {
#pragma unroll 6
        for (int q = 0; q < 6 * P; ++q) sG[(size_t)q * lanes] = g[(size_t)q * P2];  // c P + k: factor c, plane k
    }
    // copies of the column's nodes, as the update with the gather-scatter
    // folded in finds them: fixed for the run.  Bits 0-3: the x, y copies
    // there are; 4: the column lies on a Dirichlet face; 5: it has neighbours;
    // per z face (low 8-, high 12-): masked, two copies, own copy first.
    int flags = 0, dxy[4] = {0, 0, 0, 0}, olo = 0, ohi = 0;
    if (active) {
        const int nx = a.L.nel[0], ny = a.L.nel[1], ei = (int)e;
        const ElemAxis ax = elem_axis<N>(ei % nx, nx, a.L.periodic[0], a.L.faces & 1, a.L.faces & 2);
        const ElemAxis ay = elem_axis<N>((ei / nx) % ny, ny, a.L.periodic[1], a.L.faces & 4, a.L.faces & 8);
        const ElemAxis az = elem_axis<N>(ei / (nx * ny), a.L.nel[2], a.L.periodic[2], a.L.faces & 16, a.L.faces & 32);
        const LaneAxis cx = lane_axis<N>(ax, i, P3, 1), cy = lane_axis<N>(ay, j, nx * P3, P);
        const LaneAxis zlo = lane_axis<N>(az, 0, nx * ny * P3, P2), zhi = lane_axis<N>(az, N, nx * ny * P3, P2);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if ((q & 1) < cx.c && (q >> 1) < cy.c) flags |= 1 << q;
            dxy[q] = cx.d[q & 1] + cy.d[q >> 1];
        }
        const bool wall = cx.masked || cy.masked;
        flags |= (wall ? 16 : 0) | (!wall && cx.c * cy.c > 1 ? 32 : 0);
        if (!wall) flags |= (zlo.masked ? 256 : 0) | (zlo.c > 1 ? 512 : 0) | (zlo.d[0] == 0 ? 1024 : 0);
        if (!wall) flags |= (zhi.masked ? 4096 : 0) | (zhi.c > 1 ? 8192 : 0) | (zhi.d[0] == 0 ? 16384 : 0);
        // of the two z copies of a face node the one that is not the column's own
        olo = zlo.d[0] != 0 ? zlo.d[0] : zlo.d[1];
        ohi = N * P2 + (zhi.d[0] != 0 ? zhi.d[0] : zhi.d[1]);
    }

    double rho = a.st->rho, rr = a.st->rr, sigma = a.st->sigma, rho_new = a.st->rho_new;
    double alpha = a.st->alpha, beta = a.st->beta;
    const double stop2 = a.st->stop2;
    int iters = a.st->iters, done = 0;
    const int limit = a.st->limit;
    __syncthreads();  // sD

    for (int it = 1; it <= a.iters && !done; ++it) {
        const uint32_t tag = a.seq + (uint32_t)it;
        const int ov = fresh_v(o), fl = fresh_v(flags);
        // the deferred x step and the new search direction
        {
            const T al = (T)alpha, be = (T)beta;
#pragma unroll
            for (int k = 0; k < P; ++k) {
                x[k] = x[k] + al * p[k];
                p[k] = iv[k] * r[k] + be * p[k];
            }
            if (inblk) {
#pragma unroll
                for (int k = 0; k < P; ++k) su[k * P2 + ij] = p[k];
            }
            if (active) {
#pragma unroll
                for (int k = 0; k < P; ++k) a.xs[ov + k * P2] = x[k];
            }
        }
        T gn[6];
        const int gv = fresh_v(0);
        if (!GL) {
#pragma unroll
            for (int c = 0; c < 6; ++c) gn[c] = g[gv + c * P3];
        }
        __syncthreads();
        // w = A_L p: the arithmetic of the operator tile
        T wt[P];
        {
            T di[P], dj[P];
#pragma unroll
            for (int l = 0; l < P; ++l) {
                di[l] = sD[i * P + l];
                dj[l] = sD[j * P + l];
            }
#pragma unroll
            for (int k = 0; k < P; ++k) {
                const T *__restrict__ Dk = dtable<T>(N) + fresh_s(k * P);  // scalar loads, plane by plane
                T ur = 0, us = 0, ut = 0;
#pragma unroll
                for (int l = 0; l < P; ++l) {
                    ur += di[l] * su[k * P2 + j * P + l];
                    us += dj[l] * su[k * P2 + l * P + i];
                    ut += Dk[l] * p[l];
                }
                T gk[6];
#pragma unroll
                for (int c = 0; c < 6; ++c) {
                    gk[c] = GL ? sG[(size_t)(c * P + k) * lanes] : gn[c];
                    if (!GL && k + 1 < P) gn[c] = g[gv + c * P3 + (k + 1) * P2];
                }
                const T g1 = gk[0], g2 = gk[1], g3 = gk[2], g4 = gk[3], g5 = gk[4], g6 = gk[5];
                const T wr = g1 * ur + g4 * us + g5 * ut;
                const T ws = g2 * us + g4 * ur + g6 * ut;
                wt[k] = g3 * ut + g5 * ur + g6 * us;
                if (inblk) {
                    sr[k * P2 + ij] = wr;
                    ss[k * P2 + ij] = ws;
                }
                if (k % kAhead == kAhead - 1) __builtin_amdgcn_sched_barrier(0);
            }
        }
        __syncthreads();
        {
            T di[P], dj[P];
#pragma unroll
            for (int l = 0; l < P; ++l) {
                di[l] = sD[l * P + i];
                dj[l] = sD[l * P + j];
            }
            if constexpr (plane_tile<T, N, 2>()) {
                // in the order of the plane-by-plane tile
#pragma unroll
                for (int k = 0; k < P; ++k) w[k] = T(0);
#pragma unroll
                for (int k = 0; k < P; ++k) {
                    const T *__restrict__ Dk = dtable<T>(N) + fresh_s(k * P);
                    T b = 0;
#pragma unroll
                    for (int l = 0; l < P; ++l) b += di[l] * sr[k * P2 + j * P + l] + dj[l] * ss[k * P2 + l * P + i];
#pragma unroll
                    for (int kk = 0; kk < P; ++kk) w[kk] += Dk[kk] * wt[k] + (kk == k ? b : T(0));
                    if (k % kAhead == kAhead - 1) __builtin_amdgcn_sched_barrier(0);
                }
            } else {
#pragma unroll
                for (int k = 0; k < P; ++k) {
                    const T *__restrict__ Dk = dtable<T>(N) + fresh_s(k);
                    T acc = 0;
#pragma unroll
                    for (int l = 0; l < P; ++l)
                        acc += di[l] * sr[k * P2 + j * P + l] + dj[l] * ss[k * P2 + l * P + i] + Dk[l * P] * wt[l];
                    w[k] = acc;
                    if (k % kAhead == kAhead - 1) __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        double dot[1] = {0.0};
        if (active) {
            st_dev(a.w + ov, w[0]);
            st_dev(a.w + ov + N * P2, w[N]);
            if (fl & 32) {
#pragma unroll
                for (int k = 1; k < N; ++k) st_dev(a.w + ov + k * P2, w[k]);
            }
#pragma unroll
            for (int k = 0; k < P; ++k) dot[0] += (double)p[k] * (double)w[k];
        }
        if (!exchange<1>(dot, a.words, a.nwg, tag, a.wait_ticks, a.st)) return;
        sigma = dot[0];
        if (!(sigma > 0.0) || !isfinite(sigma)) {
            done = 2;
            break;
        }
        alpha = rho / sigma;
        __builtin_amdgcn_sched_barrier(0);
        // r -= alpha w, w summed over its copies; every load of the column first
        T lay[P][4], far[2][4];
        const bool side = fl & 32;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
#pragma unroll
            for (int k = 0; k < P; ++k) lay[k][q] = q == 0 ? w[k] : T(0);
            far[0][q] = far[1][q] = T(0);
            if (fl & (1 << q)) {
                const int oq = ov + dxy[q];
                if (side) {
#pragma unroll
                    for (int k = 0; k < P; ++k) lay[k][q] = ld_dev(a.w + oq + k * P2);
                }
                if (fl & 512) far[0][q] = ld_dev(a.w + oq + olo);
                if (fl & 8192) far[1][q] = ld_dev(a.w + oq + ohi);
            }
        }
        // the copies of a layer, added to s in ascending local index
        auto add = [&](T s, const T (&v)[4]) {
            s = s + v[0];
            if (fl & 2) s = s + v[1];
            if (fl & 4) s = s + v[2];
            if (fl & 8) s = s + v[3];
            return s;
        };
        if (side) {
#pragma unroll
            for (int k = 0; k < P; ++k) w[k] = add(T(0), lay[k]);
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int k = h == 0 ? 0 : N, zf = h == 0 ? fl >> 8 : fl >> 12;  // masked, two copies, own copy first
            if (zf & 2) w[k] = (zf & 4) ? add(add(T(0), lay[k]), far[h]) : add(add(T(0), far[h]), lay[k]);
            if (zf & 1) w[k] = T(0);
        }
        const T al = (T)alpha;
        double s2[2] = {0.0, 0.0};
#pragma unroll
        for (int k = 0; k < P; ++k) {
            r[k] = r[k] - al * ((fl & 16) ? T(0) : w[k]);
            // 1/mult, a power of two
            const int m3 = (int)(mlog[k / 10] >> (3 * (k % 10))) & 7;
            const double im = __longlong_as_double((long long)(1023 - m3) << 52);
            const double rd = (double)r[k];
            s2[0] += rd * rd * im;
            s2[1] += rd * (double)(iv[k] * r[k]) * im;
        }
        if (!active) s2[0] = s2[1] = 0.0;
        __builtin_amdgcn_sched_barrier(0);
        // x for the next step, on its way while the partial sums travel
#pragma unroll
        for (int k = 0; k < P; ++k) x[k] = a.xs[ov + k * P2];
        if (!exchange<2>(s2, a.words + 2 * kResidentMaxWg, a.nwg, tag, a.wait_ticks, a.st)) return;
        iters += 1;
        rr = s2[0];
        rho_new = s2[1];
        beta = s2[1] / rho;
        rho = s2[1];
        if (rr <= stop2) done = 1;
        else if (!isfinite(rr)) done = 2;
        else if (iters >= limit) done = 3;
    }
    // all workgroups are past the last exchange: the run stands unless one of
    // them has called it off
    if (tid == 0) stands = atomicCAS(&a.st->pad, 0, 1) != 2;
    __syncthreads();
    if (!stands) return;
    if (active)
#pragma unroll
        for (int k = 0; k < P; ++k) {
            a.r[o + k * P2] = r[k];
            a.p[o + k * P2] = p[k];
            a.x[o + k * P2] = x[k];
        }
    if (blockIdx.x == 0 && tid == 0) {
        a.st->rho = rho;
        a.st->rho_new = rho_new;
        a.st->sigma = sigma;
        a.st->alpha = alpha;
        a.st->beta = beta;
        a.st->rr = rr;
        a.st->iters = iters;
        a.st->done = done;
    }
}

bool resident_shape(int N, int64_t E, size_t value_bytes, int cus, size_t lds_cap, ResidentShape &s)
{
    if (N < 3 || N > 10 || E < 1) return false;
    const int P2 = (N + 1) * (N + 1), P3 = P2 * (N + 1);
    const int64_t wgs = cus < kResidentMaxWg ? cus : kResidentMaxWg;
    const int64_t epw = (E + wgs - 1) / wgs;
    const int cap = value_bytes == 8 ? resident_threads<double>(N) : resident_threads<float>(N);
    const size_t room = lds_cap > 4096 ? lds_cap - 4096 : 0;  // static LDS of the kernel
    const size_t with_g = (size_t)epw * 9 * P3 * value_bytes, without = (size_t)epw * 3 * P3 * value_bytes;
    s.g_in_lds = epw * P2 <= cap && with_g <= room;
    if (!s.g_in_lds && (epw * P2 > 512 || without > room)) return false;
    s.epw = (int)epw;
    s.nwg = (int)((E + epw - 1) / epw);
    s.threads = (int)((epw * P2 + 63) / 64 * 64);
    s.lds = s.g_in_lds ? with_g : without;
    // A launch holds its compute units to its end, and other runs wait for
    // them: below 10 ms at the measured 12 to 19 us an iteration with the
    // factors on chip, and where they are read at 17 to 19 (up to 128 KB a
    // workgroup), 25 to 34 (up to 200 KB) and 45 to 64 us.
    const size_t reads = s.g_in_lds ? 0 : (size_t)epw * 6 * P3 * value_bytes;
    s.iters = reads <= 128 * 1024 ? kResidentMaxIters : (reads <= 200 * 1024 ? 256 : 128);
    return true;
}

template <typename T>
hipError_t launch_resident(int N, const ResidentShape &s, const ResidentParams<T> &a, hipStream_t stream)
{
    if (s.nwg < 1 || s.nwg > kResidentMaxWg || a.nwg != s.nwg || a.epw != s.epw || (int64_t)s.nwg * s.epw < a.E)
        return hipErrorInvalidValue;
    switch (N) {
#define SEM_RES_CASE(n)                                                                                        \
    case n:                                                                                                    \
        if (s.g_in_lds)                                                                                        \
            hipLaunchKernelGGL((resident_kernel<T, n, true>), dim3((unsigned)s.nwg), dim3(s.threads), s.lds,    \
                               stream, a);                                                                     \
        else                                                                                                   \
            hipLaunchKernelGGL((resident_kernel<T, n, false>), dim3((unsigned)s.nwg), dim3(s.threads), s.lds,   \
                               stream, a);                                                                     \
        break;
        SEM_RES_CASE(3) SEM_RES_CASE(4) SEM_RES_CASE(5) SEM_RES_CASE(6) SEM_RES_CASE(7) SEM_RES_CASE(8)
        SEM_RES_CASE(9) SEM_RES_CASE(10)
#undef SEM_RES_CASE
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}
template hipError_t launch_resident<double>(int, const ResidentShape &, const ResidentParams<double> &, hipStream_t);
template hipError_t launch_resident<float>(int, const ResidentShape &, const ResidentParams<float> &, hipStream_t);

hipError_t upload_resident_dtables(const double *d64, const float *d32, hipStream_t s)
{
    hipError_t e = hipMemcpyToSymbolAsync(HIP_SYMBOL(c_D64), d64, sizeof(double) * kDTableSize, 0,
                                          hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return e;
    return hipMemcpyToSymbolAsync(HIP_SYMBOL(c_D32), d32, sizeof(float) * kDTableSize, 0, hipMemcpyHostToDevice, s);
}

}  // namespace sem
