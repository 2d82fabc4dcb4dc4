// resident.hpp -- CG iterations of a small mesh in one launch (resident.hip):
// every element's factors and vectors stay on chip for the whole run.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "sem_internal.hpp"

namespace sem {

constexpr int kResidentMaxWg = 256;  // workgroups of a resident run, at most
// tagged words the workgroups exchange: two per workgroup for <p, A p>, four
// for <r, r> and <r, z>
constexpr int kResidentWords = 6 * kResidentMaxWg;
constexpr int kResidentMaxIters = 512;  // iterations of a launch, at most

struct ResidentShape {
    int epw = 0;      // elements per workgroup (one workgroup per compute unit)
    int nwg = 0;      // workgroups
    int threads = 0;
    size_t lds = 0;   // dynamic LDS bytes
    bool g_in_lds = false;  // the factors stay in LDS, else they are read every iteration
    int iters = 0;          // iterations of one launch, at most
};

template <typename T>
struct ResidentParams {
    GsLattice L;
    int64_t E;
    int epw, nwg;
    const T *G, *inv;
    const uint8_t *mult;
    T *r, *p, *x, *w;
    T *xs;                // scratch for x during the run (E (N+1)^3 values)
    PcgState *st;
    uint64_t *words;      // kResidentWords
    uint32_t seq;         // tags seq + 1 .. seq + iters are unused so far
    int iters;            // iterations of this launch, at most
    uint64_t wait_ticks;  // longest wait for the other workgroups (100 MHz clock)
};

// The shape of a resident run, false when the mesh does not fit on the chip
// or the order has no kernel (3..10).  cus, lds_cap: compute units and LDS of
// a workgroup of the device.
bool resident_shape(int N, int64_t E, size_t value_bytes, int cus, size_t lds_cap, ResidentShape &s);
// Runs up to a.iters CG iterations from the state in *a.st (Jacobi, lattice
// mesh), until convergence, breakdown or the limit.  st->pad must be 0; it is
// 1 afterwards, or 2 when the workgroups did not meet within wait_ticks: then
// neither the vectors nor the state were changed.  (2 beforehand: it stays 2,
// whatever the workgroups do.)
template <typename T>
hipError_t launch_resident(int N, const ResidentShape &s, const ResidentParams<T> &a, hipStream_t stream);
hipError_t upload_resident_dtables(const double *d64, const float *d32, hipStream_t s);

}  // namespace sem
