// A HIP runtime without a device, for tests of the library's host side on the
// CPU: device memory is host memory, copies and fills are done, kernels are
// only recorded.  Loaded with global symbols before libsem.so, whose HIP calls
// it answers; an allocation can be made to fail, as on a full device.
#include <algorithm>
#include <chrono>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <thread>
#include <vector>

#include "resident.hpp"

namespace {
struct Launch {
    std::string name;
    unsigned grid, grid_y, block;
    size_t lds;
    int iters;        // resident runs
    bool has_scratch;
    hipStream_t stream;
};
std::map<const void *, std::string> names;
std::set<void *> blocks;
std::vector<Launch> launches;
thread_local hipError_t last = hipSuccess;  // kept until it is read, as the runtime does
int fail_in = -1;              // allocations until one fails
int null_uses = 0;             // copies, fills and kernels given no memory
int verdict = 0;               // what a resident run leaves in its state
int64_t allocated = 0, copied = 0;
double fill = 0.0;             // what new device memory holds
int hold_ms = 0, in_flight = 0, max_in_flight = 0;  // resident runs
std::mutex mu;  // of what follows from launches and allocations

hipError_t put(hipError_t e)
{
    if (e != hipSuccess) last = e;
    return e;
}
template <typename T>
void resident(Launch &l, void **args)
{
    const sem::ResidentParams<T> &a = *static_cast<sem::ResidentParams<T> *>(args[0]);
    l.iters = a.iters;
    l.has_scratch = a.xs && a.words && a.st;
    if (a.st) a.st->pad = verdict;
}
}  // namespace

extern "C" {

// --- the tests' side ---------------------------------------------------------
void fake_fail_in(int n) { fail_in = n; }
void fake_set_verdict(int v) { verdict = v; }
int fake_null_uses() { return null_uses; }
int64_t fake_allocated() { return allocated; }
int64_t fake_copied() { return copied; }
void fake_fill(double v) { fill = v; }
void fake_hold_ms(int ms) { hold_ms = ms; }
int fake_max_in_flight() { return max_in_flight; }
void fake_clear()
{
    launches.clear();
    max_in_flight = 0;
}
int fake_launches() { return (int)launches.size(); }
const char *fake_name(int i) { return launches[i].name.c_str(); }
unsigned fake_grid(int i) { return launches[i].grid; }
unsigned fake_grid_y(int i) { return launches[i].grid_y; }
unsigned fake_block(int i) { return launches[i].block; }
int64_t fake_stream(int i) { return (int64_t)launches[i].stream; }
int fake_iters(int i) { return launches[i].iters; }
int fake_has_scratch(int i) { return launches[i].has_scratch; }

// --- the runtime's side ------------------------------------------------------
void **__hipRegisterFatBinary(const void *)
{
    static void *handle;
    return &handle;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *device, unsigned, void *, void *, void *,
                           void *, int *)
{
    names[host] = device;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}

static thread_local dim3 cfg_grid, cfg_block;
static thread_local size_t cfg_lds;
static thread_local hipStream_t cfg_stream;
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s)
{
    cfg_grid = g;
    cfg_block = b;
    cfg_lds = lds;
    cfg_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, hipStream_t *s)
{
    *g = cfg_grid;
    *b = cfg_block;
    *lds = cfg_lds;
    *s = cfg_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t lds, hipStream_t s)
{
    std::unique_lock<std::mutex> lock(mu);
    Launch l{names[f], g.x, g.y, b.x, lds, 0, false, s};
    if (l.name.find("resident_kernel") != std::string::npos) {
        if (hold_ms) {  // the run takes its time
            max_in_flight = std::max(max_in_flight, ++in_flight);
            lock.unlock();
            std::this_thread::sleep_for(std::chrono::milliseconds(hold_ms));
            lock.lock();
            --in_flight;
        }
        if (l.name.find("resident_kernelId") != std::string::npos) resident<double>(l, args);
        else resident<float>(l, args);
    }
    // kernels of a few pointers: (n, value, out), (n, a, b, out), (n, state, x, p)
    auto given = [&](int k) {
        if (!*static_cast<void **>(args[k])) null_uses++;
    };
    if (l.name.find("fill_kernel") != std::string::npos) given(2);
    if (l.name.find("scale_kernel") != std::string::npos || l.name.find("pcg_finish_kernel") != std::string::npos) {
        given(1);
        given(2);
        given(3);
    }
    launches.push_back(l);
    return hipSuccess;
}

hipError_t hipMalloc(void **p, size_t bytes)
{
    *p = nullptr;
    std::lock_guard<std::mutex> lock(mu);
    if (fail_in >= 0 && fail_in-- == 0) return put(hipErrorOutOfMemory);
    *p = std::malloc(bytes + 8);
    for (size_t q = 0; q < bytes + 8 - 7; q += 8) std::memcpy(static_cast<char *>(*p) + q, &fill, 8);
    blocks.insert(*p);
    allocated += (int64_t)bytes;
    return hipSuccess;
}
hipError_t hipFree(void *p)
{
    std::lock_guard<std::mutex> lock(mu);
    if (p && blocks.erase(p)) std::free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind)
{
    if (n && (!d || !s)) {
        null_uses++;
        return put(hipErrorInvalidValue);
    }
    std::memcpy(d, s, n);
    copied += (int64_t)n;
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t) { return hipMemcpy(d, s, n, k); }
hipError_t hipMemset(void *d, int v, size_t n)
{
    if (n && !d) {
        null_uses++;
        return put(hipErrorInvalidValue);
    }
    std::memset(d, v, n);
    return hipSuccess;
}
hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t) { return hipMemset(d, v, n); }
hipError_t hipMemcpyToSymbolAsync(const void *, const void *, size_t, size_t, hipMemcpyKind, hipStream_t) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *)
{
    static double room[1 << 15];
    *p = room;
    return hipSuccess;
}

hipError_t hipGetDevice(int *d)
{
    *d = 0;
    return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int)
{
    std::memset(p, 0, sizeof(*p));
    std::strcpy(p->gcnArchName, "gfx950");
    return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int)
{
    *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : (a == hipDeviceAttributeMaxSharedMemoryPerBlock ? 163840 : 0);
    return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t)
{
    *n = 1;
    return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetLastError()
{
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}
const char *hipGetErrorString(hipError_t) { return "error"; }

hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned)
{
    static char many[1024];
    static int next = 0;
    *s = reinterpret_cast<hipStream_t>(many + next++ % 1024);
    return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g)
{
    *g = nullptr;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t)
{
    *e = nullptr;
    return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e)
{
    *e = nullptr;
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t)
{
    *ms = 0.0f;
    return hipSuccess;
}

}  // extern "C"
