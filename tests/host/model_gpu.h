// A model of the GPU for CPU checks of the library's host code: the HIP calls
// and kernel launches that pdbm_api.hip and pdbm_serve.hip make, defined here.
// Device memory is host memory; copies and small kernels happen at once; the
// steps of a chunk are in flight until the check lets them end (`tokens`), and
// a synchronisation of their stream, or freeing memory, waits for that.  The
// step launches are listed in `log` while `logging`.
#pragma once

#include <atomic>
#include <chrono>
#include <condition_variable>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <random>
#include <string>
#include <thread>

#include "../../paper_1308_0653_amd/csrc/pdbm_api.hip"
#include "../../paper_1308_0653_amd/csrc/pdbm_serve.hip"

// ---------------------------------------------------------- the model GPU --
namespace {
struct Gpu {
    std::mutex mu;
    std::condition_variable cv;
    long tokens = 1L << 40;  // chunks that may still end
    long launched = 0;       // chunks launched
    void *busy = nullptr;    // stream with a chunk in flight
    void *capturing = nullptr;
    long allocated = 0;
    bool logging = false;
    int copies = 0;
    struct Launch {
        char kernel;  // m, d: one or two steps marched; c: columns; p: patches
        int tiles, steps;
    };
    std::vector<Launch> log;

    void launch(void *st)
    {
        std::lock_guard<std::mutex> g(mu);
        if (st == capturing) return;
        if (busy != st) ++launched;  // several launches of one chunk
        busy = st;
        cv.notify_all();
    }
    void wait(void *st)  // st NULL: every stream
    {
        std::unique_lock<std::mutex> g(mu);
        if (!busy || (st && busy != st)) return;
        cv.wait(g, [&] { return tokens > 0 || !busy; });
        if (busy) --tokens;
        busy = nullptr;
        cv.notify_all();
    }
    void allow(long n)
    {
        std::lock_guard<std::mutex> g(mu);
        tokens = n;
        cv.notify_all();
    }
    // waits (10 s at most) until that many chunks have been launched
    bool reaches(long n)
    {
        std::unique_lock<std::mutex> g(mu);
        return cv.wait_for(g, std::chrono::seconds(10), [&] { return launched >= n; });
    }
} gpu;
int token_of;  // any address stands for a stream, event or graph
void *handle() { return std::malloc(sizeof token_of); }
}  // namespace

extern "C" {
hipError_t hipGetDeviceCount(int *n) { return *n = 1, hipSuccess; }
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600 *p, int)
{
    std::memset(p, 0, sizeof *p);
    std::strcpy(p->gcnArchName, "gfx950");
    return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipMalloc(void **p, size_t n)
{
    *p = std::malloc(n);
    std::lock_guard<std::mutex> g(gpu.mu);
    ++gpu.allocated;
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void *p)
{
    gpu.wait(nullptr);
    std::free(p);
    std::lock_guard<std::mutex> g(gpu.mu);
    --gpu.allocated;
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t)
{
    std::memcpy(d, s, n);
    if (gpu.logging) ++gpu.copies;
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { return *s = (hipStream_t)handle(), hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { return std::free((void *)s), hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { return gpu.wait((void *)s), hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return *e = (hipEvent_t)handle(), hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { return std::free((void *)e), hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t st, hipStreamCaptureStatus *s)
{
    return *s = gpu.capturing == (void *)st ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone, hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) { return gpu.capturing = (void *)s, hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g)
{
    gpu.capturing = nullptr;
    return *g = (hipGraph_t)handle(), hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t)
{
    return *e = (hipGraphExec_t)handle(), hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t s) { return gpu.launch((void *)s), hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t g) { return std::free((void *)g), hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t e) { return std::free((void *)e), hipSuccess; }
}

namespace pdbm {
#define STEPS(kernel, tiles, steps)                                        \
    {                                                                       \
        if (gpu.logging) gpu.log.push_back({kernel, tiles, (int)(steps)}); \
        gpu.launch((void *)st);                                             \
        return hipSuccess;                                                  \
    }
hipError_t launch_step(const SolveDesc *, const uint2 *, int ntiles, const int64_t *, int64_t, const int *, int, bool,
                       bool, bool, hipStream_t st) STEPS('m', ntiles, 1)
hipError_t launch_step2(const SolveDesc *, const uint2 *, int ntiles, const int64_t *, int64_t, const int *, int,
                        bool single, bool, bool, bool, hipStream_t st) STEPS('d', ntiles, single ? 1 : 2)
hipError_t launch_column(const SolveDesc *, const uint2 *, int ntiles, const int64_t *, int64_t, const int *, int, int nk,
                         bool, bool, hipStream_t st) STEPS('c', ntiles, nk)
hipError_t launch_patch(const SolveDesc *, const uint2 *, int ntiles, int, int, const int64_t *, int64_t, const int *, int,
                        int nk, bool, bool, hipStream_t st) STEPS('p', ntiles, nk)
hipError_t launch_advance(const SolveDesc *, int *, int64_t *, int, int64_t, int, hipStream_t) { return hipSuccess; }
hipError_t launch_records(const SolveDesc *, int, const int64_t *, int64_t, int64_t, hipStream_t) { return hipSuccess; }
hipError_t launch_omega(const SolveDesc &, bool, const double *, double, hipStream_t) { return hipSuccess; }
hipError_t launch_noneq(const SolveDesc &, int, bool, double *, hipStream_t) { return hipSuccess; }
hipError_t launch_init_ic(const SolveDesc &, int, bool, const pdbm_ic &, hipStream_t) { return hipSuccess; }
hipError_t launch_init_fields(const SolveDesc &, int, bool, const double *, hipStream_t) { return hipSuccess; }
hipError_t launch_planes_out(const SolveDesc &, int, bool, int, int, bool, void *, double *, hipStream_t)
{
    return hipSuccess;
}
hipError_t launch_planes_in(const SolveDesc &, int, bool, int, int, bool, const void *, const double *, hipStream_t)
{
    return hipSuccess;
}
hipError_t launch_moments(const SolveDesc &d, int, bool, double *out, const DiagCtl &dc, hipStream_t)
{
    // fields that name the solve: its step count
    for (int i = 0; out && i < 6 * d.nr * d.nt; ++i) out[i] = (double)d.nsteps;
    *dc.out = pdbm_diag{dc.step, (double)d.nsteps, 0.0, 0.0, 0, 0};
    return hipSuccess;
}
int cell_blocks(int nr, int nt) { return (nr * nt + BLOCK - 1) / BLOCK; }
int solve_waves(int nr, int nt, int rows)
{
    return nt == 1 ? (nr + COL_W - 1) / COL_W : (nr + rows - 1) / rows * ((nt + STRIP - 1) / STRIP);
}
void release_scratch_solver(int) {}
}  // namespace pdbm
