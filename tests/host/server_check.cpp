// CPU check of the request server (pdbm_serve.hip) on a model of the GPU: the
// library's host code against HIP calls and kernel launches defined here.
// Device memory is host memory; copies and small kernels happen at once; the
// steps of a chunk are in flight until the check lets them end (`tokens`), and
// a synchronisation of their stream, or freeing memory, waits for that.
//   server_check slots|memory|reports|fields|random
// Exit status 0 when every check holds.
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
    return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { return *s = (hipStream_t)handle(), hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { return std::free((void *)s), hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { return gpu.wait((void *)s), hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return *e = (hipEvent_t)handle(), hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { return std::free((void *)e), hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *s) { return *s = hipStreamCaptureStatusNone, hipSuccess; }
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
#define STEPS(...) { gpu.launch((void *)st); return hipSuccess; }
hipError_t launch_step(const SolveDesc *, const uint2 *, int, const int64_t *, int64_t, const int *, int, bool, bool,
                       bool, hipStream_t st) STEPS()
hipError_t launch_step2(const SolveDesc *, const uint2 *, int, const int64_t *, int64_t, const int *, int, bool, bool,
                        bool, bool, hipStream_t st) STEPS()
hipError_t launch_column(const SolveDesc *, const uint2 *, int, const int64_t *, int64_t, const int *, int, int, bool,
                         bool, hipStream_t st) STEPS()
hipError_t launch_patch(const SolveDesc *, const uint2 *, int, int, int, const int64_t *, int64_t, const int *, int, int,
                        bool, bool, hipStream_t st) STEPS()
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

// ------------------------------------------------------------- the checks --
namespace {

int fails = 0;
#define CHECK(c)                                                        \
    do {                                                                \
        if (!(c)) {                                                     \
            std::fprintf(stderr, "FAILED line %d: %s\n", __LINE__, #c); \
            fails++;                                                    \
        }                                                               \
    } while (0)

constexpr int CHUNK = 4;

pdbm_params params()
{
    pdbm_params p{};
    p.nr = 6;
    p.ntheta = 9;
    p.sector = 8;
    p.r_min = 0.3;
    p.r_max = 1.0;
    p.dt = 1e-4;
    p.tau = 1e-3;
    return p;
}
pdbm_ic ic()
{
    pdbm_ic i{};
    i.inner[0] = i.inner[1] = i.outer[0] = i.outer[1] = 1.0;
    return i;
}
uint64_t submit(pdbm_server *s, int64_t steps, bool fields)
{
    const pdbm_params p = params();
    const pdbm_ic i = ic();
    uint64_t id = 0;
    CHECK(pdbm_submit(s, &p, &i, steps, fields ? PDBM_KEEP_FIELDS : 0, &id) == PDBM_OK);
    return id;
}
pdbm_server *server(int slots, size_t cap)
{
    pdbm_server *s = nullptr;
    CHECK(pdbm_server_create(cap, slots, CHUNK, nullptr, &s) == PDBM_OK);
    return s;
}
pdbm_server_stats stats(pdbm_server *s)
{
    pdbm_server_stats t{};
    pdbm_server_get_stats(s, &t);
    return t;
}
// Ends within 10 s (DONE or FAILED).
bool ends(pdbm_server *s, uint64_t id, int32_t want = PDBM_DONE)
{
    for (int k = 0; k < 10000; ++k) {
        int32_t state = -1;
        if (pdbm_poll(s, id, &state, nullptr, nullptr) != PDBM_EAGAIN) return state == want;
        std::this_thread::sleep_for(std::chrono::milliseconds(1));
    }
    return false;
}

// One long solve beside short ones of one chunk each, two running at a time:
// a short one is done and its place free by the next chunk, so the long one's
// chunks serve all of them.
void places(bool by_memory)
{
    size_t bytes = 0;
    const pdbm_params p = params();
    pdbm_state_bytes(&p, &bytes);
    for (bool fields : {false, true}) {
        constexpr int N = 20;
        gpu.allow(0);
        const long before = gpu.launched;
        pdbm_server *s = by_memory ? server(64, 2 * bytes + bytes / 2) : server(2, size_t(1) << 40);
        submit(s, N * CHUNK, false);
        CHECK(gpu.reaches(before + 1));
        for (int k = 0; k + 1 < N; ++k) submit(s, CHUNK, fields);
        gpu.allow(1L << 40);
        CHECK(pdbm_server_wait(s, 20.0) == PDBM_OK);
        const pdbm_server_stats t = stats(s);
        std::printf("%s, fields %d: %ld chunks for %d\n", by_memory ? "memory" : "slots", (int)fields,
                    (long)t.steps_launched / CHUNK, N);
        CHECK(t.steps_launched == N * CHUNK && t.done == N && t.hbm_in_use == 0);
        pdbm_server_destroy(s);
        CHECK(gpu.allocated == 0);
    }
}

// A finished request beside a long one is done, and may be released, while
// the next chunk is in flight (`fields`) or before it is launched.
void results(bool fields)
{
    gpu.allow(0);
    const long before = gpu.launched;
    pdbm_server *s = server(4, size_t(1) << 40);
    const uint64_t far = submit(s, 100 * CHUNK, false);
    CHECK(gpu.reaches(before + 1));
    const uint64_t a = submit(s, CHUNK, fields), b = submit(s, CHUNK - 1, fields);
    gpu.allow(2);  // the chunk in flight, and that of the two
    CHECK(gpu.reaches(before + 3));
    if (!fields) {
        int32_t state = -1;
        CHECK(pdbm_poll(s, a, &state, nullptr, nullptr) == PDBM_OK && state == PDBM_DONE);
    }
    CHECK(ends(s, a) && ends(s, b));
    std::vector<double> out(6 * 6 * 9);
    pdbm_diag d{};
    CHECK(pdbm_poll(s, a, nullptr, fields ? out.data() : nullptr, &d) == PDBM_OK);
    CHECK(d.step == CHUNK && d.mass == CHUNK && (!fields || (out[0] == CHUNK && out.back() == CHUNK)));
    CHECK(pdbm_release(s, a) == PDBM_OK && pdbm_release(s, b) == PDBM_OK);
    CHECK(stats(s).running == 1 && stats(s).done == 2);
    int32_t state = -1;
    CHECK(pdbm_poll(s, far, &state, nullptr, nullptr) == PDBM_EAGAIN && state == PDBM_RUNNING);
    gpu.allow(1L << 40);
    CHECK(pdbm_server_wait(s, 20.0) == PDBM_OK);
    CHECK(stats(s).hbm_in_use == 0 && stats(s).done == 3);
    pdbm_server_destroy(s);
    CHECK(gpu.allocated == 0);
}

// Clients submit, poll, release and wait from three threads while chunks end
// after random times, and the server is destroyed at a random moment: at once
// after the last result, in the middle, or with requests queued.
void random_use(unsigned seed, int rounds)
{
    std::mt19937 rng(seed);
    for (int r = 0; r < rounds; ++r) {
        const bool drain = rng() % 2;
        size_t bytes = 0;
        const pdbm_params p = params();
        pdbm_state_bytes(&p, &bytes);
        pdbm_server *s = server(1 + rng() % 5, rng() % 2 ? size_t(1) << 40 : bytes * (1 + rng() % 3) + bytes / 2);
        std::vector<std::thread> clients;
        for (int c = 0; c < 3; ++c)
            clients.emplace_back([s, sd = rng(), drain] {
                std::mt19937 g(sd);
                std::vector<std::pair<uint64_t, int>> mine;
                std::vector<double> out(6 * 6 * 9);
                for (int k = 0; k < 12; ++k) {
                    const bool fields = g() % 2;
                    const int n = (int)(g() % 30);
                    mine.push_back({submit(s, n, fields), fields ? n : -1});
                    if (g() % 3 == 0) std::this_thread::yield();
                    for (size_t i = 0; i < mine.size();) {
                        pdbm_diag d{};
                        int32_t state;
                        const bool f = mine[i].second >= 0;
                        const int rc = pdbm_poll(s, mine[i].first, &state, f ? out.data() : nullptr, &d);
                        if (rc == PDBM_EAGAIN) {
                            ++i;
                            continue;
                        }
                        CHECK(rc == PDBM_OK && state == PDBM_DONE && (!f || (out[0] == mine[i].second && d.step == mine[i].second)));
                        CHECK(pdbm_release(s, mine[i].first) == PDBM_OK);
                        mine.erase(mine.begin() + i);
                    }
                }
                if (drain) CHECK(pdbm_server_wait(s, 20.0) == PDBM_OK);
                const pdbm_server_stats t = stats(s);
                CHECK(t.submitted == t.queued + t.running + t.done + t.failed);
            });
        for (auto &t : clients) t.join();
        if (drain) CHECK(stats(s).queued == 0 && stats(s).running == 0 && stats(s).hbm_in_use == 0 && stats(s).failed == 0);
        pdbm_server_destroy(s);
        CHECK(gpu.allocated == 0);
    }
}

}  // namespace

int main(int argc, char **argv)
{
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "slots") places(false);
    else if (what == "memory") places(true);
    else if (what == "reports") results(false);
    else if (what == "fields") results(true);
    else if (what == "random") random_use(argc > 2 ? std::atoi(argv[2]) : 1, argc > 3 ? std::atoi(argv[3]) : 200);
    else return 2;
    if (!fails) std::printf("server %s ok\n", what.c_str());
    return fails ? 1 : 0;
}
