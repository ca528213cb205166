// CPU check of the request server (pdbm_serve.hip) on a model of the GPU: the
// library's host code against the HIP calls and launches of model_gpu.h.
//   server_check slots|memory|reports|fields|random
// Exit status 0 when every check holds.
#include "model_gpu.h"

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
// the next chunk is in flight.
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
