// CPU test of the serving loop's host core (csrc/serve_core.{h,cpp}): once a
// server has served a number of requests at a time, serving as many again
// takes no heap allocation per request, only a few per micro-batch.  The
// records that it keeps are bounded, and a request that follows another in
// the same record returns its own beam.  Built with g++ and run by
// tests/test_serve_core_alloc_cpu.py; exits non-zero on the first failed check.
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <thread>
#include <vector>

#include "serve_core.h"

static std::atomic<long> g_allocs{0};
void *operator new(size_t n)
{
    ++g_allocs;
    void *p = std::malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }

#define CHECK(c)                                                                \
    do {                                                                        \
        if (!(c)) {                                                             \
            std::fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #c); \
            std::exit(1);                                                       \
        }                                                                       \
    } while (0)

namespace {

constexpr int N = 256, K = 32, MB = 64;

// Finishes a micro-batch at its first poll; the beam's words are the ticket's.
class FakeExecutor final : public cm::serve::Executor {
public:
    FakeExecutor() { beams.resize(cm::serve::MAX_SLOTS * MB * 2 * K); }
    bool launch(int si, const std::vector<cm::serve::Work> &b, int32_t kb, std::string *) override
    {
        for (size_t j = 0; j < b.size(); ++j)
            for (int i = 0; i < 2 * kb; ++i)
                beams[((size_t)si * MB + j) * 2 * K + i] = (uint32_t)(b[j].ticket * 64 + i);
        return true;
    }
    int poll(int, std::string *) override { return 1; }
    const uint32_t *beam(int si, size_t j) override { return &beams[((size_t)si * MB + j) * 2 * K]; }
    double kernel_us(int) override { return 1.0; }
    void kernel_clock(int, double *s, double *e) override { *s = 1.0, *e = 2.0; }
    std::vector<uint32_t> beams;
};

}  // namespace

int main()
{
    cm_server_cfg cfg{};
    cfg.precision = CM_BF16;
    cfg.k = K;
    cfg.arena_bytes = (int64_t)1 << 30;
    cfg.max_slots = 3;
    cfg.max_pending = 4 * N;
    cfg.max_sessions = N;
    cfg.max_stages = 8;
    cfg.max_batch_queries = MB;
    cfg.max_batch_cands = 1 << 20;
    FakeExecutor ex;
    cm::serve::Core core(cfg, &ex);
    std::thread worker([&] { core.run(); });
    std::string err;
    std::vector<int32_t> sid(N);
    alignas(16) static float data[64];
    std::vector<cm_request> rq(N);
    for (int s = 0; s < N; ++s) {
        CHECK(core.session_reserve(4, &sid[s], &err) == CM_OK);
        core.session_ready(sid[s], true);
        rq[s].n_cands = 10 + s;
        rq[s].sched = data;
        rq[s].terms = data;
    }
    std::vector<uint64_t> tickets(N);
    std::vector<cm_result> out(N);
    std::vector<int32_t> idx(N * K);
    std::vector<float> val(N * K);
    auto round = [&](int k) {
        for (int s = 0; s < N; ++s) {
            rq[s].k = k;
            out[s].k = K;
            out[s].idx = &idx[(size_t)s * K];
            out[s].val = &val[(size_t)s * K];
        }
        CHECK(core.submit_batch(N, sid.data(), rq.data(), tickets.data(), &err) == CM_OK);
        CHECK(core.wait_all(N, tickets.data(), 60000, out.data(), &err) == CM_OK);
        for (int s = 0; s < N; ++s) {
            CHECK(out[s].n == k);
            for (int i = 0; i < k; ++i) {
                const uint32_t want = (uint32_t)(tickets[s] * 64 + K + i);
                CHECK((uint32_t)idx[s * K + i] == (uint32_t)(tickets[s] * 64 + i));
                CHECK(std::memcmp(&val[s * K + i], &want, 4) == 0);
            }
            CHECK(out[s].t_submit_us <= out[s].t_admit_us && out[s].t_admit_us <= out[s].t_done_us);
        }
    };
    for (int r = 0; r < 3; ++r) round(K);
    const int R = 20;
    const long a0 = g_allocs;
    for (int r = 0; r < R; ++r) round(r % 3 ? K : 5);
    const double per_request = (double)(g_allocs - a0) / (R * N);
    std::printf("allocations per request: %.3f\n", per_request);
    CHECK(per_request < 0.5);
    core.stop();
    worker.join();
    std::printf("all checks passed\n");
    return 0;
}
