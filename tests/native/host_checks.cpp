// host_checks.cpp -- checks of the library's host code on the CPU, on the stand-in runtime of hip_stub/.
//   host_checks NAME
// runs one check; it prints what is wrong and exits 1, or exits 0.
#include <sc.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <string>
#include <vector>

#include <hip/hip_runtime.h>

#include "sc_host.h"
#include "stub.h"

static int failures = 0;
#define EXPECT(cond, ...)                                   \
    do {                                                    \
        if (!(cond)) {                                      \
            std::printf("%s:%d: %s: ", __FILE__, __LINE__, #cond); \
            std::printf(__VA_ARGS__);                       \
            std::printf("\n");                              \
            ++failures;                                     \
        }                                                   \
    } while (0)
#define OK(call) EXPECT((call) == SC_OK, "%s", sc_last_error())

static void no_violations(const char *where)
{
    std::map<std::string, int> count;
    for (auto &v : stub::violations) count[v]++;
    for (auto &c : count) EXPECT(false, "%s: %s (%d times)", where, c.first.c_str(), c.second);
}

struct Request {
    std::vector<double> k, spectrum, obs, t;
    sc_request q{};
    Request(int n_r, int n_phi, int n_k, int n_obs, int consistent)
    {
        for (int i = 0; i < n_k; ++i) {
            k.push_back(2.0 * M_PI * (1.0 + 0.01 * i));
            spectrum.push_back(1.0);
            spectrum.push_back(0.1 * i);
        }
        for (int i = 0; i < n_obs; ++i)
            for (int c = 0; c < 3; ++c) obs.push_back(std::sin(1.0 + 3.0 * i + c));
        t = {0.0, 1.0, 2.0};
        q.f = 20.0;
        q.r_max = 30.0;
        q.n_r = n_r;
        q.n_phi = n_phi;
        q.n_k = n_k;
        q.k = k.data();
        q.spectrum = spectrum.data();
        q.w0 = 15.0;
        q.consistent = consistent;
        q.n_obs = n_obs;
        q.obs = obs.data();
        q.prec = SC_FP32_SPLIT;
        q.n_t = 3;
        q.t = t.data();
        q.dk = 0.1;
    }
};

// Idle blocks of the server's cache are given back (an allocation failed, the server ends) only behind the
// work on them: a served FP32 request whose current does not factor, each of its allocations failing once.
static void idle_blocks()
{
    int reached = 0;
    for (int n = 1; n <= 80; ++n) {
        sc_ctx *ctx = nullptr;
        sc_server *s = nullptr;
        OK(sc_ctx_create(0, nullptr, &ctx));
        OK(sc_server_create(ctx, size_t(20) << 30, 4, 20.0, &s));
        stub::clear();
        for (int i = 0; i < 2; ++i) {
            Request r(40 + 20 * i, 48 + 20 * i, 3 + i, 300 + 100 * i, 1);
            uint64_t ticket = 0;
            stub::fail_alloc_at = i == 1 ? n : 0;
            OK(sc_server_submit(s, &r.q, &ticket));
            const sc_status st = sc_server_wait(s, ticket, 10000.0, nullptr, nullptr, nullptr, nullptr, nullptr);
            EXPECT(st == SC_OK || (st == SC_E_NOMEM && i == 1), "%s", sc_last_error());   // (the job buffer's is not retried)
            reached += i == 1 && stub::fail_alloc_at == 0;
            stub::fail_alloc_at = 0;
        }
        OK(sc_server_destroy(s));
        OK(sc_ctx_destroy(ctx));
        no_violations("failed allocation");
        if (failures) return;
    }
    EXPECT(reached > 10, "%d", reached);
    EXPECT(stub::live_bytes() == 0, "%zu bytes not freed", stub::live_bytes());
}

// A block from the cache counts with its own size, which may be a quarter more than was asked for.
static void block_sizes()
{
    sc::BlockCache cache;
    cache.limit = 64 << 20;
    {
        sc::DevBuf a, b;
        EXPECT(a.reserve(10 << 20, {nullptr, &cache}) == SC_OK, "reserve");
        a.release();
        const long long before = stub::allocations();
        EXPECT(b.reserve(9 << 20, {nullptr, &cache}) == SC_OK && stub::allocations() == before, "the idle block was not taken");
        EXPECT(b.bytes == 10 << 20, "%zu bytes counted of %d held", b.bytes, 10 << 20);
    }
    cache.trim();
    EXPECT(stub::live_bytes() == 0, "%zu bytes not freed", stub::live_bytes());
}

// Blocks of sizes that nobody asks for again do not fill the cache for good.
static void block_turnover()
{
    sc::BlockCache cache;
    cache.limit = 16 << 20;
    {
        sc::DevBuf all[8];
        for (auto &a : all) EXPECT(a.reserve(2 << 20, {nullptr, &cache}) == SC_OK, "reserve");
    }
    EXPECT(cache.held == cache.limit, "%zu bytes wait", cache.held);
    for (size_t n : {size_t(9) << 20, size_t(13) << 20}) {
        sc::DevBuf a, b;
        EXPECT(a.reserve(n, {nullptr, &cache}) == SC_OK, "reserve");
        a.release();
        EXPECT(cache.held <= cache.limit, "%zu bytes wait", cache.held);
        const long long before = stub::allocations();
        EXPECT(b.reserve(n, {nullptr, &cache}) == SC_OK && stub::allocations() == before,
               "a block of %zu bytes was not kept", n);
    }
    cache.trim();
    EXPECT(stub::live_bytes() == 0, "%zu bytes not freed", stub::live_bytes());
    no_violations("turnover");
}

// Serving a request whose current factors, no thread waits for the device.
static void no_waits()
{
    for (sc_precision prec : {SC_FP32_SPLIT, SC_FP64}) {
        sc_ctx *ctx = nullptr;
        sc_server *s = nullptr;
        OK(sc_ctx_create(0, nullptr, &ctx));
        OK(sc_server_create(ctx, size_t(20) << 30, 4, 20.0, &s));
        Request r(60, 64, 3, 900, 0);
        r.q.prec = prec;
        uint64_t ticket = 0;
        const long long before = stub::waits;
        OK(sc_server_submit(s, &r.q, &ticket));
        OK(sc_server_wait(s, ticket, 10000.0, nullptr, nullptr, nullptr, nullptr, nullptr));
        EXPECT(stub::waits == before, "%lld waits", stub::waits - before);
        OK(sc_server_destroy(s));
        OK(sc_ctx_destroy(ctx));
    }
    no_violations("served requests");
}

// ------------------------------------------------------------------------------ single problems

struct Problem {
    sc_prob *p = nullptr;
    void *points = nullptr;
    // `direct`: the points in device memory, so that the sum is taken node by node
    Problem(sc_ctx *ctx, int n_r, int n_phi, int n_k, int n_obs, bool direct, double k0 = 2.0 * M_PI)
    {
        std::vector<double> k, obs;
        for (int i = 0; i < n_k; ++i) k.push_back(k0 * (1.0 + 0.01 * i));
        for (int i = 0; i < 3 * n_obs; ++i) obs.push_back(std::sin(1.0 + 3.0 * i));
        OK(sc_prob_create(ctx, &p));
        OK(sc_set_mirror(p, 20.0, 30.0, n_r, n_phi));
        OK(sc_set_frequencies(p, k.data(), n_k));
        OK(sc_set_incident_gaussian(p, 15.0, 0.0, nullptr, 0));
        if (direct) {
            (void)hipMalloc(&points, sizeof(double) * obs.size());
            memcpy(points, obs.data(), sizeof(double) * obs.size());
        }
        OK(sc_set_observation(p, direct ? (double *)points : obs.data(), n_obs, direct));
    }
    ~Problem()
    {
        OK(sc_prob_destroy(p));
        if (points) (void)hipFree(points);
    }
    void launch(int chunk) const
    {
        sc_launch l{};
        l.chunk = chunk;
        OK(sc_set_launch(p, &l));
    }
    int reported() const
    {
        sc_timing t{};
        OK(sc_get_timing(p, &t));
        return t.chunk;
    }
};

// A chunk that the caller, a tuned entry or a batch launch sets is the one the direct sum takes, and sc_get_timing
// tells the one it took.
static void chunks()
{
    sc_ctx *ctx = nullptr;
    OK(sc_ctx_create(0, nullptr, &ctx));
    for (sc_precision prec : {SC_FP32_SPLIT, SC_FP64, SC_FP32}) {
        Problem a(ctx, 80, 64, 3, 200, true);
        auto evaluate = [&](int want) {
            stub::clear();
            OK(sc_evaluate(a.p, prec, nullptr, nullptr, 0));
            const stub::Launch &l = stub::launches.back();
            EXPECT(!l.mm && (want == 0 ? l.chunk < 2048 : l.chunk == want), "took %d for %d", l.chunk, want);
            EXPECT(a.reported() == l.chunk, "reported %d, took %d", a.reported(), l.chunk);
        };
        evaluate(0);
        for (int chunk : {64, 256, 2048, 4096}) {
            a.launch(chunk);
            evaluate(chunk);
        }
        OK(sc_set_launch(a.p, nullptr));
        sc_launch shape{1, 4, 1024, 0, 1};
        OK(sc_set_batch_launch(ctx, prec, &shape));
        sc_prob *one[1] = {a.p};
        stub::clear();
        OK(sc_evaluate_batch(ctx, one, 1, prec));
        EXPECT(stub::launches.back().chunk == 1024 && a.reported() == 1024, "%d", stub::launches.back().chunk);
        OK(sc_set_batch_launch(ctx, prec, nullptr));
        // a tuned entry, written as sc_autotune_save does (layouts 0 ... 2, so that one of them is this problem's)
        FILE *f = fopen("tune.txt", "w");
        for (int layout = 0; layout < 3; ++layout) fprintf(f, "%d %d 7 1 12 1 4 512 0 1\n", (int)prec, layout);
        fclose(f);
        OK(sc_autotune_load(ctx, "tune.txt"));
        evaluate(512);
    }
    OK(sc_ctx_destroy(ctx));
}

// The partials of a batch stay within 8 GiB (the documented cap for few nodes), whether the chunk is raised to
// that end or only not shortened, and with compacted sums beside them.
static void batch_cap()
{
    const double cap = 8.0 * 1073741824.0;
    for (bool mixed : {false, true}) {
        sc_ctx *ctx = nullptr;
        OK(sc_ctx_create(0, nullptr, &ctx));
        {
            std::vector<Problem *> ps;
            std::vector<sc_prob *> h;
            // 12 x 4 B x 64 frequencies x 768 points x 25 chunks of 384 nodes: 59 MB each; 15 MB at 2048 nodes
            for (int i = 0; i < 190; ++i) ps.push_back(new Problem(ctx, 95, 100, 64, 700, !mixed || i % 2));
            for (Problem *p : ps) h.push_back(p->p);
            OK(sc_evaluate_batch(ctx, h.data(), (int)h.size(), SC_FP32_SPLIT));
            double held = 0.0;
            for (const stub::PartialUse &u : stub::partials()) held += (double)u.bytes;
            EXPECT(held < cap, "%.1f GB of partials", held * 1e-9);
            for (Problem *p : ps) delete p;
        }
        // and where the chunk had to be raised, it stays raised: 12 x 4 B x 256 x 16384 points x 51 chunks = 10.3 GB
        {
            Problem big(ctx, 320, 320, 256, 16384, true);
            sc_prob *one[1] = {big.p};
            stub::clear();
            OK(sc_evaluate_batch(ctx, one, 1, SC_FP32_SPLIT));
            EXPECT(stub::launches.back().chunk == 4096 && big.reported() == 4096, "%d", stub::launches.back().chunk);
        }
        OK(sc_ctx_destroy(ctx));
    }
}

// Each candidate seems faster than the one before: tuning a compacted sum times nothing that cannot differ, and
// what it keeps is not taken by direct sums of the same sizes.
static void tuner()
{
    static float ms;
    ms = 1000.0f;
    stub::elapsed = [] { return ms -= 1.0f; };
    for (sc_precision prec : {SC_FP32_SPLIT, SC_FP64}) {
        sc_ctx *ctx = nullptr;
        OK(sc_ctx_create(0, nullptr, &ctx));
        {
            Problem a(ctx, 200, 200, 4, 2000, false), b(ctx, 200, 200, 4, 2000, true);
            sc_launch before{}, after{}, best{};
            OK(sc_get_launch(b.p, prec, &before));
            stub::clear();
            OK(sc_autotune(a.p, prec, 1e6, &best));
            EXPECT(stub::launches[0].n_tot < 20000, "not compacted");
            const size_t n = stub::launches.size();
            EXPECT(n <= (prec == SC_FP64 ? 40 : 2), "%zu evaluations", n);
            EXPECT(best.chunk == before.chunk, "a chunk of %d for a sum without one", best.chunk);
            if (prec == SC_FP32_SPLIT) EXPECT(best.obs_per_lane == before.obs_per_lane, "%d", best.obs_per_lane);
            OK(sc_get_launch(b.p, prec, &after));
            EXPECT(memcmp(&before, &after, sizeof before) == 0, "the direct sum's launch changed");
            OK(sc_get_launch(a.p, prec, &after));
            EXPECT(memcmp(&best, &after, sizeof best) == 0, "the tuned launch is not taken");
            OK(sc_autotune_save(ctx, "tune.txt"));
            OK(sc_autotune_load(ctx, "tune.txt"));
            sc_prob *ps[1] = {a.p};
            stub::clear();
            OK(sc_autotune_batch(ctx, ps, 1, prec, 1e6, &best));
            EXPECT(stub::launches.size() <= (prec == SC_FP64 ? 24u : 2u) && best.chunk == 0, "%zu evaluations, chunk %d",
                   stub::launches.size(), best.chunk);
            // a direct sum is tuned as ever: the last candidate, one workgroup per CU and the largest chunk tried
            OK(sc_set_batch_launch(ctx, prec, nullptr));
            OK(sc_autotune(b.p, prec, 1e6, &best));
            EXPECT(best.chunk == 16384 && best.blocks_per_cu == 1, "%d %d", best.chunk, best.blocks_per_cu);
        }
        OK(sc_ctx_destroy(ctx));
    }
    stub::elapsed = nullptr;
}

// Results for another device's memory are copied there: no kernel of this one writes to it.
static void other_device()
{
    sc_ctx *ctx = nullptr;
    OK(sc_ctx_create(0, nullptr, &ctx));
    {
        Problem a(ctx, 80, 64, 3, 200, false);
        void *E = nullptr, *B = nullptr;
        const size_t n = sizeof(float) * 6 * 3 * 200;
        (void)hipMalloc(&E, n);
        (void)hipMalloc(&B, n);
        for (const void *x : {(const void *)nullptr, (const void *)E, (const void *)B}) {
            stub::elsewhere = x;
            OK(sc_evaluate(a.p, SC_FP32_SPLIT, E, B, 1));
        }
        OK(sc_ctx_synchronize(ctx));
        (void)hipFree(E);
        (void)hipFree(B);
    }
    OK(sc_ctx_destroy(ctx));
    no_violations("results elsewhere");
}

int main(int argc, char **argv)
{
    const std::map<std::string, std::function<void()>> checks = {
        {"idle_blocks", idle_blocks},
        {"block_sizes", block_sizes},
        {"block_turnover", block_turnover},
        {"no_waits", no_waits},
        {"chunks", chunks},
        {"batch_cap", batch_cap},
        {"tuner", tuner},
        {"other_device", other_device},
    };
    if (argc == 2 && checks.count(argv[1])) {
        checks.at(argv[1])();
        return failures ? 1 : 0;
    }
    std::printf("which check?\n");
    return 2;
}
