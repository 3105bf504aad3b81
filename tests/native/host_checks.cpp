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

int main(int argc, char **argv)
{
    const std::map<std::string, std::function<void()>> checks = {
        {"idle_blocks", idle_blocks},
        {"block_sizes", block_sizes},
        {"block_turnover", block_turnover},
        {"no_waits", no_waits},
    };
    if (argc == 2 && checks.count(argv[1])) {
        checks.at(argv[1])();
        return failures ? 1 : 0;
    }
    std::printf("which check?\n");
    return 2;
}
