// stub.cpp -- the stand-in HIP runtime and launchers (see stub.h).
#include "stub.h"

#include <hip/hip_runtime.h>
#include <stdlib.h>
#include <string.h>
#include <sys/mman.h>

#include <algorithm>
#include <chrono>
#include <initializer_list>
#include <map>
#include <mutex>
#include <thread>

#include "sc_internal.h"

using Clock = std::map<const void *, long long>;   // stream -> work ordered before
using Time = std::chrono::steady_clock;

struct StubStream {
    Clock before;
    long long seq = 0;
    Time::time_point end{};
    std::string last;
};
struct StubEvent {
    Clock before;
    Time::time_point at{};
};

namespace stub {
std::vector<std::string> violations;
std::vector<Launch> launches;
long long fail_alloc_at = 0, fail_allocs = 0;
bool fields_factor = false;
float (*elapsed)() = nullptr;
double sim = 0.0;
long long waits = 0;
const void *elsewhere = nullptr;
}  // namespace stub
using namespace stub;

namespace {

std::recursive_mutex mu;
Clock host;
size_t live = 0, peak = 0;
long long n_alloc = 0;
StubStream null_stream;

struct Use {
    long long seq;
    std::string what;
};
struct Alloc_ {
    size_t bytes;
    bool partials = false;
    std::map<StubStream *, Use> uses;
};
std::map<char *, Alloc_> allocs;
#define LOCK std::lock_guard<std::recursive_mutex> lk_(mu)

StubStream *real(hipStream_t s) { return s ? s : &null_stream; }
void merge(Clock &a, const Clock &b)
{
    for (auto &x : b) a[x.first] = std::max(a[x.first], x.second);
}

void check(StubStream *s, Alloc_ &a, const std::string &what)
{
    for (auto &u : a.uses) {
        if (u.first == s) continue;
        auto it = s->before.find(u.first);
        if (it == s->before.end() || it->second < u.second.seq)
            violations.push_back(what + " is not ordered behind " + u.second.what);
    }
}

// One piece of work on a stream that touches these addresses, `us` long.
void work(hipStream_t st, const char *what, std::initializer_list<const void *> ptrs, double us = 3.0)
{
    LOCK;
    StubStream *s = real(st);
    merge(s->before, host);
    ++s->seq;
    s->before[s] = s->seq;
    for (const void *p : ptrs) {
        if (!p) continue;
        auto it = allocs.upper_bound((char *)p);
        if (it == allocs.begin()) continue;
        --it;
        if ((char *)p >= it->first + it->second.bytes) continue;
        if (it->first == elsewhere && strcmp(what, "copy") != 0) violations.push_back(std::string(what) + " on another device's memory");
        check(s, it->second, what);
        it->second.uses[s] = {s->seq, what};
    }
    if (sim > 0.0)
        s->end = std::max(s->end, Time::now()) + std::chrono::nanoseconds((long long)(us * 1e3 * sim));
}

hipError_t take(void **p, size_t n)
{
    LOCK;
    ++n_alloc;
    if (fail_alloc_at > 0 && --fail_alloc_at == 0) {
        if (fail_allocs > 0) {
            --fail_allocs;
            fail_alloc_at = 1;
        }
        return hipErrorOutOfMemory;
    }
    n = (n + 4095) / 4096 * 4096;
    void *q = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (q == MAP_FAILED) return hipErrorOutOfMemory;
    allocs[(char *)q].bytes = n;
    live += n;
    peak = std::max(peak, live);
    *p = q;
    return hipSuccess;
}
hipError_t give(void *p, StubStream *s)
{
    LOCK;
    auto it = allocs.find((char *)p);
    if (it == allocs.end()) {
        violations.push_back("free of an unknown address");
        return hipErrorInvalidValue;
    }
    if (s) {
        merge(s->before, host);
        check(s, it->second, "free");
    }
    live -= it->second.bytes;
    munmap(p, it->second.bytes);
    allocs.erase(it);
    return hipSuccess;
}
// The host waits for what `before` holds.
void host_waits(const Clock &before)
{
    for (auto &x : before)
        if (host[x.first] < x.second) {
            ++waits;
            break;
        }
    merge(host, before);
}
void wait_until(Time::time_point t)
{
    if (sim > 0.0) std::this_thread::sleep_until(t);
}

}  // namespace

namespace stub {
size_t live_bytes() { LOCK; return live; }
size_t peak_bytes() { LOCK; return peak; }
long long allocations() { LOCK; return n_alloc; }
std::vector<PartialUse> partials()
{
    LOCK;
    std::vector<PartialUse> v;
    for (auto &a : allocs)
        if (a.second.partials) v.push_back({a.first, a.second.bytes});
    return v;
}
void clear()
{
    LOCK;
    launches.clear();
    violations.clear();
    peak = live;
}
}  // namespace stub

hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p)
{
    LOCK;
    auto it = allocs.upper_bound((char *)p);
    if (it == allocs.begin() || (char *)p >= std::prev(it)->first + std::prev(it)->second.bytes) return hipErrorInvalidValue;
    a->type = hipMemoryTypeDevice;
    a->device = std::prev(it)->first == elsewhere ? 1 : 0;
    return hipSuccess;
}
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int) { p->multiProcessorCount = 256; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "stand-in error"; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = new StubStream; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }   // (kept: its address names it in the clocks)
hipError_t hipStreamSynchronize(hipStream_t st)
{
    Time::time_point t;
    {
        LOCK;
        t = real(st)->end;
    }
    wait_until(t);
    LOCK;
    host_waits(real(st)->before);
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t st, hipEvent_t e, unsigned)
{
    LOCK;
    merge(real(st)->before, e->before);
    real(st)->end = std::max(real(st)->end, e->at);
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t *e) { *e = new StubEvent; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { delete e; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t st)
{
    LOCK;
    e->before = real(st)->before;
    e->at = std::max(real(st)->end, Time::now());
    return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e)
{
    LOCK;
    if (sim > 0.0 && Time::now() < e->at) return hipErrorNotReady;
    merge(host, e->before);
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e)
{
    Time::time_point t;
    {
        LOCK;
        t = e->at;
    }
    wait_until(t);
    LOCK;
    host_waits(e->before);
    return hipSuccess;
}
hipError_t hipEventElapsedTime(float *ms, hipEvent_t a, hipEvent_t b)
{
    *ms = elapsed ? elapsed() : std::chrono::duration<float, std::milli>(b->at - a->at).count();
    return hipSuccess;
}
hipError_t hipMallocRaw(void **p, size_t n) { return take(p, n); }
hipError_t hipMallocAsyncRaw(void **p, size_t n, hipStream_t) { return take(p, n); }
hipError_t hipFree(void *p)
{
    // (waits for the device)
    LOCK;
    return give(p, nullptr);
}
hipError_t hipFreeAsync(void *p, hipStream_t s) { return give(p, real(s)); }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = malloc(n); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMemGetInfo(size_t *f, size_t *t) { *f = *t = size_t(288) << 30; return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t st)
{
    work(st, "copy", {d, s}, 2.0 + n / 5e4);
    if (k == hipMemcpyHostToDevice || n <= (1 << 20)) memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind k)
{
    hipMemcpyAsync(d, s, n, k, nullptr);
    return hipStreamSynchronize(nullptr);
}
hipError_t hipDeviceGetDefaultMemPool(hipMemPool_t *p, int) { *p = (hipMemPool_t)&null_stream; return hipSuccess; }
hipError_t hipMemPoolGetAttribute(hipMemPool_t, hipMemPoolAttr, void *v) { *(uint64_t *)v = 0; return hipSuccess; }
hipError_t hipMemPoolSetAttribute(hipMemPool_t, hipMemPoolAttr, void *) { return hipSuccess; }
hipError_t hipMemPoolTrimTo(hipMemPool_t, size_t) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *s) { *p = (void *)s; return hipSuccess; }

// ------------------------------------------------------------------------------ launchers
namespace sc {

typedef const double *cd;
#define OK return hipSuccess

hipError_t launch_node_tables(hipStream_t st, int, int, double, cd r, cd wr, cd c, cd s, double, double *p64, float *p32,
                              double *nrm, double *wgt, double *tan, double *h64, float *h32)
{
    work(st, "node tables", {r, wr, c, s, p64, p32, nrm, wgt, tan, h64, h32});
    OK;
}
hipError_t launch_surface_records(hipStream_t st, int, int, cd a, cd b, cd c, cd d, cd e, double *p64, float *p32,
                                  double *nrm, double *wgt, double *tan, double *h64, float *h32)
{
    work(st, "surface records", {a, b, c, d, e, p64, p32, nrm, wgt, tan, h64, h32});
    OK;
}
hipError_t launch_obs_prep(hipStream_t st, cd x, int, int, double *o64, float *o32)
{
    work(st, "points", {x, o64, o32});
    OK;
}
hipError_t launch_tables_from_fields(hipStream_t st, int, int, int, cd k, cd p, cd n, cd w, cd t, cd E, cd B, double *tab)
{
    work(st, "tables from fields", {k, p, n, w, t, E, B, tab});
    OK;
}
static void factored(hipStream_t st, const char *what, const FactorOut &o, bool factors)
{
    work(st, what, {o.pos32, o.pos64, o.tabf, o.posf, o.betaf, o.tabp, o.tabf64, o.posf64, o.betaf64, o.bad});
    for (int b = 0; b < 4 && !factors; ++b) o.bad[b] = o.epoch;
}
hipError_t launch_tables_beam(hipStream_t st, int n_k, int, int n_tot, cd k, cd p, cd n, cd w, cd t, int beam, double,
                              double, cd spec, int consistent, cd modes, int, double *tab64, int, const FactorOut *out,
                              double *part, double *P)
{
    work(st, "beam tables", {k, p, n, w, t, spec, modes, tab64, part, P}, 10.0 + 1.5e-5 * n_k * n_tot);
    if (out) factored(st, "beam tables", *out, !(beam == 3 || (beam == 0 && consistent)));
    OK;
}
hipError_t launch_tables_cast(hipStream_t st, int n_k, int n_tot, cd k, cd p, cd t64, const float *t32, float *out, int)
{
    work(st, "cast", {k, p, t64, t32, out}, 5.0 + 2e-5 * n_k * n_tot);
    OK;
}
hipError_t launch_power_fields(hipStream_t st, int, int, int, cd n, cd w, cd E, cd B, double *part, double *P)
{
    work(st, "power", {n, w, E, B, part, P});
    OK;
}
int64_t power_partial_count(int n_k, int n_tot) { return (int64_t)n_k * std::max(64, (n_tot + 63) / 64); }
hipError_t launch_tables_scale(hipStream_t st, int, int, int, cd f, double *t64, float *t32)
{
    work(st, "scale", {f, t64, t32});
    OK;
}
hipError_t launch_tables_factor(hipStream_t st, int, int, cd k, cd t64, const FactorOut &out)
{
    work(st, "factor", {k, t64});
    factored(st, "factor", out, fields_factor);
    OK;
}
hipError_t launch_tables_polar(hipStream_t st, int64_t, const float *f, float *p) { work(st, "polar", {f, p}); OK; }
hipError_t launch_maxwell_freq(hipStream_t st, int, int, int, double, cd k, const void *E, const void *B, double *w,
                               double *mx, double *o)
{
    work(st, "maxwell", {k, E, B, w, mx, o});
    OK;
}
hipError_t launch_maxwell_time(hipStream_t st, int, int, int, double, double, const void *E, const void *B, double *w,
                               double *mx, double *o)
{
    work(st, "maxwell", {E, B, w, mx, o});
    OK;
}
int diag_slots() { return 32; }
int energy_partial_count(int n_t) { return 64 * n_t; }
hipError_t launch_energy(hipStream_t st, int, int, int, const void *E, const void *B, double, double *part, double *W)
{
    work(st, "energy", {E, B, part, W});
    OK;
}

static void quad(hipStream_t st, const QuadJob *jobs, const QuadJob &one, int n_jobs, const void *counter, int per_lane)
{
    const QuadJob *js = jobs ? jobs : &one;
    double values = 0.0;
    for (int i = 0; i < n_jobs; ++i) {
        const QuadJob &j = js[i];
        const double per = (j.mm ? 128.0 * j.mm : 64.0 * per_lane) * std::min(j.chunk, j.n_tot);
        values += (double)j.n_tiles * per;
    }
    for (int i = 0; i < n_jobs; ++i) {
        const QuadJob &j = js[i];
        work(st, "quadrature", {j.tab, j.pos, j.obs, j.hinv, j.beta, j.tabp, j.mtab, j.mscale, j.k, j.partial, jobs, counter},
             i ? 0.0 : 12.0 + values / 1.2e6);
    }
    LOCK;
    for (int i = 0; i < n_jobs; ++i) {
        auto it = allocs.upper_bound((char *)js[i].partial);
        if (it != allocs.begin()) std::prev(it)->second.partials = true;
    }
    launches.push_back({js[0].mm ? "matrix" : "direct", js[0].chunk, js[0].n_tot, js[0].n_chunks, js[0].mm, js[0].form,
                        n_jobs, (long long)js[0].n_tiles});
}
hipError_t launch_quad(hipStream_t st, int, int opl, int fpb, int, int, const QuadJob &one, const QuadJob *jobs, int n,
                       int64_t, unsigned int *counter)
{
    quad(st, jobs, one, n, counter, opl * fpb);
    OK;
}
hipError_t launch_quad_mm_one(hipStream_t st, int, const QuadJob &job) { quad(st, nullptr, job, 1, nullptr, 0); OK; }
hipError_t launch_quad_mm(hipStream_t st, int, const QuadJob *jobs, int n, int64_t)
{
    quad(st, jobs, jobs[0], n, nullptr, 0);
    OK;
}
size_t mm_scale_bytes(int n_k) { return (size_t)n_k * (64 + 640); }
hipError_t launch_mm_tables(hipStream_t st, int, int, int, cd k, double, const float *c, const float *p, float *s, void *m)
{
    work(st, "packed rows", {k, c, p, s, m});
    OK;
}
hipError_t launch_reduce(hipStream_t st, int, const void *p, int, int, int, int, cd k, int, int, int, void *E, void *B,
                         void *E2, void *B2)
{
    work(st, "reduction", {p, k, E, B, E2, B2}, 10.0);
    OK;
}
hipError_t launch_compact_geometry(hipStream_t st, const CompactPlan &, int, int, double, cd r, double *a, double *b, int,
                                   void *p, void *h)
{
    work(st, "compact geometry", {r, a, b, p, h}, 10.0);
    OK;
}
hipError_t launch_compact_tables(hipStream_t st, const CompactPlan &, int n_r, int n_phi, int, int n_k, int, int,
                                 const void *t, const void *p, cd a, cd b, double *T, void *o)
{
    work(st, "compact tables", {t, p, a, b, T, o}, 20.0 + 1.6e-5 * n_k * (double)n_r * n_phi);
    OK;
}
size_t twiddle_bytes(int n_k, int n_t) { return (size_t)16 * n_k * ((n_t + 7) / 8 * 8); }
hipError_t launch_twiddles(hipStream_t st, int, cd k, int, cd t, double, double *tw) { work(st, "twiddles", {k, t, tw}); OK; }
hipError_t launch_time(hipStream_t st, int, int n_k, int n_t, int64_t n_x, cd tw, const void *E, const void *B, void *Et,
                       void *Bt)
{
    work(st, "time", {tw, E, B, Et, Bt}, 5.0 + 3.7e-7 * n_k * n_t * (double)n_x);
    OK;
}
hipError_t launch_fill_u32(hipStream_t st, unsigned int *p, unsigned int v, int n)
{
    work(st, "fill", {p});
    for (int i = 0; i < n; ++i) p[i] = v;
    OK;
}
int quad_max_blocks_per_cu(int, int, int, int) { return 4; }

}  // namespace sc
