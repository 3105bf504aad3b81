// stub.h -- what the CPU tests of the host code see of the stand-in runtime (hip/hip_runtime.h, stub.cpp).
//
// Device memory is host memory of the process; launchers move no data but note which allocations they
// touch.  Every stream and the host carry a vector clock (which work of which stream they are ordered
// behind), and each use and each stream-ordered free of an allocation is checked against the work of other
// streams that touched it: work that is not ordered before is a violation.
#pragma once
#include <stddef.h>

#include <string>
#include <vector>

namespace stub {

struct Launch {
    std::string name;
    int chunk, n_tot, n_chunks, mm, form, n_jobs;   // of the first job of a quadrature
    long long tiles;
};

extern std::vector<std::string> violations;   // in order, with the names of the two works
extern std::vector<Launch> launches;          // quadratures since the start (or the last clear())
extern long long fail_alloc_at;               // the n-th device allocation from now on fails (0: none) ...
extern long long fail_allocs;                 // ... and this many after it
extern bool fields_factor;                    // outcome of the factoring test of fields from the caller
extern float (*elapsed)();                    // what hipEventElapsedTime gives, if set (ms)
extern double sim;                            // > 0: device work takes time (a model of it), times this

extern const void *elsewhere;                 // an allocation of another device; work here that touches it is a violation
extern long long waits;                       // waits of the host for work that it did not know to be done

struct PartialUse {
    const void *block;
    size_t bytes;
};
std::vector<PartialUse> partials();           // the live allocations that quadratures have written partials to

size_t live_bytes();    // device memory not freed
size_t peak_bytes();
long long allocations();
void clear();           // launches, violations, peak

}  // namespace stub
