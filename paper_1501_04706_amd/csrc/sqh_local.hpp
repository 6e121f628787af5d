// Host interface of the workgroup-local hull kernels (sqh_local.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace sqh {

constexpr int kLocalPoints = 4096;    // points one workgroup holds in LDS
constexpr int kLocalStatPasses = 64;  // passes whose sizes are noted

// Written by the last kernel of a call straight into pinned host memory.
struct LocalStatus {
    int h;      // hull vertices (all sets)
    int err;    // kErr* flags
    int left;   // 1: nothing was written, the general path has to run
    int passes;
    int first_v;
    uint32_t orient, orient_exact, cmp_exact;
    unsigned long long t0, t1;  // device clock (100 MHz) at the call's start and end
    int pass_v[kLocalStatPasses], pass_s[kLocalStatPasses];
};

struct LocalArgs {
    const float2* xy;
    int n;
    int32_t* out;
    int64_t cap;
    int64_t* out_off;  // null, or {0, h} of a batch of one set
    int fp64;
    int sieve;         // larger sets: the sieve may be used
    LocalStatus* status;
};

// One set of at most kLocalMax points on one workgroup.
constexpr int kLocalMax = 65535;
hipError_t launch_local_one(const LocalArgs& a, hipStream_t st);

}  // namespace sqh
