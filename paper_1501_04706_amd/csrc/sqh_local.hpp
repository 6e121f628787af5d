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
    unsigned long long orient, orient_exact, cmp_exact;
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

// A batch of sets (at most kBatchSetMax points each; larger ones leave the
// whole batch to the general path).
constexpr int kBatchSetMax = 1 << 20;
struct Pocket;
struct DenseSet;
struct BatchCtl;
struct BatchArgs {
    const float2* xy;
    const int64_t* set_off;  // null: one set [0, N)
    int N, G;
    int32_t* out;
    int64_t cap;
    int64_t* out_off;        // may be null
    int fp64, sieve;
    LocalStatus* status;
    // workspace
    int* start;        // G + 1: set offsets
    int* hcnt;         // G: hull sizes
    int* order;        // G: sets by size class
    int* hbuf;         // N: each set's hull from its first slot
    float* slots;      // 3 N words: pocket points
    Pocket* pockets;   // pocket records ...
    int* todo[3];      // ... and their indices by solver size
    int pocket_cap;
    float* slots2;     // 3 N words: ring nodes
    DenseSet* dense;
    int dense_cap;
    BatchCtl* ctl;
};
size_t batch_ctl_bytes();
size_t pocket_bytes();
size_t dense_bytes();
hipError_t launch_batch(const BatchArgs& a, int cus, hipStream_t st);

}  // namespace sqh
