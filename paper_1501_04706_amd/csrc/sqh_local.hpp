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
    int left;   // nothing was written: 1: the ring kernels or the general path have to run; 2: launch_rest
                // has to; 3: the general path has to; 4: the same, and the set is no ring
    int passes;
    int first_v;
    int line;   // the sieve's edges took the static line filter
    unsigned long long orient, orient_exact, cmp_exact;
    unsigned long long t0, t1;  // device clock (100 MHz) at the call's start and end
    int pass_v[kLocalStatPasses], pass_s[kLocalStatPasses];
    // launch_batch: sets that the batch kernels do not take (hcnt -1)
    int refused;
    int64_t refused_points;
    // launch_pre
    int pre_n;  // points kept (-1: a coordinate is not finite)
    unsigned long long pre_orient, pre_t0, pre_t1;
};

// Called before (open) and after every launch of a call.
typedef int (*LaunchMark)(void* ctx, const char* name, int open, hipStream_t st);

// One set of at most kLocalPoints points on one workgroup.
struct LocalArgs {
    const float2* xy;
    const int* ids;  // the points' indices (null: their places)
    int n;
    int32_t* out;
    int64_t cap;
    int fp64;
    LocalStatus* status;
};
hipError_t launch_local_one(const LocalArgs& a, hipStream_t st);

// One set of more than kLocalPoints points past the sieve: the polygon of a
// sample's extreme points, every point against its slabs and edges, and the
// hull of the points left.
struct SieveCtl;
struct SieveArgs {
    const float2* xy;
    const int* ids;    // the points' indices (null: their places) ...
    const float2* all; // ... in this array (else xy)
    int n;
    int32_t* out;
    int64_t cap;
    LocalStatus* status;
    float* X[2];       // n each: points past the slabs, points past the edges
    float* Y[2];
    int* I[2];
    float2* lxy;       // n: chunk hulls
    int* lid;
    int* lcnt;         // n / 64 or more: their sizes
    SieveCtl* ctl;
    // one of an engine's requests (else null): its hull size and bad flag, and
    // what follows (as LocalStatus::left)
    int *h_dev, *bad_dev, *gate;
};
size_t sieve_ctl_bytes();
hipError_t launch_sieve(const SieveArgs& a, int cus, hipStream_t st, LaunchMark mark, void* ctx);
hipError_t launch_rest(const SieveArgs& a, int cus, hipStream_t st, LaunchMark mark, void* ctx);

// The pre-filter of a single set: its subset to out_xy, out_id (n each).
struct PreCtl;
struct PreArgs {
    const float2* xy;
    int n;
    int quad;  // the extremes in x and y only
    float2* out_xy;
    int* out_id;
    LocalStatus* status;
    PreCtl* ctl;
};
size_t pre_ctl_bytes();
hipError_t launch_pre(const PreArgs& a, int cus, hipStream_t st, LaunchMark mark, void* ctx);

// One large ring of points (a set the sieve left).
struct RingCtl;
struct RingPocket;
struct RingArgs {
    const float2* xy;
    const int* ids;      // the points' indices (null: their places)
    int n;
    int32_t* out;
    int64_t cap;
    int line;            // passed on to the status
    LocalStatus* status;
    uint16_t* wid;       // n
    int* off;            // 512 x 512 words
    float4* slots;       // n: points by wedge, then wedge nodes
    float4* slots2;      // n: points by pocket, then pocket nodes
    RingPocket* pockets;
    int pocket_cap;
    RingCtl* ctl;
    int *h_dev, *bad_dev;  // as the sieve's
    const int* gate;       // run only if this is 1
};
size_t ring_ctl_bytes();
hipError_t launch_ring(const RingArgs& a, int cus, hipStream_t st, LaunchMark mark, void* ctx);

// A batch of sets. Those of more than kBatchSetMax points, and those whose ring
// cannot be cut, are refused: the general path takes them as a batch of their
// own (launch_refused_gather, launch_refused_put). If they hold most of the
// points, or the mode has no certificates for sets past one workgroup's LDS, it
// takes the whole batch.
constexpr int kBatchSetMax = 1 << 20;
constexpr int kEngineSetMax = 1 << 18; // an engine's larger requests have launches of their own
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
    int* hcnt;         // G: hull sizes (-1: refused)
    int* order;        // G: sets by size class
    int* hbuf;         // N: each set's hull from its first slot
    float4* slots;     // N: pocket points
    float4* slots2;    // N: ring nodes
    Pocket* pockets;   // pocket records ...
    int* todo[3];      // ... and their indices by solver size
    int pocket_cap;
    DenseSet* dense;
    int dense_cap;
    BatchCtl* ctl;
    // an engine's requests (null for a batch): offsets in place of set_off,
    // where each hull goes in hbuf, a flag for each set with a non-finite
    // coordinate, and the host's copies of sizes and flags. Sets of more than
    // kEngineSetMax points are left out.
    const int *off32, *hpos_src;
    int *hpos, *bad, *h_host, *bad_host;
};
size_t batch_ctl_bytes();
hipError_t launch_batch(const BatchArgs& a, int cus, hipStream_t st);
// (all: the refused sets have their hulls)
hipError_t launch_batch_emit(const BatchArgs& a, int cus, hipStream_t st, int all = 0);
// The refused sets, in order, as a batch: set r is rset[r], its points from
// off[r] on of xy (n of them in g sets, as the status says).
struct RefusedArgs {
    int n, g;
    int* rset;         // g
    int64_t* off;      // g + 1 (3 if g is 1)
    float2* xy;        // n
    const int32_t* out;      // the batch's hulls ...
    const int64_t* out_off;  // ... and their places (g + 1)
};
hipError_t launch_refused_gather(const BatchArgs& a, const RefusedArgs& r, int cus, hipStream_t st);
hipError_t launch_refused_put(const BatchArgs& a, const RefusedArgs& r, int cus, hipStream_t st);

}  // namespace sqh
