// Hulls computed by one workgroup each: small single sets (device and launch
// code, gfx950).
#include "sqh_local.hpp"
#include "sqh_solve.hpp"
#include "sqh_sieve.hpp"

namespace sqh {

static_assert(kLocalStatPasses == kSolvePasses, "the status holds the solver's passes");

constexpr int kSmallT = 256, kSmallP = 1024;            // small sets: four workgroups to a compute unit
constexpr int kMidT = 1024, kMidP = kLocalPoints;       // the rest

__device__ __forceinline__ void stats_clear(SolveStats& s)
{
    if ((int)threadIdx.x < kSolvePasses) {
        s.pass_v[threadIdx.x] = 0;
        s.pass_s[threadIdx.x] = 0;
    }
    if (threadIdx.x == 0) s.passes = 0;
}

// The counters of every thread, summed over the workgroup into c[0..2] (LDS).
__device__ __forceinline__ void counters_sum(const Counters& ctr, uint32_t* c)
{
    const uint32_t v[3] = {ctr.orient, ctr.orient_exact, ctr.cmp_exact};
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const uint32_t s = (uint32_t)wave_total((int)v[i]);
        if (lane_id() == 0 && s) atomicAdd(&c[i], s);
    }
}

// One set of n points, the hull to out (first cap vertices), the status to
// the host. Sets of more than P points go through the sieve.
template <int T, int P, bool SIEVE>
__global__ __launch_bounds__(T) void k_local_one(LocalArgs a)
{
    __shared__ SolveLds<P> L;
    __shared__ SolveStats st;
    __shared__ uint32_t csum[3];
    const int t = (int)threadIdx.x;
    const unsigned long long t0 = t == 0 ? wall_clock64() : 0ull;
    Counters ctr = {0u, 0u, 0u};
    stats_clear(st);
    if (t < 3) csum[t] = 0u;
    if (t == 0) L.bad = 0;
    __syncthreads();
    const bool f64 = a.fp64 != 0;
    int h;
    if constexpr (SIEVE) {
        h = solve_set<T, P>(L, a.xy, a.n, f64, ctr, &st);
    } else {
        const int cnt = load_points<T, P>(L, a.xy, a.n, a.n);
        h = L.bad ? kSetBad : (cnt == 0 ? 0 : solve<T, P>(L, cnt, true, 0, 0, 0, f64, ctr, &st));
    }
    counters_sum(ctr, csum);
    if (h > 0) {
        for (int r = t; r < h; r += T)
            if (r < a.cap) gst(a.out + r, L.id[L.ring[r]]);
    }
    __syncthreads();
    LocalStatus* s = a.status;
    if (t < kSolvePasses) {
        s->pass_v[t] = st.pass_v[t];
        s->pass_s[t] = st.pass_s[t];
    }
    if (t == 0) {
        s->h = h > 0 ? h : 0;
        s->err = h == kSetBad ? kErrNonFinite : 0;
        s->left = h == kSetDense ? 1 : 0;
        s->passes = st.passes;
        s->first_v = st.pass_v[0];
        s->orient = csum[0];
        s->orient_exact = csum[1];
        s->cmp_exact = csum[2];
        s->t0 = t0;
        s->t1 = wall_clock64();
        if (a.out_off && h >= 0) {
            a.out_off[0] = 0;
            a.out_off[1] = h;
        }
    }
}

// Up to 1024 points four waves hold the set, up to 4096 sixteen; more go past
// the sieve first. One ordinary launch, status straight to host memory: 124 us
// a call before (a reset, a cooperative launch of every compute unit and a
// copy back) and 32 us now for 1000 points of a square (15 us on the device),
// 242 and 68 us for 20,011 points of a disk.
hipError_t launch_local_one(const LocalArgs& a, hipStream_t st)
{
    if (a.n <= kSmallP) k_local_one<kSmallT, kSmallP, false><<<1, kSmallT, 0, st>>>(a);
    else if (a.n <= kMidP) k_local_one<kMidT, kMidP, false><<<1, kMidT, 0, st>>>(a);
    else k_local_one<kMidT, kMidP, true><<<1, kMidT, 0, st>>>(a);
    return hipGetLastError();
}

}  // namespace sqh
