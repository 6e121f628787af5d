// The workgroup-local hull kernels (device and launch code, gfx950): small
// single sets, batches, and the launches of the sieve, the pre-filter and the
// ring kernels.
#include <algorithm>

#include "sqh_local.hpp"
#include "sqh_solve.hpp"
#include "sqh_sieve.hpp"
#include "sqh_dense.hpp"

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

// A call's counters, a line to every 32nd workgroup: atomics on one address
// follow each other at 14 ns, so that the counts of some thousand waves took
// longer than the kernels that made them (60 of 94 us of the sieve on a grid,
// 120 of 210 us of a circle's pockets).
constexpr int kCtrSlots = 32;
struct alignas(128) CtrSlot {
    unsigned long long c[3];
};
// Adds the workgroup's counters; sum: three words of LDS, zero before.
__device__ __forceinline__ void ctr_flush(CtrSlot* slots, const Counters& ctr, uint32_t* sum)
{
    counters_sum(ctr, sum);
    __syncthreads();
    const int t = (int)threadIdx.x;
    if (t < 3 && sum[t]) atomicAdd(&slots[(int)blockIdx.x % kCtrSlots].c[t], (unsigned long long)sum[t]);
}
__device__ __forceinline__ unsigned long long ctr_total(const CtrSlot* slots, int i)
{
    unsigned long long v = 0ull;
#pragma unroll
    for (int k = 0; k < kCtrSlots; ++k) v += __hip_atomic_load(&slots[k].c[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return v;
}

}  // namespace sqh
#include "sqh_sieve_large.hpp"
#include "sqh_ring.hpp"
#include "sqh_subset.hpp"
namespace sqh {

// One set of at most P points, the hull to out (first cap vertices), the
// status to the host.
template <int T, int P>
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
    const int cnt = load_points<T, P>(L, a.xy, a.n, a.n, a.ids);
    const int h = L.bad ? kSetBad : (cnt == 0 ? 0 : solve<T, P, true>(L, cnt, 0, 0, a.fp64 != 0, ctr, &st));
    counters_sum(ctr, csum);
    for (int r = t; r < h; r += T)
        if (r < a.cap) gst(a.out + r, L.id[L.ring[r]]);
    __syncthreads();
    LocalStatus* s = a.status;
    if (t < kSolvePasses) {
        s->pass_v[t] = st.pass_v[t];
        s->pass_s[t] = st.pass_s[t];
    }
    if (t == 0) {
        s->h = h > 0 ? h : 0;
        s->err = h == kSetBad ? kErrNonFinite : 0;
        s->left = 0;
        s->passes = st.passes;
        s->first_v = st.pass_v[0];
        s->line = 0;
        s->orient = csum[0];
        s->orient_exact = csum[1];
        s->cmp_exact = csum[2];
        s->t0 = t0;
        s->t1 = wall_clock64();
    }
}

// Up to 1024 points four waves hold the set, up to 4096 sixteen. One ordinary
// launch, status straight to host memory: 124 us a call before (a reset, a
// cooperative launch of every compute unit and a copy back) and 32 us now for
// 1000 points of a square (15 us on the device).
hipError_t launch_local_one(const LocalArgs& a, hipStream_t st)
{
    if (a.n <= kSmallP) k_local_one<kSmallT, kSmallP><<<1, kSmallT, 0, st>>>(a);
    else k_local_one<kMidT, kMidP><<<1, kMidT, 0, st>>>(a);
    return hipGetLastError();
}

// ---- batches ---------------------------------------------------------------

constexpr int kClasses = 6;  // sets of up to 2^10, 2^12, 2^14, 2^16, 2^18, 2^20 points
constexpr int kTasks = 3;  // pocket solvers: a wave, four waves, sixteen
constexpr int kTaskT[kTasks] = {64, 256, 1024}, kTaskP[kTasks] = {kWavePts + 2, 1024, kLocalPoints};

// The solvers' passes, a line or more to every 8th workgroup (as the counters).
constexpr int kStatLines = 8;
struct alignas(128) BatchStats {
    int passes, pass_v[kSolvePasses], pass_s[kSolvePasses];
};
struct BatchCtl {
    int err, left;
    int stop;  // err | left as k_batch_init found them: for kernels that set err themselves
    int n_refused;
    unsigned long long refused_points;
    int n_small, n_big;         // queue lengths: class 0; classes 5 .. 1
    int head_big, n_task[kTasks];
    int n_pocket, n_dense;
    unsigned long long t0;
    CtrSlot ctr[kCtrSlots];
    BatchStats st[kStatLines];
};
static_assert(sizeof(Pocket) == 32, "pockets fit the child records' space");

size_t batch_ctl_bytes() { return sizeof(BatchCtl); }

// A workgroup's share of the batch's counters.
struct BatchAcc {
    SolveStats st;
    uint32_t c[3];
};
__device__ __forceinline__ void acc_init(BatchAcc& A)
{
    stats_clear(A.st);
    if (threadIdx.x < 3) A.c[threadIdx.x] = 0u;
    __syncthreads();
}
__device__ __forceinline__ void acc_flush(BatchAcc& A, const Counters& ctr, BatchCtl* ctl)
{
    ctr_flush(ctl->ctr, ctr, A.c);
    const int t = (int)threadIdx.x;
    BatchStats& S = ctl->st[(int)blockIdx.x % kStatLines];
    if (t < kSolvePasses) {
        if (A.st.pass_v[t]) atomicAdd(&S.pass_v[t], A.st.pass_v[t]);
        if (A.st.pass_s[t]) atomicAdd(&S.pass_s[t], A.st.pass_s[t]);
    }
    if (t == 0 && A.st.passes) atomicMax(&S.passes, A.st.passes);
}

__device__ __forceinline__ int set_class(int n)
{
    return n <= 1 << 10 ? 0 : (n <= 1 << 12 ? 1 : (n <= 1 << 14 ? 2 : (n <= 1 << 16 ? 3 : (n <= 1 << 18 ? 4 : 5))));
}

// The batch's offsets checked and its sets queued by size class, the largest
// first (one workgroup: a few loads per set).
__global__ __launch_bounds__(1024) void k_batch_init(BatchArgs a)
{
    __shared__ int n[kClasses], at[kClasses], s_err, s_left, s_over;
    __shared__ unsigned long long s_over_points;
    const int t = (int)threadIdx.x;
    BatchCtl* ctl = a.ctl;
    for (int i = t; i < (int)(sizeof(BatchCtl) / sizeof(int)); i += 1024) reinterpret_cast<int*>(ctl)[i] = 0;
    if (t < kClasses) n[t] = 0;
    if (t == 0) { s_err = 0; s_left = 0; s_over = 0; s_over_points = 0ull; }
    __syncthreads();
    for (int pass = 0; pass < 2; ++pass) {
        for (int s = t; s < a.G; s += 1024) {
            const int64_t v = a.off32 ? a.off32[s] : (a.set_off ? gld(a.set_off + s) : 0);
            const int64_t w = a.off32 ? a.off32[s + 1] : (a.set_off ? gld(a.set_off + s + 1) : a.N);
            const bool ok = v >= 0 && w >= v && w <= a.N && (s > 0 || v == 0) && (s < a.G - 1 || w == a.N);
            if (pass == 0) {
                if (!ok) { s_err = 1; continue; }
                a.start[s] = (int)v;
                if (s == a.G - 1) a.start[a.G] = (int)w;
                const int m = (int)(w - v);
                a.hcnt[s] = 0;
                if (a.bad) {
                    a.bad[s] = 0;
                    a.hpos[s] = a.hpos_src[s];
                    if (m > kEngineSetMax) continue;
                }
                if (m > kLocalPoints && !a.sieve) s_left = 1;
                if (m > kBatchSetMax) {
                    a.hcnt[s] = -1;
                    atomicAdd(&s_over, 1);
                    atomicAdd(&s_over_points, (unsigned long long)m);
                    continue;
                }
                if (m > 0) atomicAdd(&n[set_class(m)], 1);
            } else {
                const int m = (int)(w - v);
                if (m > 0 && m <= (a.bad ? kEngineSetMax : kBatchSetMax)) a.order[atomicAdd(&at[set_class(m)], 1)] = s;
            }
        }
        __syncthreads();
        if (pass == 0 && (s_err || s_left)) break;
        if (pass == 0 && t == 0) {
            // classes 5, 4, .. 1 make the big queue, class 0 the small one
            int run = 0;
            for (int c = kClasses - 1; c >= 0; --c) {
                at[c] = run;
                run += n[c];
            }
            ctl->n_small = n[0];
            ctl->n_big = run - n[0];
        }
        __syncthreads();
    }
    if (t == 0) {
        const int err = s_err ? kErrBounds : 0;
        const int left = ((s_left || 3 * s_over_points > 2ull * (unsigned long long)a.N) && !s_err) ? 1 : 0;
        ctl->err = err;
        ctl->left = left;
        ctl->stop = err | left;
        ctl->n_refused = s_over;
        ctl->refused_points = s_over_points;
        ctl->t0 = wall_clock64();
    }
}

__device__ __forceinline__ void put_hull(const BatchArgs& a, int s, int base, int h, const int* id, const uint16_t* ring,
                                         int T)
{
    if (h == kSetBad) {
        if (threadIdx.x == 0) {
            if (a.bad) a.bad[s] = 1;
            else atomicOr(&a.ctl->err, kErrNonFinite);
        }
        return;
    }
    int* out = a.hbuf + (a.hpos ? a.hpos[s] : base);
    for (int r = (int)threadIdx.x; r < h; r += T) gst(out + r, id[ring[r]]);
    if (threadIdx.x == 0) a.hcnt[s] = h;  // (a ring's comes later)
}

// Sets of up to kSmallP points, a workgroup each.
__global__ __launch_bounds__(kSmallT, 4) void k_batch_small(BatchArgs a)
{
    __shared__ SolveLds<kSmallP> L;
    __shared__ BatchAcc A;
    const BatchCtl* ctl = a.ctl;
    if (ctl->stop) return;
    Counters ctr = {0u, 0u, 0u};
    acc_init(A);
    const int ns = ctl->n_small, nb = ctl->n_big;
    for (int i = (int)blockIdx.x; i < ns; i += (int)gridDim.x) {
        const int s = a.order[nb + i], base = a.start[s], n = a.start[s + 1] - base;
        if (threadIdx.x == 0) L.bad = 0;
        lds_barrier();
        const int cnt = load_points<kSmallT, kSmallP>(L, a.xy + base, n, n);
        const int h = L.bad ? kSetBad : solve<kSmallT, kSmallP, true>(L, cnt, 0, 0, a.fp64 != 0, ctr, &A.st);
        put_hull(a, s, base, h, L.id, L.ring, kSmallT);
        lds_barrier();
    }
    acc_flush(A, ctr, a.ctl);
}

// A ring of points: cut into pockets for the chain solves that follow.
// False if it cannot be (the set is refused).
template <int T, int P>
__device__ __forceinline__ bool cut_pockets(const BatchArgs& a, SolveLds<P>& L, int h, int s, int base, int n,
                                            Counters& ctr)
{
    static_assert(sizeof(DenseLds) <= offsetof(SolveLds<P>, kmin), "the tables take the solve's space");
    constexpr int U = 4;
    DenseLds& D = *reinterpret_cast<DenseLds*>(&L);
    __shared__ int s_t0, s_d, s_q[kTasks];
    const int t = (int)threadIdx.x;
    const int K = min(min(max(4, n / kDenseTarget), h / 2), kDenseMaxK);
    if (K < 4 || K > kDenseMaxK) return false;
    if (!dense_build<T, P>(L, h, K, D)) return false;
    const float2* xy = a.xy + base;
    bool bad = false;
    // each point's pocket (kept in the ring nodes' space), counted; a step's
    // points are loaded a step ahead
    uint16_t* pid = reinterpret_cast<uint16_t*>(a.slots2 + base);
    float2 nv[U];
    auto fetch = [&](int q0) {
#pragma unroll
        for (int j = 0; j < U; ++j) nv[j] = gld(xy + min(q0 + t + T * j, n - 1));
    };
    fetch(0);
    for (int q0 = 0; q0 < n; q0 += T * U) {
        float2 v[U];
#pragma unroll
        for (int j = 0; j < U; ++j) v[j] = nv[j];
        fetch(q0 + T * U);
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int q = q0 + t + T * j;
            const bool fin = (int)isfinite(v[j].x) & (int)isfinite(v[j].y);
            bad |= !fin;
            if (q < n && fin) {
                const int k = pocket_of(D, K, v[j].x, v[j].y, q, ctr);
                pid[q] = (uint16_t)k;
                if (k >= 0) atomicAdd(&D.cnt[k], 1);
            }
        }
    }
    if (__ballot(bad) && lane_id() == 0) L.bad = 1;
    lds_barrier();
    if (L.bad) return true;
    // slot ranges (one more than its points for v_k), by one wave
    if (t < 64) {
        int run = 0;
        bool over = false;
        for (int k0 = 0; k0 < K; k0 += 64) {
            const int k = k0 + t, c = k < K ? D.cnt[k] + 1 : 0;
            over |= c > kTaskP[kTasks - 1] - 1;
            const int inc = wave_incl_sum(c);
            if (k < K) D.cur[k] = run + inc - c;
            run += __builtin_amdgcn_readlane(inc, 63);
        }
        over = __ballot(over) != 0ull;
        if (t == 0 && over) D.bad = 1;
        if (t == 0 && !over) {
            const int d = atomicAdd(&a.ctl->n_dense, 1);
            s_t0 = atomicAdd(&a.ctl->n_pocket, K);
            const bool fits = s_t0 + K <= a.pocket_cap;
            if (d < a.dense_cap) gst(a.dense + d, DenseSet{s, s_t0, fits ? K : 0, 0, D.c.x, D.c.y, {0, 0}});
            if (d >= a.dense_cap || !fits) D.bad = 1;
            s_d = d;
        }
    }
    lds_barrier();
    if (D.bad) return false;
    // the points to their pockets
    constexpr int V = 8;
    for (int q0 = 0; q0 < n; q0 += T * V) {
        float2 v[V];
        int k[V];
#pragma unroll
        for (int j = 0; j < V; ++j) {
            const int q = min(q0 + t + T * j, n - 1);
            v[j] = gld(xy + q);
            k[j] = pid[q];
        }
#pragma unroll
        for (int j = 0; j < V; ++j) {
            const int q = q0 + t + T * j;
            if (q < n && k[j] < K)
                gst(a.slots + base + atomicAdd(&D.cur[k[j]], 1), make_float4(v[j].x, v[j].y, __int_as_float(q), 0.0f));
        }
    }
    if (t < kTasks) s_q[t] = 0;
    lds_barrier();
    // the pockets' records and, by solver size, their places in its list (one
    // global atomic per list and set)
    auto size_of = [](int len) { return len + 2 <= kTaskP[0] ? 0 : (len + 2 <= kTaskP[1] ? 1 : 2); };
    for (int k = t; k < K; k += T)
        if (D.cnt[k] > 0) atomicAdd(&s_q[size_of(D.cnt[k])], 1);
    lds_barrier();
    if (t < kTasks && s_q[t] > 0) s_q[t] = atomicAdd(&a.ctl->n_task[t], s_q[t]);
    lds_barrier();
    for (int k = t; k < K; k += T) {
        const float2 v = D.v[k], w = D.v[k + 1 < K ? k + 1 : 0];
        const int len = D.cnt[k], off = base + D.cur[k] - len;
        Pocket p;
        p.ax = v.x; p.ay = v.y; p.bx = w.x; p.by = w.y;
        p.aid = D.id[k]; p.off = off; p.len = len; p.ring = s_d;
        if (len == 0) {
            // the vertex alone
            gst(a.slots + off, make_float4(v.x, v.y, __int_as_float(p.aid), 0.0f));
            p.len = 1;
        } else {
            const int c = size_of(len);
            a.todo[c][atomicAdd(&s_q[c], 1)] = s_t0 + k;
        }
        gst(a.pockets + s_t0 + k, p);
    }
    return true;
}

// A set left to the general path.
__device__ __noinline__ void refuse(BatchCtl* ctl, int n)
{
    atomicAdd(&ctl->n_refused, 1);
    atomicAdd(&ctl->refused_points, (unsigned long long)n);
}

// Larger sets, the largest first. (Two workgroups of 512 threads and 2048 points
// to a compute unit, so that one fills the other's waits, took as long, and
// their smaller samples cut less even pockets.)
__global__ __launch_bounds__(kMidT) void k_batch_big(BatchArgs a)
{
    constexpr int T = kMidT, P = kMidP;
    __shared__ SolveLds<P> L;
    __shared__ BatchAcc A;
    __shared__ int s_i;
    BatchCtl* ctl = a.ctl;
    if (ctl->stop) return;
    Counters ctr = {0u, 0u, 0u};
    acc_init(A);
    const int nb = ctl->n_big;
    for (;;) {
        if (threadIdx.x == 0) {
            s_i = atomicAdd(&ctl->head_big, 1);
            L.bad = 0;
        }
        lds_barrier();
        const int i = s_i;
        if (i >= nb) break;
        const int s = a.order[i], base = a.start[s], n = a.start[s + 1] - base;
        int sample = 0;
        int h = solve_set<T, P>(L, a.xy + base, n, a.fp64 != 0, ctr, &A.st, &sample);
        if (h == kSetDense) {
            const bool ok = sample > 0 && cut_pockets<T, P>(a, L, sample, s, base, n, ctr);
            if (L.bad) h = kSetBad;
            else if (ok) h = 0;
            else if (threadIdx.x == 0) refuse(ctl, n);  // (h: -1)
        }
        put_hull(a, s, base, h, L.id, L.ring, T);
        lds_barrier();
    }
    acc_flush(A, ctr, ctl);
}

__device__ __forceinline__ void put_nodes(float4* slot, const float2* xy, const int* id, const uint16_t* ring, int nodes,
                                          int T)
{
    for (int r = (int)threadIdx.x; r < nodes; r += T) {
        const int q = ring[r];
        gst(slot + r, make_float4(xy[q].x, xy[q].y, __int_as_float(id[q]), 0.0f));
    }
}

// The pockets' chains: each pocket's nodes (v_k, then the chain) replace its
// points. Pockets of up to kWavePts points are a wave's, with no barriers.
// Bound by instruction issue: 21M points in 140K pockets take 349 us; the sort's
// exchanges through the LDS crossbar made it 434, QuickHull by waves 1150.
constexpr int kPocketWaves = 4;
__global__ __launch_bounds__(64 * kPocketWaves) void k_batch_pocket(BatchArgs a)
{
    __shared__ WaveLds Ws[kPocketWaves];
    __shared__ uint32_t csum[3];
    BatchCtl* ctl = a.ctl;
    const int nt = ctl->n_task[0];
    if (nt == 0 || (ctl->err | ctl->left)) return;
    if (threadIdx.x < 3) csum[threadIdx.x] = 0u;
    __syncthreads();
    const int lane = lane_id(), w = (int)(threadIdx.x >> 6);
    WaveLds& W = Ws[w];
    Counters ctr = {0u, 0u, 0u};
    for (int i = (int)blockIdx.x * kPocketWaves + w; i < nt; i += (int)gridDim.x * kPocketWaves) {
        const int j = gld(a.todo[0] + i);
        const Pocket p = gld(a.pockets + j);
        const float2 c = make_float2(gld(&a.dense[p.ring].cx), gld(&a.dense[p.ring].cy));
        float4* slot = a.slots + p.off;
#pragma unroll
        for (int r = 0; r < kWavePts / 64; ++r) {
            const int q = lane + 64 * r;
            if (q < p.len) {
                const float4 v = gld(slot + q);
                W.xy[0][q] = make_float2(v.x, v.y);
                W.id[q] = __float_as_int(v.z);
            }
        }
        wave_sync();
        int f;
        const int m = wave_chain<false>(W, p.len, c, make_float2(p.ax, p.ay), make_float2(p.bx, p.by), f, ctr);
        for (int q = lane; q < m; q += 64)
            gst(slot + q + 1, make_float4(W.xy[f][q].x, W.xy[f][q].y, __int_as_float(W.id[W.at[f][q]]), 0.0f));
        if (lane == 0) {
            gst(slot, make_float4(p.ax, p.ay, __int_as_float(p.aid), 0.0f));
            gst(&a.pockets[j].len, m + 1);
        }
        wave_sync();
    }
    ctr_flush(ctl->ctr, ctr, csum);
}

// Larger pockets: the passes.
template <int C>
__global__ __launch_bounds__(kTaskT[C], 4) void k_batch_chain(BatchArgs a)
{
    constexpr int T = kTaskT[C], P = kTaskP[C];
    __shared__ SolveLds<P> L;
    __shared__ BatchAcc A;
    BatchCtl* ctl = a.ctl;
    const int nt = ctl->n_task[C];
    if (nt == 0 || (ctl->err | ctl->left)) return;
    Counters ctr = {0u, 0u, 0u};
    acc_init(A);
    const int t = (int)threadIdx.x;
    for (int i = (int)blockIdx.x; i < nt; i += (int)gridDim.x) {
        const int j = a.todo[C][i];
        const Pocket p = gld(a.pockets + j);
        float4* slot = a.slots + p.off;
        for (int r = t; r < p.len; r += T) {
            const float4 v = gld(slot + r);
            L.xy[r] = make_float2(v.x, v.y);
            L.id[r] = __float_as_int(v.z);
        }
        if (t == 0) {
            L.xy[p.len] = make_float2(p.ax, p.ay);
            L.id[p.len] = p.aid;
            L.xy[p.len + 1] = make_float2(p.bx, p.by);
            L.id[p.len + 1] = -1;
        }
        lds_barrier();
        const int nodes = solve<T, P, false>(L, p.len + 2, p.len, p.len + 1, a.fp64 != 0, ctr, &A.st);
        put_nodes(slot, L.xy, L.id, L.ring, nodes, T);
        if (t == 0) a.pockets[j].len = nodes;
        lds_barrier();
    }
    acc_flush(A, ctr, ctl);
}

// The rings: the pockets' nodes as one list, a workgroup per set, and the
// removal rounds over it until every node is strictly convex; then the hull
// from its lexicographic minimum. 270 us for 1365 rings of 21M points (304 with
// three loads a node; QuickHull over the joined chains took 885).
constexpr int kRingT = 512;
__global__ __launch_bounds__(kRingT) void k_batch_ring(BatchArgs a)
{
    constexpr int W = kRingT / 64;
    __shared__ int s_at[kDenseMaxK + 1], s_off[kDenseMaxK];
    __shared__ int red[W];
    __shared__ int s_start;
    __shared__ unsigned long long s_min;
    __shared__ uint32_t csum[3];
    BatchCtl* ctl = a.ctl;
    if (ctl->err | ctl->left) return;
    if (threadIdx.x < 3) csum[threadIdx.x] = 0u;
    __syncthreads();
    Counters ctr = {0u, 0u, 0u};
    const int t = (int)threadIdx.x, lane = lane_id(), w = t >> 6, nd = ctl->n_dense;
    for (int i = (int)blockIdx.x; i < nd; i += (int)gridDim.x) {
        const DenseSet ds = gld(a.dense + i);
        const int K = ds.k, base = gld(a.start + ds.set);
        if (K == 0) continue;  // (uniform: a refused set)
        for (int k = t; k < K; k += kRingT) {
            s_at[k] = gld(&a.pockets[ds.t0 + k].len);
            s_off[k] = gld(&a.pockets[ds.t0 + k].off);
        }
        if (t == 0) s_min = ~0ull;
        __syncthreads();
        if (w == 0) {
            int run = 0;
            for (int k0 = 0; k0 < K; k0 += 64) {
                const int k = k0 + lane, c = k < K ? s_at[k] : 0;
                const int in = wave_incl_sum(c);
                if (k < K) s_at[k] = run + in - c;
                run += __builtin_amdgcn_readlane(in, 63);
            }
            if (lane == 0) s_at[K] = run;
        }
        __syncthreads();
        int m = s_at[K];
        // two lists of this set's slots: the nodes go from one to the other
        const NodesGlobal list = {{a.slots2 + base, a.slots + base}};
        for (int k = w; k < K; k += W) {
            const float4* src = a.slots + s_off[k];
            const int q0 = s_at[k], len = s_at[k + 1] - q0;
            for (int e = lane; e < len; e += 64) list.put(0, q0 + e, gld(src + e));
        }
        __syncthreads();
        int f;
        m = ring_rounds<kRingT, true>(list, m, make_float2(ds.cx, ds.cy), f, red, ctr);
        uint64_t lo = ~0ull;
        for (int q = t; q < m; q += kRingT) {
            const uint64_t v = lex_key(list.get(f, q));
            lo = v < lo ? v : lo;
        }
        lo = wave_min_u64(lo);
        if (lane == 63) atomicMin(&s_min, (unsigned long long)lo);
        __syncthreads();
        for (int q = t; q < m; q += kRingT)
            if (lex_key(list.get(f, q)) == s_min) s_start = q;  // (one node: the ring's positions differ)
        __syncthreads();
        const int st = s_start;
        int* out = a.hbuf + (a.hpos ? gld(a.hpos + ds.set) : base);
        for (int q = t; q < m; q += kRingT) {
            const int r = q >= st ? q - st : q - st + m;
            gst(out + r, __float_as_int(list.get(f, q).z));
        }
        if (t == 0) a.hcnt[ds.set] = m;
        __syncthreads();
    }
    ctr_flush(ctl->ctr, ctr, csum);
}

// Offsets and hulls to the caller, the status to the host. Workgroup b takes a
// contiguous share of the sets, kEmitT at a time, and copies their hulls as one
// run of the output (each thread finds its element's set by bisection, so
// that one large hull does not hold a wave up).
constexpr int kEmitT = 256;
__global__ __launch_bounds__(kEmitT) void k_batch_emit(BatchArgs a, int all_sets)
{
    constexpr int W = kEmitT / 64;
    __shared__ int red[W];
    __shared__ int s_at[kEmitT], s_src[kEmitT];
    const BatchCtl* ctl = a.ctl;
    const int t = (int)threadIdx.x, lane = lane_id(), w = t >> 6, b = (int)blockIdx.x, nb = (int)gridDim.x;
    // (refused sets of an engine are left out, those of a batch are waited for)
    const int refused = all_sets ? 0 : ctl->n_refused;
    const int bad = ctl->err | ctl->left | (refused && !a.h_host);
    const int per = (a.G + nb - 1) / nb;
    const int s0 = min(b * per, a.G), s1 = min(s0 + per, a.G);
    int run = 0;
    if (!bad) {
        int v = 0;
        for (int s = t; s < s0; s += kEmitT) v += max(gld(a.hcnt + s), 0);
        v = wave_total(v);
        if (lane == 0) red[w] = v;
        __syncthreads();
#pragma unroll
        for (int u = 0; u < W; ++u) run += red[u];
        for (int c0 = s0; c0 < s1; c0 += kEmitT) {
            const int s = c0 + t, hs = s < s1 ? gld(a.hcnt + s) : 0, h = max(hs, 0);
            const int inc = wave_incl_sum(h);
            __syncthreads();
            if (lane == 63) red[w] = inc;
            __syncthreads();
            int before = 0, all = 0;
#pragma unroll
            for (int u = 0; u < W; ++u) {
                before += u < w ? red[u] : 0;
                all += red[u];
            }
            s_at[t] = before + inc - h;
            s_src[t] = s < s1 ? gld((a.hpos ? a.hpos : a.start) + s) : 0;
            if (s < s1 && a.h_host) {
                a.h_host[s] = hs;
                a.bad_host[s] = gld(a.bad + s);
            }
            if (s < s1 && a.out_off) a.out_off[s] = (int64_t)(run + before + inc - h);
            __syncthreads();
            for (int o = t; o < all; o += kEmitT) {
                int l = 0;  // the last set starting at or before o (empty ones share their start with the next)
#pragma unroll
                for (int d = kEmitT / 2; d >= 1; d >>= 1)
                    if (s_at[l + d] <= o) l += d;
                if (run + o < a.cap) gst(a.out + run + o, gld(a.hbuf + s_src[l] + (o - s_at[l])));
            }
            run += all;
        }
    }
    if (b == nb - 1) {
        LocalStatus* s = a.status;
        if (t < kSolvePasses) {
            int v = 0, g = 0, most = 0;
#pragma unroll
            for (int k = 0; k < kStatLines; ++k) {
                v += ctl->st[k].pass_v[t];
                g += ctl->st[k].pass_s[t];
                most = max(most, ctl->st[k].passes);
            }
            s->pass_v[t] = v;
            s->pass_s[t] = g;
            if (t == 0) {
                s->first_v = v;
                s->passes = most;
            }
        }
        if (t == 0) {
            if (!bad && a.out_off) a.out_off[a.G] = run;
            s->h = bad ? 0 : run;
            s->err = ctl->err;
            s->left = ctl->err ? 0 : ctl->left;
            s->refused = (ctl->err | ctl->left) ? 0 : refused;
            s->refused_points = (int64_t)ctl->refused_points;
            s->line = 0;
            s->orient = ctr_total(ctl->ctr, 0);
            s->orient_exact = ctr_total(ctl->ctr, 1);
            s->cmp_exact = ctr_total(ctl->ctr, 2);
            s->t0 = ctl->t0;
            s->t1 = wall_clock64();
        }
    }
}

hipError_t launch_batch(const BatchArgs& a, int cus, hipStream_t st)
{
    k_batch_init<<<1, 1024, 0, st>>>(a);
    if (a.N > kSmallP) k_batch_big<<<std::min(a.G, cus), kMidT, 0, st>>>(a);
    k_batch_small<<<std::min(a.G, 4 * cus), kSmallT, 0, st>>>(a);
    if (a.sieve && a.N > kLocalPoints) {  // (no smaller set is cut into pockets)
        k_batch_chain<2><<<cus, kTaskT[2], 0, st>>>(a);
        k_batch_chain<1><<<4 * cus, kTaskT[1], 0, st>>>(a);
        k_batch_pocket<<<6 * cus, 64 * kPocketWaves, 0, st>>>(a);
        k_batch_ring<<<std::min(a.G, 4 * cus), kRingT, 0, st>>>(a);
    }
    return hipGetLastError();
}
hipError_t launch_batch_emit(const BatchArgs& a, int cus, hipStream_t st, int all)
{
    k_batch_emit<<<std::min((a.G + 3) / 4, 4 * cus), kEmitT, 0, st>>>(a, all);
    return hipGetLastError();
}

// The refused sets' numbers and places, in order (one workgroup).
__global__ __launch_bounds__(1024) void k_refused_plan(BatchArgs a, RefusedArgs r)
{
    __shared__ int red[16];
    const int t = (int)threadIdx.x;
    int g = 0;
    int64_t n = 0;
    for (int s0 = 0; s0 < a.G; s0 += 1024) {
        const int s = s0 + t;
        const bool mine = s < a.G && gld(a.hcnt + s) < 0;
        const int m = mine ? gld(a.start + s + 1) - gld(a.start + s) : 0;
        int sets, points;  // (of 1024 sets: less than 2^31)
        const int k = block_prefix<1024>(mine ? 1 : 0, red, &sets), p = block_prefix<1024>(m, red, &points);
        if (mine) {
            r.rset[g + k] = s;
            r.off[g + k] = n + p;
        }
        g += sets;
        n += points;
    }
    if (t == 0) {
        r.off[g] = n;
        if (g == 1) r.off[2] = n;
    }
}
// Their points back to back.
__global__ __launch_bounds__(256) void k_refused_gather(BatchArgs a, RefusedArgs r)
{
    for (int i = (int)(blockIdx.x * 256 + threadIdx.x); i < r.n; i += (int)(gridDim.x * 256)) {
        int l = 0, u = r.g;
        while (u - l > 1) {
            const int m = (l + u) >> 1;
            if (gld(r.off + m) <= i) l = m;
            else u = m;
        }
        gst(r.xy + i, gld(a.xy + gld(a.start + gld(r.rset + l)) + (i - (int)gld(r.off + l))));
    }
}
// Their hulls to where the batch's are, a workgroup per set.
__global__ __launch_bounds__(256) void k_refused_put(BatchArgs a, RefusedArgs r)
{
    for (int k = (int)blockIdx.x; k < r.g; k += (int)gridDim.x) {
        const int s = gld(r.rset + k), h = (int)(gld(r.out_off + k + 1) - gld(r.out_off + k));
        const int32_t* src = r.out + gld(r.out_off + k);
        int* dst = a.hbuf + gld(a.start + s);
        for (int i = (int)threadIdx.x; i < h; i += 256) gst(dst + i, gld(src + i));
        if (threadIdx.x == 0) a.hcnt[s] = h;
    }
}
hipError_t launch_refused_gather(const BatchArgs& a, const RefusedArgs& r, int cus, hipStream_t st)
{
    k_refused_plan<<<1, 1024, 0, st>>>(a, r);
    k_refused_gather<<<std::min((r.n + 255) / 256, 8 * cus), 256, 0, st>>>(a, r);
    return hipGetLastError();
}
hipError_t launch_refused_put(const BatchArgs& a, const RefusedArgs& r, int cus, hipStream_t st)
{
    k_refused_put<<<std::min(r.g, 4 * cus), 256, 0, st>>>(a, r);
    return hipGetLastError();
}

size_t sieve_ctl_bytes() { return sizeof(SieveCtl); }

// Up to kSieveSmall points one workgroup's sample of 1024 leaves few enough
// points (3.3 % of a disk); the larger sample of up to 128K points leaves
// 0.13 % plus the polygon's own 0.04 %, so up to kSieveMid the sieve's last
// workgroup can solve them, and from there the second polygon is expected.
// The sieve's workgroups take at least 2048 points each. *rest: what k_rest
// needs if the status asks for it (left == 2).
constexpr int kSieveSmall = 100'000, kSieveMid = 1'500'000;
hipError_t launch_sieve(const SieveArgs& a, int cus, hipStream_t st, LaunchMark mark, void* ctx)
{
    const int npairs = a.n >> 1;
    const bool mid = a.n <= kSieveMid;
    const int ns = std::max(1, std::min({mid ? cus : 2 * cus, kSieveGrid, npairs / 1024}));
    const int share = 2 * ((((npairs + ns - 1) / ns) + 63) & ~63);
    auto timed = [&](const char* name, auto&& launch) {
        mark(ctx, name, 1, st);
        launch();
        mark(ctx, name, 0, st);
    };
    const int ne = a.n <= kSieveSmall ? 0 : std::min(kExtremeGrid, cus);
    if (ne) timed("k_extreme", [&] { k_extreme<<<ne, kExtremeT, 0, st>>>(a); });
    timed("k_polygon", [&] { k_polygon<<<1, 1024, 0, st>>>(a, ne); });
    if (mid) {
        timed("k_sieve_solve", [&] { k_sieve_solve<<<ns, kMidT, 0, st>>>(a, share); });
        if (a.gate) k_rest<<<cus, kMidT, 0, st>>>(a, ns, share, 0);
    } else {
        timed("k_sieve", [&] { k_sieve<<<ns, kSieveT, 0, st>>>(a); });
        timed("k_rest", [&] { k_rest<<<std::min(64, cus), kMidT, 0, st>>>(a, ns, share, 1); });
    }
    return hipGetLastError();
}
// The points k_sieve_solve found too many (their second polygon is not there:
// kLocalPoints at a time).
hipError_t launch_rest(const SieveArgs& a, int cus, hipStream_t st, LaunchMark mark, void* ctx)
{
    const int npairs = a.n >> 1, ns = std::max(1, std::min({cus, kSieveGrid, npairs / 1024}));
    const int share = 2 * ((((npairs + ns - 1) / ns) + 63) & ~63);
    mark(ctx, "k_rest", 1, st);
    k_rest<<<cus, kMidT, 0, st>>>(a, ns, share, 0);
    mark(ctx, "k_rest", 0, st);
    return hipGetLastError();
}

size_t pre_ctl_bytes() { return sizeof(PreCtl); }
hipError_t launch_pre(const PreArgs& a, int cus, hipStream_t st, LaunchMark mark, void* ctx)
{
    // (workgroups of at least 4096 points; as few as fill the chip, because their
    // reservations and tickets follow each other at 14 ns)
    const int nb = std::max(1, std::min({cus, kPreGrid, a.n / 4096}));
    mark(ctx, "k_pre_extremes", 1, st);
    k_pre_extremes<<<nb, kPreT, 0, st>>>(a);
    mark(ctx, "k_pre_extremes", 0, st);
    mark(ctx, "k_pre_keep", 1, st);
    k_pre_keep<<<nb, kPreT, 0, st>>>(a, nb);
    mark(ctx, "k_pre_keep", 0, st);
    return hipGetLastError();
}

static_assert(sizeof(RingPocket) == 32, "pockets fit the segments' space");
size_t ring_ctl_bytes() { return sizeof(RingCtl); }

hipError_t launch_ring(const RingArgs& a, int cus, hipStream_t st, LaunchMark mark, void* ctx)
{
    const int nb = std::max(1, std::min({2 * cus, kRingGrid, a.n / 4096}));
    auto timed = [&](const char* name, auto&& launch) {
        mark(ctx, name, 1, st);
        launch();
        mark(ctx, name, 0, st);
    };
    timed("k_ring_rays", [&] { k_ring_rays<<<1, 1024, 0, st>>>(a); });
    timed("k_ring_count", [&] { k_ring_count<<<nb, 1024, 0, st>>>(a); });
    timed("k_ring_scan", [&] { k_ring_scan<<<kRays / 64, 1024, 0, st>>>(a, nb); });
    timed("k_ring_scatter", [&] { k_ring_scatter<<<nb, 1024, 0, st>>>(a); });
    timed("k_ring_cut", [&] { k_ring_cut<<<kRays, 1024, 0, st>>>(a); });
    timed("k_ring_pocket", [&] { k_ring_pocket<<<6 * cus, 64 * kRingWaves, 0, st>>>(a); });
    timed("k_ring_wedge", [&] { k_ring_wedge<<<kRays, kWedgeT, 0, st>>>(a); });
    timed("k_ring_join", [&] { k_ring_join<<<1, 1024, 0, st>>>(a); });
    timed("k_ring_emit", [&] { k_ring_emit<<<64, kRingEmitT, 0, st>>>(a); });
    return hipGetLastError();
}

}  // namespace sqh
