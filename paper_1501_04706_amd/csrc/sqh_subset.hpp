// The pre-filter as ordinary launches (device code, gfx950): the host learns
// the subset's size and the sieve or the LDS solve takes the subset.
//
// k_pre_extremes reads the points for the eight extremes, k_pre_keep reads
// them again and appends those that the polygon does not certify inside, with
// their indices. Both are bound by the reads (8 bytes a point each; the second
// writes 12 bytes a kept point). As one cooperative kernel with a workgroup to
// a compute unit and two grid barriers this took 81 us for 5M points of a
// disk, and the general kernel after it 584 us on the 498K kept; these take 14
// and 32 us (42 with twice the workgroups of half the threads: the second waits
// on its reservations, one for 16K points now), and the sieve 82 us for the
// subset.
#pragma once
#include "sqh_prefilter.hpp"
#include "sqh_solve.hpp"

namespace sqh {

constexpr int kPreT = 1024, kPreGrid = 256;
struct PreCtl {
    int keep, pad;
    unsigned int done, pad2;
    unsigned long long t0;
    unsigned long long ext[kPreGrid][8];
    int bad[kPreGrid];
};

// Workgroup b's pairs of points [pb, pe).
__device__ __forceinline__ void pre_share(int n, int b, int nb, int& pb, int& pe)
{
    const int np = (n + 1) >> 1, per = (((np + nb - 1) / nb) + 63) & ~63;
    pb = (int)min((long long)b * per, (long long)np);
    pe = (int)min((long long)pb + per, (long long)np);
}
// U pairs to a thread from pair p on: points 2 q and 2 q + 1 (an odd last one
// twice; past pe any). An 8-byte aligned input is read a point at a time.
template <int U>
__device__ __forceinline__ void pre_pairs(const float2* xy, int n, int p, int pe, float4 (&v)[U])
{
    const int t = (int)threadIdx.x;
    if ((reinterpret_cast<uintptr_t>(xy) & 15u) == 0 && p + kPreT * U <= min(pe, n >> 1)) {
#pragma unroll
        for (int j = 0; j < U; ++j) v[j] = gld(reinterpret_cast<const float4*>(xy) + p + kPreT * j + t);
        return;
    }
#pragma unroll
    for (int j = 0; j < U; ++j) {
        const int q = min(p + kPreT * j + t, pe - 1);
        const float2 u = gld(xy + 2 * (size_t)q), w = gld(xy + min(2 * q + 1, n - 1));
        v[j] = make_float4(u.x, u.y, w.x, w.y);
    }
}

__global__ __launch_bounds__(kPreT) void k_pre_extremes(PreArgs a)
{
    constexpr int U = 4;
    __shared__ unsigned long long best[8];
    __shared__ int s_bad;
    PreCtl* ctl = a.ctl;
    const int t = (int)threadIdx.x, b = (int)blockIdx.x, n = a.n;
    if (t < 8) best[t] = ext_none(t);
    if (t == 0) {
        s_bad = 0;
        if (b == 0) {
            ctl->keep = 0;
            ctl->done = 0u;
            ctl->t0 = wall_clock64();
        }
    }
    int pb, pe;
    pre_share(n, b, (int)gridDim.x, pb, pe);
    ExtLane L;
    L.init();
    bool bad = false;
    for (int p = pb; p < pe; p += kPreT * U) {
        float4 v[U];
        pre_pairs<U>(a.xy, n, p, pe, v);
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int q = p + kPreT * j + t;
            if (q < pe) {
                bad |= !((int)isfinite(v[j].x) & (int)isfinite(v[j].y) & (int)isfinite(v[j].z) & (int)isfinite(v[j].w));
                L.add(v[j].x, v[j].y, 2 * q);
                L.add(v[j].z, v[j].w, min(2 * q + 1, n - 1));
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const uint64_t key = ext_key(k, L.v[k], L.id[k]);
        const uint64_t m = ext_is_max(k) ? wave_max_u64(key) : wave_min_u64(key);
        if (lane_id() == 63) {
            if (ext_is_max(k)) atomicMax(&best[k], (unsigned long long)m);
            else atomicMin(&best[k], (unsigned long long)m);
        }
    }
    if (__ballot(bad) && lane_id() == 0) s_bad = 1;
    __syncthreads();
    if (t < 8) gst(&ctl->ext[b][t], best[t]);
    if (t == 0) ctl->bad[b] = s_bad;
}

__global__ __launch_bounds__(kPreT) void k_pre_keep(PreArgs a, int ne)
{
    constexpr int U = 8;
    __shared__ unsigned long long best[8];
    __shared__ float corner[2][8];
    __shared__ KeepLds keep_lds;
    __shared__ int s_bad, s_cnt, s_base, s_last;
    PreCtl* ctl = a.ctl;
    LocalStatus* st = a.status;
    const int t = (int)threadIdx.x, b = (int)blockIdx.x, n = a.n;
    if (t < 8) best[t] = ext_none(t);
    if (t == 0) { s_bad = 0; s_cnt = 0; }
    __syncthreads();
    {
        const int k = t & 7;
        uint64_t m = ext_none(k);
        for (int e = t >> 3; e < ne; e += kPreT / 8) m = ext_pick(k, m, gld(&ctl->ext[e][k]));
        if (ext_is_max(k)) atomicMax(&best[k], (unsigned long long)m);
        else atomicMin(&best[k], (unsigned long long)m);
        if (t < ne && ctl->bad[t]) s_bad = 1;
    }
    __syncthreads();
    if (s_bad) {
        if (b == 0 && t == 0) {
            st->h = 0;
            st->err = kErrNonFinite;
            st->left = 0;
            st->pre_n = -1;
        }
        return;
    }
    if (t < 8) {
        const float2 c = gld(a.xy + ext_index(t, best[t]));  // n > 0: every direction has a point
        corner[0][t] = c.x;
        corner[1][t] = c.y;
    }
    __syncthreads();
    float cx[8], cy[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        cx[k] = rfl_f(corner[0][k]);
        cy[k] = rfl_f(corner[1][k]);
    }
    KeepEdges E;
    keep_build(E, keep_lds, cx, cy, a.quad != 0);
    __syncthreads();  // keep_lds
    int pb, pe;
    pre_share(n, b, (int)gridDim.x, pb, pe);
    Counters ctr = {0u, 0u, 0u};
    for (int p = pb; p < pe; p += kPreT * U) {
        // 2 U points to a thread, one reservation for all of them
        float4 v[U];
        pre_pairs<U>(a.xy, n, p, pe, v);
        uint32_t keep = 0u;
        int cnt = 0;
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int q = p + kPreT * j + t;
            const bool k0 = q < pe && keep_point(E, keep_lds, v[j].x, v[j].y, ctr);
            const bool k1 = q < pe && 2 * q + 1 < n && keep_point(E, keep_lds, v[j].z, v[j].w, ctr);
            keep |= ((uint32_t)k0 | ((uint32_t)k1 << 1)) << (2 * j);
            cnt += (int)__popcll(__ballot(k0)) + (int)__popcll(__ballot(k1));
        }
        int at = 0;
        if (lane_id() == 0 && cnt) at = atomicAdd(&s_cnt, cnt);
        at = __builtin_amdgcn_readfirstlane(at);
        __syncthreads();
        if (t == 0) {
            s_base = s_cnt ? atomicAdd(&ctl->keep, s_cnt) : 0;
            s_cnt = 0;
        }
        __syncthreads();
        at += s_base;
        if (cnt) {
#pragma unroll
            for (int j = 0; j < 2 * U; ++j) {
                const bool kp = (keep >> j) & 1u;
                const uint64_t M = __ballot(kp);
                if (kp) {
                    const float4 w = v[j >> 1];
                    const int d = at + bits_below(M);
                    gst(a.out_xy + d, (j & 1) ? make_float2(w.z, w.w) : make_float2(w.x, w.y));
                    gst(a.out_id + d, 2 * (p + kPreT * (j >> 1) + t) + (j & 1));
                }
                at += (int)__popcll(M);
            }
        }
    }
    if (!finishes_last(&ctl->done, (int)gridDim.x, &s_last)) return;
    if (t == 0) {
        st->err = 0;
        st->pre_n = __hip_atomic_load(&ctl->keep, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        st->pre_orient = (unsigned long long)n * (unsigned long long)E.n;
        st->pre_t0 = ctl->t0;
        st->pre_t1 = wall_clock64();
    }
}

}  // namespace sqh
