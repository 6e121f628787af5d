// One set of more than kLocalPoints points past the sieve (device code, gfx950).
//
// Ordinary launches that never wait for one another, with one read of the
// input, instead of a stream over it for each of the seed, the split and the
// first compaction and one over the survivors for every pass:
//   k_extreme  the extreme points of a sample in kDirs directions (the paper's
//              first mode, section 4.2, takes the four axis directions)
//   k_polygon  their polygon: its slabs and edges (small sets: the sample too)
//   k_sieve    every point against its slab, the few left against the edges;
//              the extreme points of those left in kDirs2 directions
//   k_rest     those left past the second polygon, and their hull (QuickHull,
//              section 4); many points left: kLocalPoints to a workgroup first
// Sets that leave few points take k_sieve_solve for the last two.
// A set that keeps many points (a ring) is left to other paths.
//
// Bound by the read: k_sieve streams 20M points of a square in 34 us (4.7 TB/s;
// a plain copy reaches 5.1), of a disk in 42 us (more points past the slabs).
// The other kernels are latency: k_extreme 9 us, k_polygon 14, k_rest 37 (square)
// to 64 us (disk), about a third of it the last workgroup's passes. Before, seed,
// split, first compaction and passes took 375 and 560 us a call, now 110 and 149.
// k_sieve_solve takes 32 us for 20K points, 45 for 1M.
#pragma once
#include "sqh_sieve.hpp"
#include "sqh_dense.hpp"

namespace sqh {

constexpr int kSlabs = 1024;       // slabs of a polygon
constexpr int kDirs = 128;         // directions of the sample's polygon
constexpr int kDirs2 = 256;        // ... and of the second one
constexpr int kExtremeGrid = 256;  // workgroups of k_extreme, at most
constexpr int kSieveT = 512;
constexpr int kSieveGrid = 1024;   // workgroups of the sieve, at most
constexpr int kRestOne = 1 << 16;  // up to this many points left one workgroup takes them
constexpr int kRestRaw = 256;      // points of a workgroup's share that are few
constexpr int kRestHull = 1024;    // hulls of more vertices are left to other paths
constexpr int kFlatMost = 1 << 18; // sets of copies or on a line: up to this many points stay

struct SieveCtl {
    int left, err, h, kB, line;
    unsigned int done;
    float Mx, My;
    float x0, y0, sx, sy;  // directions are taken of ((x - x0) sx, (y - y0) sy)
    Slabs slabs;
    unsigned long long t0;
    CtrSlot ctr[kCtrSlots];
    int cnt2[kSieveGrid];  // points each sieve workgroup left
    unsigned long long best2[kDirs2];
    float2 bins[kSlabs];
    float2 ring[kDirs];
    unsigned long long best[kExtremeGrid][kDirs];
};

// Direction j of K as (cos, sin) of 2 pi j / K, scaled. Rounding does not
// matter: the polygon's vertices are points of the set whichever are chosen.
__device__ __forceinline__ float2 direction(int j, int K, float sx, float sy)
{
    float s, c;
    sincospif(2.0f * (float)j / (float)K, &s, &c);
    return make_float2(c * sx, s * sy);
}

// A running extreme: the largest projection, and the point that has it.
struct Extreme {
    float v;
    int id;
    __device__ __forceinline__ void add(float2 u, float x, float y, int i)
    {
        const float p = fmaf(u.x, x, u.y * y);
        const bool t = p > v;
        v = t ? p : v;
        id = t ? i : id;
    }
    __device__ __forceinline__ unsigned long long key() const
    {
        return id < 0 ? 0ull : ((unsigned long long)order_key(v) << 32) | (uint32_t)id;
    }
};

// The extent of 1024 spread points (one per thread, `probe`), which scales the
// directions: x0, y0, sx, sy. lo, hi: two LDS words each, set to ~0 and 0.
struct Frame {
    float x0, y0, sx, sy;
};
__device__ __forceinline__ Frame sample_frame(float2 probe, unsigned int* lo, unsigned int* hi)
{
    const bool ok = (int)isfinite(probe.x) & (int)isfinite(probe.y);
    const uint32_t k[2] = {order_key(probe.x), order_key(probe.y)};
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const uint64_t mn = wave_min_u64(ok ? (uint64_t)k[c] : ~0ull), mx = wave_max_u64(ok ? (uint64_t)k[c] : 0ull);
        if (lane_id() == 63) {
            atomicMin(&lo[c], (unsigned int)min(mn, (uint64_t)~0u));
            atomicMax(&hi[c], (unsigned int)mx);
        }
    }
    __syncthreads();
    auto back = [](uint32_t v) { return __uint_as_float((v & 0x80000000u) ? v ^ 0x80000000u : ~v); };
    Frame f;
    f.x0 = back(lo[0]);
    f.y0 = back(lo[1]);
    const float ex = back(hi[0]) - f.x0, ey = back(hi[1]) - f.y0;
    f.sx = (ex > 0.0f && ex < INFINITY) ? 1.0f / ex : 1.0f;
    f.sy = (ey > 0.0f && ey < INFINITY) ? 1.0f / ey : 1.0f;
    return f;
}

// Extremes of 64 points held one to a lane (p, index id; cnt of them), in the
// directions lane + 64 k: the points are handed out lane by lane and a
// direction never leaves its lane, so there is no reduction across lanes.
template <int D>
__device__ __forceinline__ void wave_extremes(const float2 (&u)[D], Extreme (&e)[D], float x, float y, int id, int cnt)
{
    for (int i = 0; i < cnt; ++i) {
        const float px = rl_f(x, i), py = rl_f(y, i);
        const int pi = rl_i(id, i);
#pragma unroll
        for (int k = 0; k < D; ++k) e[k].add(u[k], px, py, pi);
    }
}
template <int D>
__device__ __forceinline__ void extremes_init(float2 (&u)[D], Extreme (&e)[D], const Frame& f)
{
#pragma unroll
    for (int k = 0; k < D; ++k) {
        u[k] = direction(lane_id() + 64 * k, 64 * D, f.sx, f.sy);
        e[k].v = -INFINITY;
        e[k].id = -1;
    }
}

// Wave number w of nw takes 8 runs of 8 neighbouring points, spread over the
// set: lane l point l % 8 of run l / 8.
__device__ __forceinline__ int sample_place(int n, int w, int nw)
{
    const long long r = (long long)w * 8 + (lane_id() >> 3);
    return min((int)(r * n / ((long long)nw * 8)), n - 8) + (lane_id() & 7);
}

__device__ __forceinline__ void sieve_ctl_init(SieveCtl* ctl, const Frame& f)
{
    const int t = (int)threadIdx.x;
    if (t == 0) {
        ctl->left = 0; ctl->err = 0; ctl->done = 0u;
        ctl->x0 = f.x0; ctl->y0 = f.y0; ctl->sx = f.sx; ctl->sy = f.sy;
    }
    if (t < kDirs2) ctl->best2[t] = 0ull;
    if (t < 3 * kCtrSlots) ctl->ctr[t / 3].c[t % 3] = 0ull;
}

// The extremes of a sample of 64 points per wave.
constexpr int kExtremeT = 512;
__global__ __launch_bounds__(kExtremeT) void k_extreme(SieveArgs a)
{
    __shared__ unsigned int lo[2], hi[2];
    __shared__ unsigned long long best[kDirs];
    const int t = (int)threadIdx.x, lane = lane_id(), b = (int)blockIdx.x, n = a.n;
    SieveCtl* ctl = a.ctl;
    if (b == 0 && t == 0) ctl->t0 = wall_clock64();
    const float2 probe = gld(a.xy + (int)((long long)t * n / kExtremeT));
    const int q = sample_place(n, b * (kExtremeT / 64) + (t >> 6), (int)gridDim.x * (kExtremeT / 64));
    const float2 p = gld(a.xy + q);
    if (t < 2) { lo[t] = ~0u; hi[t] = 0u; }
    if (t < kDirs) best[t] = 0ull;
    __syncthreads();
    const Frame f = sample_frame(probe, lo, hi);
    float2 u[kDirs / 64];
    Extreme e[kDirs / 64];
    extremes_init(u, e, f);
    wave_extremes(u, e, p.x - f.x0, p.y - f.y0, q, 64);
#pragma unroll
    for (int k = 0; k < kDirs / 64; ++k) atomicMax(&best[lane + 64 * k], e[k].key());
    __syncthreads();
    if (t < kDirs) gst(&ctl->best[b][t], best[t]);
    if (b == 0) sieve_ctl_init(ctl, f);
}

// One wave: the points v[0][0 .. n) (extremes in directions that turn
// counter-clockwise) reduced to a strictly convex polygon around a point, by
// the removal rounds of sqh_dense.hpp; counter-clockwise from its
// lexicographic minimum in `out`. Returns its size, or 0 if they do not make
// one. Extremes of rounded projections may come out of order: the polygon is
// used only if every step turns about its centre and all of them turn once.
__device__ __forceinline__ int wave_polygon(float2* v0, float2* v1, int n, float2* out, Counters& ctr)
{
    const int lane = lane_id();
    float2* src = v0;
    float2* dst = v1;
    for (;;) {
        int m = 0;
        for (int i0 = 0; i0 < n; i0 += 64) {
            const int i = i0 + lane;
            bool keep = false;
            float2 p = make_float2(0.0f, 0.0f);
            if (i < n) {
                p = src[i];
                const float2 o = src[i > 0 ? i - 1 : n - 1], q = src[i + 1 < n ? i + 1 : 0];
                const bool copy = p.x == o.x && p.y == o.y, twin = p.x == q.x && p.y == q.y;
                keep = !copy && (twin || orient_of(o, p, q, ctr) > 0);
            }
            const uint64_t M = __ballot(keep);
            if (keep) dst[m + bits_below(M)] = p;
            m += (int)__popcll(M);
        }
        wave_sync();
        float2* s = src;
        src = dst;
        dst = s;
        if (m == n || m < 3) { n = m; break; }
        n = m;
    }
    if (n < 3) return 0;
    const float2 a = src[0], b = src[n / 3], d = src[2 * n / 3];
    const float2 c = make_float2((float)(((double)a.x + (double)b.x + (double)d.x) / 3.0),
                                 (float)(((double)a.y + (double)b.y + (double)d.y) / 3.0));
    bool bad = false;
    int up = 0;
    uint64_t lo = ~0ull;
    int at = 0;
    for (int i = lane; i < n; i += 64) {
        const float2 p = src[i], q = src[i + 1 < n ? i + 1 : 0];
        bad |= orient_exact(c.x, c.y, p.x, p.y, q.x, q.y) <= 0;
        up += p.y < c.y && q.y >= c.y;
        const uint64_t k = ((uint64_t)order_key(p.x + 0.0f) << 32) | order_key(p.y + 0.0f);
        if (k < lo) { lo = k; at = i; }
    }
    if (__ballot(bad) || wave_total(up) != 1) return 0;
    const uint64_t mn = wave_min_u64(lo);
    const uint64_t first = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(mn >> 32), 63) << 32) |
                           (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)mn, 63);
    const uint64_t who = __ballot(lo == first);
    const int st = __builtin_amdgcn_readlane(at, (int)__builtin_ctzll(who));
    for (int i = lane; i < n; i += 64) {
        const int r = i >= st ? i - st : i - st + n;
        out[r] = src[i];
    }
    wave_sync();
    return n;
}

// y extent and |x|, |y| bounds of a polygon (one wave's work, all lanes get it).
__device__ __forceinline__ void wave_extent(const float2* v, int h, float& mx, float& my, float& ext)
{
    float xl = INFINITY, xh = -INFINITY, yl = INFINITY, yh = -INFINITY;
    for (int i = lane_id(); i < h; i += 64) {
        xl = fminf(xl, v[i].x); xh = fmaxf(xh, v[i].x);
        yl = fminf(yl, v[i].y); yh = fmaxf(yh, v[i].y);
    }
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
        xl = fminf(xl, __shfl_xor(xl, m)); xh = fmaxf(xh, __shfl_xor(xh, m));
        yl = fminf(yl, __shfl_xor(yl, m)); yh = fmaxf(yh, __shfl_xor(yh, m));
    }
    mx = fmaxf(fabsf(xl), fabsf(xh));
    my = fmaxf(fabsf(yl), fabsf(yh));
    ext = fmaxf(xh - xl, yh - yl);
}

// The static line filter's domain: |coordinates| at most 2^60 and not far from
// the origin compared with the extent.
__device__ __forceinline__ bool line_domain(float mx, float my, float ext)
{
    return fmaxf(mx, my) <= 0x1p60f && mx <= 8.0f * ext && my <= 8.0f * ext;
}

// The polygon of a sample's extremes. ne > 0: those k_extreme left; ne == 0:
// the sample (64 points per wave) is taken here, for sets so small that one
// workgroup's 1024 points sieve them well enough.
__global__ __launch_bounds__(1024) void k_polygon(SieveArgs a, int ne)
{
    __shared__ unsigned long long best[kDirs];
    __shared__ unsigned int lo[2], hi[2];
    __shared__ float2 v[3][kDirs];
    __shared__ float2 bins[kSlabs];
    __shared__ int s_h, s_kb, s_line, s_keep, s_new;
    __shared__ float s_m[2];
    SieveCtl* ctl = a.ctl;
    const int t = (int)threadIdx.x, lane = lane_id();
    const unsigned long long t0 = wall_clock64();
    Counters ctr = {0u, 0u, 0u};
    const float2 probe = gld(a.xy + (int)((long long)t * a.n / 1024));
    if (t < kDirs) best[t] = 0ull;
    if (t < 2) { lo[t] = ~0u; hi[t] = 0u; }
    if (t == 0) { s_keep = 0; s_new = 0; }
    if (ne > 0) {
        __syncthreads();
        unsigned long long k = 0ull;
        constexpr int W = 1024 / kDirs, U = 8;
        for (int b = t / kDirs; b < ne; b += W * U) {
            unsigned long long o[U];
#pragma unroll
            for (int j = 0; j < U; ++j) o[j] = gld(&ctl->best[min(b + W * j, ne - 1)][t % kDirs]);
#pragma unroll
            for (int j = 0; j < U; ++j) k = o[j] > k ? o[j] : k;
        }
        atomicMax(&best[t % kDirs], k);
    } else {
        const int q = sample_place(a.n, t >> 6, 16);
        const float2 p = gld(a.xy + q);
        __syncthreads();
        const Frame f = sample_frame(probe, lo, hi);
        float2 u[kDirs / 64];
        Extreme e[kDirs / 64];
        extremes_init(u, e, f);
        wave_extremes(u, e, p.x - f.x0, p.y - f.y0, q, 64);
#pragma unroll
        for (int k = 0; k < kDirs / 64; ++k) atomicMax(&best[lane + 64 * k], e[k].key());
        sieve_ctl_init(ctl, f);
        if (t == 0) ctl->t0 = t0;
    }
    __syncthreads();
    if (t < 64) {
        // (the id of a direction without a finite projection is 0: any point will do)
        v[0][lane] = gld(a.xy + (uint32_t)best[lane]);
        v[0][lane + 64] = gld(a.xy + (uint32_t)best[lane + 64]);
        wave_sync();
        const bool fin = (int)isfinite(v[0][lane].x) & (int)isfinite(v[0][lane].y) & (int)isfinite(v[0][lane + 64].x) &
                         (int)isfinite(v[0][lane + 64].y);
        // (a non-finite coordinate is reported by the sieve, which sees every point)
        const int h = __ballot(!fin) ? 0 : wave_polygon(v[0], v[1], kDirs, v[2], ctr);
        float mx, my, ext;
        wave_extent(v[2], h, mx, my, ext);
        if (lane == 0) {
            s_h = h;
            s_m[0] = mx; s_m[1] = my;
            s_line = h >= 3 && line_domain(mx, my, ext);
        }
    }
    __syncthreads();
    const int h = s_h;
    const Slabs sl = build_slabs<1024>(v[2], h, bins, kSlabs, &s_kb);
    gst(ctl->bins + t, bins[t]);
    if (t < h) gst(ctl->ring + t, v[2][t]);
    // how many of 1024 spread points it keeps: a ring of points is not for it
    const bool kp = !slab_inside(sl, bins, probe.x, probe.y) &&
                    !(h >= 3 && chain_inside(v[2], h, s_kb, s_line != 0, s_m[0], s_m[1], probe.x, probe.y,
                                             ctr.orient_exact));
    const uint64_t M = __ballot(kp);
    if (lane == 0) atomicAdd(&s_keep, (int)__popcll(M));
    __syncthreads();
    // ... and, where it matters, how many of those are no copies of its vertices
    if (s_keep > 256) {  // (uniform)
        const bool copy = kp && h >= 3 && chain_copy(v[2], h, s_kb, probe.x, probe.y);
        const uint64_t N = __ballot(kp && !copy);
        if (lane == 0) atomicAdd(&s_new, (int)__popcll(N));
        __syncthreads();
    }
    if (t == 0) {
        ctl->h = h;
        ctl->kB = s_kb;
        ctl->line = s_line;
        ctl->Mx = s_m[0];
        ctl->My = s_m[1];
        ctl->slabs = sl;
        // (three quarters of a ring or an arc are kept, and the ring kernels take
        // it; between the two the general path is the better guess)
        if (h >= 3 && s_new > 256) ctl->left = s_new > 768 ? 1 : 3;
        // what stays are copies, or there is no polygon (points on a line): kMidP
        // at a time that takes 150 us for 1M points of one position and 4 ms for
        // 20M, the general path 70 and 90
        else if (s_keep > 256 && a.n > kFlatMost) ctl->left = 4;
    }
}
static_assert(kSlabs == 1024, "a thread of k_polygon per slab");

// The hulls of chunks c0, c0 + 1, .. (sizes cnt) gathered in L; returns the
// number of points, and in *next the first chunk that did not fit.
template <int T, int P>
__device__ __forceinline__ int gather_hulls(SolveLds<P>& L, const SieveArgs& a, const int* cnt, int c0, int nc, int at,
                                            int* s_next, int* s_at)
{
    const int t = (int)threadIdx.x;
    // one wave finds the places, 64 chunks at a time
    int c = c0;
    for (;;) {
        lds_barrier();
        if (t < 64) {
            const int k = c + t, n = k < nc ? max(gld(cnt + k), 0) : 0;
            const int end = at + wave_incl_sum(n);
            const uint64_t over = __ballot(end > P);
            const int fit = over ? __builtin_ctzll(over) : 64;
            s_at[t] = end - n;
            if (t == 0) s_next[0] = fit;
            if (t == (fit > 0 ? fit - 1 : 0)) s_next[1] = fit > 0 ? end : at;
        }
        lds_barrier();
        const int fit = min(s_next[0], nc - c), end = s_next[1];
        // a wave copies a chunk's hull
        for (int k = t >> 6; k < fit; k += T / 64) {
            const int n = max(gld(cnt + c + k), 0), d = s_at[k];
            for (int r = t & 63; r < n; r += 64) {
                L.xy[d + r] = gld(a.lxy + (size_t)(c + k) * P + r);
                L.id[d + r] = gld(a.lid + (size_t)(c + k) * P + r);
            }
        }
        at = end;
        c += fit;
        if (c >= nc || fit < 64) break;
    }
    lds_barrier();
    if (t == 0) s_next[0] = c;
    lds_barrier();
    return at;
}

// Where each of ns sieve workgroups' points start among all points left (pre,
// ns + 1 LDS words); a share of `per` points per workgroup.
template <int T>
__device__ __forceinline__ int rest_places(const SieveCtl* ctl, int ns, bool none, int* pre)
{
    const int t = (int)threadIdx.x;
    for (int k = t; k < ns; k += T)
        pre[k] = none ? 0 : __hip_atomic_load(&ctl->cnt2[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    if (t < 64) {
        int run = 0;
        for (int k0 = 0; k0 < ns; k0 += 64) {
            const int c = k0 + t < ns ? pre[k0 + t] : 0;
            const int in = wave_incl_sum(c);
            if (k0 + t < ns) pre[k0 + t] = run + in - c;
            run += __builtin_amdgcn_readlane(in, 63);
        }
        if (t == 0) pre[ns] = run;
    }
    __syncthreads();
    return pre[ns];
}
// The place of point i of those left (shares start as the sieve placed them).
__device__ __forceinline__ size_t rest_place(const int* pre, int ns, int per, int n, int i)
{
    int l = 0, u = ns;  // the last workgroup starting at or before the point
    while (u - l > 1) {
        const int m = (l + u) >> 1;
        if (pre[m] <= i) l = m;
        else u = m;
    }
    return (size_t)min((long long)l * per, (long long)(n & ~1)) + (i - pre[l]);
}

// True on the workgroup that finishes last of nb, with the others' writes
// visible. s_last: one LDS word.
__device__ __forceinline__ bool finishes_last(unsigned int* done, int nb, int* s_last)
{
    __syncthreads();
    if (threadIdx.x == 0) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        const unsigned int k = __hip_atomic_fetch_add(done, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *s_last = k == (unsigned int)nb - 1u;
        if (*s_last) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    }
    __syncthreads();
    return *s_last != 0;
}

// The call's end: the hull L.ring[0 .. h) (h < 0, or more than kRestHull
// vertices: left to other paths) and the status. One workgroup.
template <int T, int P>
__device__ __forceinline__ void rest_finish(const SieveArgs& a, SolveLds<P>& L, int h, int M, const SolveStats& st,
                                            const Counters& ctr, uint32_t* csum)
{
    SieveCtl* ctl = a.ctl;
    const int t = (int)threadIdx.x;
    const int err = __hip_atomic_load(&ctl->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const bool left = ctl->left || h < 0 || h > kRestHull;
    const int hh = (err || left) ? 0 : h;
    for (int r = t; r < hh; r += T)
        if (r < a.cap) gst(a.out + r, L.id[L.ring[r]]);
    counters_sum(ctr, csum);
    __syncthreads();
    LocalStatus* s = a.status;
    if (t < kSolvePasses) {
        s->pass_v[t] = st.pass_v[t];
        s->pass_s[t] = st.pass_s[t];
    }
    if (t == 0) {
        s->h = hh;
        s->err = err;
        const int code = (!err && left) ? (ctl->left ? ctl->left : 1) : 0;
        s->left = code;
        s->passes = st.passes;
        s->first_v = M;
        s->line = ctl->line;
        // one side test per point of the sieve (which did not run if k_polygon left the set)
        const unsigned long long sum[3] = {csum[0] + (ctl->left ? 0ull : (unsigned long long)a.n), csum[1], csum[2]};
        s->orient = ctr_total(ctl->ctr, 0) + sum[0];
        s->orient_exact = ctr_total(ctl->ctr, 1) + sum[1];
        s->cmp_exact = ctr_total(ctl->ctr, 2) + sum[2];
        if (code)  // (the ring kernels go on from these)
            for (int i = 0; i < 3; ++i) atomicAdd(&ctl->ctr[0].c[i], sum[i]);
        s->t0 = ctl->t0;
        s->t1 = wall_clock64();
        if (a.gate) {
            *a.h_dev = hh;
            *a.bad_dev = err != 0;
            *a.gate = code;
        }
    }
}

// What a sieve workgroup keeps in LDS.
struct SieveLds {
    float2 bins[kSlabs];
    float2 ring[kDirs];
    unsigned long long best[kDirs2];
};

// The one read of the input. Workgroup b takes a contiguous share of whole
// rows of point pairs; its points left go to the same places of the work
// buffers (from the share's first), so that no workgroup waits or counts for
// another.
template <int T>
__device__ __forceinline__ void sieve_share(const SieveArgs& a, SieveLds& S, int* s_cnt)
{
    constexpr int U = 4;  // pairs per thread and step
    SieveCtl* ctl = a.ctl;
    const int t = (int)threadIdx.x, lane = lane_id(), b = (int)blockIdx.x, nb = (int)gridDim.x, n = a.n;
    const int npairs = n >> 1;  // (an odd last point is handled by the last workgroup)
    const int per = (((npairs + nb - 1) / nb) + 63) & ~63;
    const int pb = (int)min((long long)b * per, (long long)npairs), pe = min(pb + per, npairs);
    const int first = 2 * pb;
    // (an 8-byte aligned input is read a point at a time)
    const bool wide = (reinterpret_cast<uintptr_t>(a.xy) & 15u) == 0;
    auto pair = [&](int p) {
        if (wide) return gld(reinterpret_cast<const float4*>(a.xy) + p);
        const float2 u = gld(a.xy + 2 * (size_t)p), v = gld(a.xy + 2 * (size_t)p + 1);
        return make_float4(u.x, u.y, v.x, v.y);
    };
    float4 nv[U];
    auto fetch = [&](int p) {
        if (p + T * U <= pe) {
#pragma unroll
            for (int j = 0; j < U; ++j) nv[j] = pair(p + T * j + t);
        } else if (p < pe) {
#pragma unroll
            for (int j = 0; j < U; ++j) nv[j] = pair(min(p + T * j + t, pe - 1));
        }
    };
    fetch(pb);  // (in flight while the tables load)
    const Slabs sl = ctl->slabs;
    const int h = ctl->h, kB = ctl->kB, line = ctl->line;
    const float Mx = ctl->Mx, My = ctl->My;
    for (int i = t; i < kSlabs; i += T) S.bins[i] = gld(ctl->bins + i);
    if (t < h) S.ring[t] = gld(ctl->ring + t);
    if (t < kDirs2) S.best[t] = 0ull;
    if (t < 4) s_cnt[t] = 0;  // points past the slabs, past the edges; non-finite; exact tests
    uint32_t n_exact = 0u;
    __syncthreads();
    bool bad = false;
    for (int p = pb; p < pe; p += T * U) {
        float4 v[U];
        uint32_t keep = 0u;
#pragma unroll
        for (int j = 0; j < U; ++j) v[j] = nv[j];
        fetch(p + T * U);
#pragma unroll
        for (int j = 0; j < U; ++j) {
            keep |= (uint32_t)!slab_inside(sl, S.bins, v[j].x, v[j].y) << (2 * j);
            keep |= (uint32_t)!slab_inside(sl, S.bins, v[j].z, v[j].w) << (2 * j + 1);
        }
        if (p + T * U > pe) {
#pragma unroll
            for (int j = 0; j < U; ++j)
                if (p + T * j + t >= pe) keep &= ~(3u << (2 * j));
        }
        if (!__ballot(keep != 0u)) continue;
        // one reservation for the wave, then its points row by row
        int cnt = 0;
#pragma unroll
        for (int j = 0; j < 2 * U; ++j) cnt += (int)__popcll(__ballot((keep >> j) & 1u));
        int at = 0;
        if (lane == 0) at = atomicAdd(&s_cnt[0], cnt);
        at = first + __builtin_amdgcn_readfirstlane(at);
#pragma unroll
        for (int j = 0; j < 2 * U; ++j) {
            const bool kp = (keep >> j) & 1u;
            const uint64_t M = __ballot(kp);
            if (kp) {
                const float x = (j & 1) ? v[j >> 1].z : v[j >> 1].x, y = (j & 1) ? v[j >> 1].w : v[j >> 1].y;
                // (a non-finite coordinate is inside no slab)
                bad |= !((int)isfinite(x) & (int)isfinite(y));
                const int d = at + bits_below(M);
                gst(a.X[0] + d, x);
                gst(a.Y[0] + d, y);
                const int q = 2 * (p + T * (j >> 1) + t) + (j & 1);
                gst(a.I[0] + d, a.ids ? gld(a.ids + q) : q);
            }
            at += (int)__popcll(M);
        }
    }
    if ((n & 1) && b == nb - 1 && t == 0) {
        const float2 v = gld(a.xy + n - 1);
        if (!slab_inside(sl, S.bins, v.x, v.y)) {
            bad |= !((int)isfinite(v.x) & (int)isfinite(v.y));
            const int d = first + atomicAdd(&s_cnt[0], 1);
            gst(a.X[0] + d, v.x);
            gst(a.Y[0] + d, v.y);
            gst(a.I[0] + d, a.ids ? gld(a.ids + n - 1) : n - 1);
        }
    }
    if (__ballot(bad) && lane == 0) s_cnt[2] = 1;
    __syncthreads();
    // the points past the slabs against the edges (written by this workgroup:
    // the barrier orders them)
    const int m = s_cnt[0];
    for (int i0 = 0; i0 < m; i0 += T) {
        const int i = i0 + t;
        float x = 0.0f, y = 0.0f;
        int id = 0;
        if (i < m) { x = gld(a.X[0] + first + i); y = gld(a.Y[0] + first + i); id = gld(a.I[0] + first + i); }
        const bool kp = i < m && !(h >= 3 && chain_inside(S.ring, h, kB, line != 0, Mx, My, x, y, n_exact));
        const uint64_t M = __ballot(kp);
        if (!M) continue;
        int at = 0;
        if (lane == 0) at = atomicAdd(&s_cnt[1], (int)__popcll(M));
        at = __builtin_amdgcn_readfirstlane(at);
        if (kp) {
            const int d = first + at + bits_below(M);
            gst(a.X[1] + d, x);
            gst(a.Y[1] + d, y);
            gst(a.I[1] + d, id);
        }
    }
    n_exact = (uint32_t)wave_total((int)n_exact);
    if (lane == 0 && n_exact) atomicAdd(&s_cnt[3], (int)n_exact);
    __syncthreads();
    if (t == 0) {
        if (s_cnt[3]) atomicAdd(&ctl->ctr[b % kCtrSlots].c[1], (unsigned long long)s_cnt[3]);
        __hip_atomic_store(&ctl->cnt2[b], s_cnt[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (s_cnt[2]) atomicOr(&ctl->err, kErrNonFinite);
    }
}

// Large sets: the share, then the extremes of its points left, for the second
// polygon.
__global__ __launch_bounds__(kSieveT, 4) void k_sieve(SieveArgs a)
{
    __shared__ SieveLds S;
    __shared__ int s_cnt[4];
    SieveCtl* ctl = a.ctl;
    if (ctl->left) return;
    sieve_share<kSieveT>(a, S, s_cnt);
    const int t = (int)threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int left = s_cnt[1];
    if (left == 0) return;
    const int npairs = a.n >> 1, nb = (int)gridDim.x, per = (((npairs + nb - 1) / nb) + 63) & ~63;
    const int first = 2 * (int)min((long long)blockIdx.x * per, (long long)npairs);
    const Frame f = {ctl->x0, ctl->y0, ctl->sx, ctl->sy};
    float2 u[kDirs2 / 64];
    Extreme e[kDirs2 / 64];
    extremes_init(u, e, f);
    // at most 512 of them, spread: up to 64 to a wave
    const int step = (left + 511) / 512, take = (left + step - 1) / step, each = (take + 7) / 8;
    const int i0 = w * each, cnt = max(min(each, take - i0), 0);
    float x = 0.0f, y = 0.0f;
    int id = 0;
    if (lane < cnt) {
        const int d = first + (i0 + lane) * step;
        x = gld(a.X[1] + d) - f.x0;
        y = gld(a.Y[1] + d) - f.y0;
        id = gld(a.I[1] + d);
    }
    wave_extremes(u, e, x, y, id, cnt);
#pragma unroll
    for (int k = 0; k < kDirs2 / 64; ++k) atomicMax(&S.best[lane + 64 * k], e[k].key());
    __syncthreads();
    if (t < kDirs2) {
        const unsigned long long k = S.best[t];
        if (k > __hip_atomic_load(&ctl->best2[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(&ctl->best2[t], k);
    }
}
static_assert(kSieveT == 512 && kDirs2 <= kSieveT, "eight waves take the points left");

// The points left, at most kMidP of them, and their hull, by one workgroup.
template <int T, int P>
__device__ __forceinline__ int rest_solve(const SieveArgs& a, SolveLds<P>& L, const int* pre, int ns, int per, int M,
                                          Counters& ctr, SolveStats* st)
{
    for (int i = (int)threadIdx.x; i < M; i += T) {
        const size_t d = rest_place(pre, ns, per, a.n, i);
        L.xy[i] = make_float2(gld(a.X[1] + d), gld(a.Y[1] + d));
        L.id[i] = gld(a.I[1] + d);
    }
    lds_barrier();
    return solve<T, P, true>(L, M, 0, 0, false, ctr, st);
}

// Smaller sets: the share, and the last workgroup solves the points left (more
// than kMidP of them are k_rest's).
__global__ __launch_bounds__(kMidT) void k_sieve_solve(SieveArgs a, int per)
{
    __shared__ SolveLds<kMidP> L;
    __shared__ SolveStats st;
    __shared__ uint32_t csum[3];
    __shared__ int s_cnt[4], s_last;
    static_assert(sizeof(SieveLds) <= sizeof(L.bins), "the tables take the solve's keys' space");
    const int t = (int)threadIdx.x, nb = (int)gridDim.x;
    SieveCtl* ctl = a.ctl;
    if (ctl->left) {
        if (blockIdx.x == 0 && t == 0) {
            LocalStatus* s = a.status;
            s->left = ctl->left;
            s->err = 0;
            s->line = ctl->line;
            s->orient = s->orient_exact = s->cmp_exact = 0ull;
            s->t0 = ctl->t0;
            s->t1 = wall_clock64();
            if (a.gate) *a.gate = ctl->left;
        }
        return;
    }
    sieve_share<kMidT>(a, *reinterpret_cast<SieveLds*>(&L.bins[0]), s_cnt);
    if (!finishes_last(&ctl->done, nb, &s_last)) return;
    stats_clear(st);
    if (t < 3) csum[t] = 0u;
    Counters ctr = {0u, 0u, 0u};
    int* pre = reinterpret_cast<int*>(&L.seg[0][0]);  // (free until the solve; nb + 1 words)
    static_assert(sizeof(L.seg) >= sizeof(int) * (kSieveGrid + 1), "the places fit");
    const int err = __hip_atomic_load(&ctl->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const int M = rest_places<kMidT>(ctl, nb, err != 0, pre);
    if (M > kMidP) {  // (uniform) k_rest takes them
        if (t == 0) {
            ctl->done = 0u;
            a.status->left = 2;
            if (a.gate) *a.gate = 2;
        }
        return;
    }
    const int h = M > 0 ? rest_solve<kMidT, kMidP>(a, L, pre, nb, per, M, ctr, &st) : 0;
    rest_finish<kMidT, kMidP>(a, L, h, M, st, ctr, csum);
}

// The points left by ns sieve workgroups: at most kMidP of them solved by one
// workgroup; at most kRestOne past the second polygon first (where the sieve
// left its extremes); more, kLocalPoints at a time. The last workgroup to finish solves what remains.
__global__ __launch_bounds__(kMidT) void k_rest(SieveArgs a, int ns, int per, int second)
{
    __shared__ SolveLds<kMidP> L;
    __shared__ SolveStats st;
    __shared__ uint32_t csum[3];
    __shared__ int s_pre[kSieveGrid + 1], s_at[64], s_next[2], s_last;
    __shared__ float s_m[2];
    SieveCtl* ctl = a.ctl;
    const int t = (int)threadIdx.x, lane = lane_id(), b = (int)blockIdx.x, nb = (int)gridDim.x;
    if (a.gate && !second && *a.gate != 2) return;
    const int none = ctl->left | ctl->err;
    stats_clear(st);
    if (t < 3) csum[t] = 0u;
    const int M = rest_places<kMidT>(ctl, ns, none != 0, s_pre);
    Counters ctr = {0u, 0u, 0u};
    if (M <= kMidP) {
        if (b != 0) return;
        const int h = M > 0 ? rest_solve<kMidT, kMidP>(a, L, s_pre, ns, per, M, ctr, &st) : 0;
        rest_finish<kMidT, kMidP>(a, L, h, M, st, ctr, csum);
        return;
    }
    const bool thin = second && M <= kRestOne;
    const int nc = thin ? nb : (M + kMidP - 1) / kMidP;
    for (int c = b; c < nc; c += nb) {
        int cnt;
        lds_barrier();
        if (thin) {
            // workgroup b's share against the second polygon (one list each)
            float2* v = L.bins;  // (free between solves)
            const float2* all = a.ids ? a.all : a.xy;
            if (t < 64) {
#pragma unroll
                for (int k = 0; k < kDirs2 / 64; ++k) v[lane + 64 * k] = gld(all + (uint32_t)ctl->best2[lane + 64 * k]);
                wave_sync();
                const int p = wave_polygon(v, v + kDirs2, kDirs2, v + 2 * kDirs2, ctr);
                float mx, my, ext;
                wave_extent(v + 2 * kDirs2, p, mx, my, ext);
                uint64_t hi = 0ull;
                int at = 0;
                for (int i = lane; i < p; i += 64) {
                    const float2 q = v[2 * kDirs2 + i];
                    const uint64_t k = ((uint64_t)order_key(q.x + 0.0f) << 32) | order_key(q.y + 0.0f);
                    if (k > hi) { hi = k; at = i; }
                }
                const uint64_t top = wave_max_u64(hi);
                if (lane == 63) { s_m[0] = mx; s_m[1] = my; s_at[0] = 0; s_at[1] = p >= 3 && line_domain(mx, my, ext); s_next[0] = p; }
                const uint64_t who = __ballot(hi == (((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(top >> 32), 63) << 32) |
                                                     (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)top, 63)));
                if (lane == (int)__builtin_ctzll(who)) s_next[1] = at;  // the lexicographic maximum
            }
            __syncthreads();
            const int p = s_next[0], kB = s_next[1];
            const bool line = s_at[1] != 0;
            const float mx = s_m[0], my = s_m[1];
            for (int i0 = b * kMidT; i0 < M; i0 += nb * kMidT) {
                const int i = i0 + t;
                const size_t d = rest_place(s_pre, ns, per, a.n, min(i, M - 1));
                const float2 q = make_float2(gld(a.X[1] + d), gld(a.Y[1] + d));
                const int id = gld(a.I[1] + d);
                const bool kp = i < M && !(p >= 3 && chain_inside(v + 2 * kDirs2, p, kB, line, mx, my, q.x, q.y,
                                                                  ctr.orient_exact));
                const uint64_t K = __ballot(kp);
                if (!K) continue;
                int at = 0;
                if (lane == 0) at = atomicAdd(&s_at[0], (int)__popcll(K));
                at = __builtin_amdgcn_readfirstlane(at) + bits_below(K);
                if (kp && at < kMidP) {
                    L.xy[at] = q;
                    L.id[at] = id;
                    if (at < kRestRaw) {
                        gst(a.lxy + (size_t)c * kMidP + at, q);
                        gst(a.lid + (size_t)c * kMidP + at, id);
                    }
                }
            }
            __syncthreads();
            cnt = s_at[0];
            if (cnt > kMidP) {  // (uniform)
                if (t == 0) gst(a.lcnt + c, kMidP + 1);
                continue;
            }
        } else {
            const int c0 = c * kMidP;
            cnt = min(kMidP, M - c0);
            for (int i = t; i < cnt; i += kMidT) {
                const size_t q = rest_place(s_pre, ns, per, a.n, c0 + i);
                L.xy[i] = make_float2(gld(a.X[1] + q), gld(a.Y[1] + q));
                L.id[i] = gld(a.I[1] + q);
            }
            lds_barrier();
        }
        // what the second polygon thins goes on as it is; what it does not (copies
        // of its vertices: 57K points made the last workgroup solve 14 times, 1.5 ms)
        int h = cnt;
        if (!thin || cnt > kRestRaw) {
            h = solve<kMidT, kMidP, true>(L, cnt, 0, 0, false, ctr, nullptr);
            for (int r = t; r < h; r += kMidT) {
                const int q = L.ring[r];
                gst(a.lxy + (size_t)c * kMidP + r, L.xy[q]);
                gst(a.lid + (size_t)c * kMidP + r, L.id[q]);
            }
        }
        if (t == 0) gst(a.lcnt + c, h);
    }
    ctr_flush(ctl->ctr, ctr, csum);
    ctr = Counters{0u, 0u, 0u};
    if (!finishes_last(&ctl->done, nb, &s_last)) return;
    if (t < 3) csum[t] = 0u;
    int c = 0, at = 0, h = -1;
    for (;;) {
        const int n = gather_hulls<kMidT, kMidP>(L, a, a.lcnt, c, nc, at, s_next, s_at);
        const int next = s_next[0];
        const bool end = next >= nc;
        if (next == c && !end) break;  // (one hull and the last ones' do not fit together)
        h = solve<kMidT, kMidP, true>(L, n, 0, 0, false, ctr, end ? &st : nullptr);
        if (end) break;
        // their hull's points to the front, then the next chunks
        float2 v[kMidP / kMidT];
        int id[kMidP / kMidT];
#pragma unroll
        for (int r = 0; r < kMidP / kMidT; ++r) {
            const int i = t + kMidT * r;
            if (i < h) { v[r] = L.xy[L.ring[i]]; id[r] = L.id[L.ring[i]]; }
        }
        lds_barrier();
#pragma unroll
        for (int r = 0; r < kMidP / kMidT; ++r) {
            const int i = t + kMidT * r;
            if (i < h) { L.xy[i] = v[r]; L.id[i] = id[r]; }
        }
        at = h;
        c = next;
        h = -1;
        lds_barrier();
    }
    rest_finish<kMidT, kMidP>(a, L, h, M, st, ctr, csum);
}

}  // namespace sqh
