// One large ring of points (device code, gfx950): a set of which the sieve
// would keep many points, or whose hull has many vertices.
//
// The sort-then-remove of sqh_dense.hpp over the whole chip, with wedges cut by
// rays instead of vertices: rays from a centre c through arbitrary points r_k.
//   k_ring_rays     kRays rays at equal shares of a sample's points by angle
//   k_ring_count    every point's wedge (exactly), points per wedge
//   k_ring_scan     where each workgroup's points of a wedge start
//   k_ring_scatter  the points to their wedge's slots
//   k_ring_cut      a workgroup per wedge: into pockets of about 100 points
//   k_ring_pocket   a wave per pocket: sorted by angle about c, exactly, and
//                   reduced by the removal rounds (the two ends stay: their
//                   neighbours are elsewhere)
//   k_ring_wedge    a workgroup per wedge: the rounds over its pockets' nodes
//   k_ring_join     the wedges joined at their seams into the hull
//   k_ring_emit     its indices and the status
// Every removed point lies in the triangle of c and two points of the set, so
// it is no hull vertex as long as c is inside the hull, and what is left is a
// polygon around c with only strictly convex nodes: both are checked before
// anything is written, and a set that fails is left to the streaming path.
//
// The passes of the streaming path kept nearly every point of a circle for 9
// of its 16 passes: 1530 us for 5M points. Here each point is read four times
// and written twice: rays 19, count 17, scan 16, scatter 41, cut 56, pockets
// 113, wedges 31, join 42, emit 6 us, and 35 us of the sieve's kernels that
// found the ring. The pockets are bound by instruction issue (the sort's 28
// steps and about 8 rounds of 100 points each), the rest by latency.
#pragma once
#include "sqh_dense.hpp"

namespace sqh {

constexpr int kRays = 512;
constexpr int kRingSample = 8192;
constexpr float kRayFar = 1024.0f;  // a ray's point, in extents from the centre
constexpr int kSubRays = 512;       // pockets of a wedge, at most
constexpr int kSubBins = 1024;
constexpr int kPocketTarget = 100;
// A wave takes a pocket and a workgroup cuts a wedge, so that copies of one
// point, or a cluster in one direction, make the whole call wait for them (4097
// points, 2458 of them copies of one: 2.5 ms, because a wave sorts 256 copies by
// index in 180 us). Sets with a pocket of far more points than its wedge's
// others, or a wedge of more than eight times its even share, go to other paths.
__device__ __forceinline__ int pocket_most(int len, int want) { return 256 + 4 * (len / want); }
__device__ __forceinline__ int wedge_most(int n) { return n / 64 + (1 << 14); }
constexpr int kRingGrid = 512;      // workgroups of the count and the scatter, at most

struct RingPocket {
    float ax, ay, bx, by;  // points of its two rays (rounded)
    int off, len, pad[2];  // its slots
};
struct RingWedge {
    int first, cnt;  // its pockets
    int off, len;    // its nodes after k_ring_wedge
};
struct RingCtl {
    int left, err, n_pocket, nr;  // nr: rays
    float2 c, inv;  // the centre; 1 / half extents
    unsigned long long t0;
    CtrSlot ctr[kCtrSlots];
    int tot[kRays];
    float2 ray[kRays + 1];  // (ray[nr] repeats the first)
    uint16_t lut[kRingBins];  // the ray at or before a bin's start
    RingWedge wedge[kRays];
    unsigned long long low[kRays];  // a wedge's lexicographic minimum ...
    int low_at[kRays];              // ... and its node
    // the hull: pieces of consecutive nodes [pre, pre + its count) from
    // off, piece k's first vertex is the hull's at[k]th
    int pieces, h, start, buf;
    int off[kRays], at[kRays + 1];
    int bad, pad;  // bad: the nodes are no star around c
};

__device__ __forceinline__ bool gate_shut(const RingArgs& a) { return a.gate && *a.gate != 1; }

__device__ __forceinline__ float2 ring_dir(int b)  // a bin's start
{
    constexpr int Q = kRingBins / 4;
    const int k = b / Q;
    const float f = (float)(b % Q) * (1.0f / Q), g = 1.0f - f;
    // (by signs: as four cases the compiler, AMD clang 22, left the last one's y unset)
    const float sx = k == 1 || k == 2 ? -1.0f : 1.0f, sy = k >= 2 ? -1.0f : 1.0f;
    return make_float2(sx * ((k & 1) ? f : g), sy * ((k & 1) ? g : f));
}

// Block-wide exclusive prefix of v (T threads); *tot the sum. red: T / 64 words.
template <int T>
__device__ __forceinline__ int block_prefix(int v, int* red, int* tot)
{
    const int lane = lane_id(), w = (int)(threadIdx.x >> 6);
    const int inc = wave_incl_sum(v);
    __syncthreads();
    if (lane == 63) red[w] = inc;
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int u = 0; u < T / 64; ++u) {
        before += u < w ? red[u] : 0;
        all += red[u];
    }
    *tot = all;
    return before + inc - v;
}

__global__ __launch_bounds__(1024) void k_ring_rays(RingArgs a)
{
    __shared__ unsigned int lo[2], hi[2];
    __shared__ int hist[kRingBins], red[16], s_bad;
    __shared__ float2 ray[kRays];
    __shared__ int bin[kRays];
    RingCtl* ctl = a.ctl;
    if (gate_shut(a)) return;
    const int t = (int)threadIdx.x, lane = lane_id(), n = a.n;
    constexpr int U = kRingSample / 1024;
    // the centre: of three vertices of the sieve's polygon (its control block
    // is where this one goes), inside the hull also where the box's is not
    const SieveCtl* sieve = reinterpret_cast<const SieveCtl*>(ctl);
    const int ph = sieve->h;
    const bool poly = ph >= 3;
    const float2 pa = sieve->ring[0], pb = sieve->ring[poly ? ph / 3 : 0], pc = sieve->ring[poly ? 2 * ph / 3 : 0];
    // (the call's clock and counters go on from the sieve's)
    const unsigned long long t0 = sieve->t0, before = t < 3 ? ctr_total(sieve->ctr, t) : 0ull;
    __syncthreads();
    if (t == 0) {
        ctl->t0 = t0;
        ctl->left = 0; ctl->err = 0; ctl->n_pocket = 0;
        ctl->bad = 0;
        s_bad = 0;
    }
    if (t < 3 * kCtrSlots) ctl->ctr[t / 3].c[t % 3] = before;
    if (t < 2) { lo[t] = ~0u; hi[t] = 0u; }
    for (int b = t; b < kRingBins; b += 1024) hist[b] = 0;
    float2 p[U];
#pragma unroll
    for (int j = 0; j < U; ++j) p[j] = gld(a.xy + (int)((long long)(t + 1024 * j) * n / kRingSample));
    uint32_t box[4] = {~0u, ~0u, 0u, 0u};
#pragma unroll
    for (int j = 0; j < U; ++j) {
        if (!((int)isfinite(p[j].x) & (int)isfinite(p[j].y))) continue;
        const uint32_t x = order_key(p[j].x), y = order_key(p[j].y);
        box[0] = min(box[0], x); box[1] = min(box[1], y);
        box[2] = max(box[2], x); box[3] = max(box[3], y);
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        const uint64_t mn = wave_min_u64(box[c]), mx = wave_max_u64(box[2 + c]);
        if (lane == 63) {
            atomicMin(&lo[c], (unsigned int)mn);
            atomicMax(&hi[c], (unsigned int)mx);
        }
    }
    __syncthreads();
    auto back = [](uint32_t v) { return __uint_as_float((v & 0x80000000u) ? v ^ 0x80000000u : ~v); };
    const double xl = back(lo[0]), xh = back(hi[0]), yl = back(lo[1]), yh = back(hi[1]);
    const float2 c = poly ? make_float2((float)(((double)pa.x + (double)pb.x + (double)pc.x) / 3.0),
                                        (float)(((double)pa.y + (double)pb.y + (double)pc.y) / 3.0))
                          : make_float2((float)(0.5 * (xl + xh)), (float)(0.5 * (yl + yh)));
    const float ex = (float)(0.5 * (xh - xl)), ey = (float)(0.5 * (yh - yl));
    const bool ok = ex > 0x1p-50f && ex < 0x1p50f && ey > 0x1p-50f && ey < 0x1p50f &&
                    fabsf(c.x) <= kRayFar * ex && fabsf(c.y) <= kRayFar * ey;
    const float ix = ok ? 1.0f / ex : 0.0f, iy = ok ? 1.0f / ey : 0.0f;
#pragma unroll
    for (int j = 0; j < U; ++j) {
        if (!((int)isfinite(p[j].x) & (int)isfinite(p[j].y))) continue;
        bool near;
        atomicAdd(&hist[ring_bin((p[j].x - c.x) * ix, (p[j].y - c.y) * iy, near)], 4);
    }
    __syncthreads();
    // every bin weighs one more (a quarter of a sample point), so that no
    // wedge comes near half a turn; a ray where a share of the weight ends
    constexpr int E = kRingBins / 1024;
    int w[E], sum = 0;
#pragma unroll
    for (int j = 0; j < E; ++j) {
        w[j] = hist[t * E + j] + 1;
        sum += w[j];
    }
    int all;
    int at = block_prefix<1024>(sum, red, &all);
    bool on[E];
    int rays = 0;
#pragma unroll
    for (int j = 0; j < E; ++j) {
        const int b = t * E + j;
        const int was = b > 0 ? hist[b - 1] + 1 : 0;
        on[j] = b == 0 || (long long)at * kRays / all != (long long)(at - was) * kRays / all;
        rays += on[j];
        at += w[j];
    }
    int nr;
    int k = block_prefix<1024>(rays, red, &nr);  // (nr <= kRays)
#pragma unroll
    for (int j = 0; j < E; ++j) {
        const int b = t * E + j;
        if (on[j]) bin[k++] = b;
        ctl->lut[b] = (uint16_t)(k - 1);
    }
    __syncthreads();
    if (t < nr) {
        // far out, where the rounding of the point turns the ray least
        const float2 d = ring_dir(bin[t]);
        ray[t] = make_float2(c.x + kRayFar * ex * d.x, c.y + kRayFar * ey * d.y);
    }
    __syncthreads();
    if (t < nr) {
        const float2 r = ray[t], q = ray[t + 1 < nr ? t + 1 : 0];
        if (!ok || orient_exact(c.x, c.y, r.x, r.y, q.x, q.y) <= 0) s_bad = 1;
        gst(ctl->ray + t, r);
        if (t == 0) gst(ctl->ray + nr, r);
    }
    __syncthreads();
    if (t == 0) {
        ctl->c = c;
        ctl->inv = make_float2(ix, iy);
        ctl->nr = nr;
        if (s_bad) ctl->left = 1;
    }
}

// The last of the rays r[0 .. K) (r[K] repeats the first) at or before p,
// exactly, from a guess near it. -1 if p is c.
__device__ __forceinline__ int wedge_of(const float2* r, int K, float2 c, int k, float px, float py, Counters& ctr)
{
    bool sure = false;
    for (int s = 0; s < 8; ++s) {
        const float2 v = r[k], w = r[k + 1];
        const Orient32 o0 = orient32p(c.x, c.y, v.x, v.y, px, py), o1 = orient32p(c.x, c.y, w.x, w.y, px, py);
        const bool after = o0.d > o0.es, before = o1.d < -o1.es;
        ctr.orient += 2;
        if (after && before) { sure = true; break; }
        if (!(fabsf(o0.d) > o0.es) || !(fabsf(o1.d) > o1.es)) break;  // (undecided)
        // past ray k + 1, or before ray k
        if (after) k = k + 1 < K ? k + 1 : 0;
        else k = k > 0 ? k - 1 : K - 1;
    }
    if (__ballot(!sure)) {
        if (!sure) {
            if (px == c.x && py == c.y) return -1;
            ctr.orient_exact += 2;
            bool in = false;
            for (int tries = 0; tries <= K && !in; ++tries) {
                const float2 v = r[k], w = r[k + 1];
                const int s0 = orient_exact(c.x, c.y, v.x, v.y, px, py), s1 = orient_exact(c.x, c.y, w.x, w.y, px, py);
                in = s0 >= 0 && s1 < 0;
                if (in) break;
                if (s0 < 0) k = k > 0 ? k - 1 : K - 1;
                else k = k + 1 < K ? k + 1 : 0;
            }
            if (!in) return -1;
        }
    }
    return k;
}

// The share of workgroup b of nb: whole rows of 64 points.
__device__ __forceinline__ void ring_share(int n, int b, int nb, int& q0, int& q1)
{
    const int per = (((n + nb - 1) / nb) + 63) & ~63;
    q0 = (int)min((long long)b * per, (long long)n);
    q1 = (int)min((long long)q0 + per, (long long)n);
}

__global__ __launch_bounds__(1024) void k_ring_count(RingArgs a)
{
    constexpr int U = 4;
    __shared__ float2 ray[kRays + 1];
    __shared__ uint16_t lut[kRingBins];
    __shared__ int cnt[kRays], s_bad;
    __shared__ uint32_t csum[3];
    RingCtl* ctl = a.ctl;
    if (gate_shut(a)) return;
    if (ctl->left) return;
    const int t = (int)threadIdx.x, b = (int)blockIdx.x;
    for (int k = t; k <= ctl->nr; k += 1024) ray[k] = gld(ctl->ray + k);
    for (int k = t; k < kRingBins; k += 1024) lut[k] = ctl->lut[k];
    if (t < kRays) cnt[t] = 0;
    if (t < 3) csum[t] = 0u;
    if (t == 0) s_bad = 0;
    const float2 c = ctl->c, inv = ctl->inv;
    const int nr = ctl->nr;
    __syncthreads();
    Counters ctr = {0u, 0u, 0u};
    int q0, q1;
    ring_share(a.n, b, (int)gridDim.x, q0, q1);
    bool bad = false;
    for (int q = q0; q < q1; q += 1024 * U) {
        float2 v[U];
#pragma unroll
        for (int j = 0; j < U; ++j) v[j] = gld(a.xy + min(q + t + 1024 * j, q1 - 1));
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int i = q + t + 1024 * j;
            const bool fin = (int)isfinite(v[j].x) & (int)isfinite(v[j].y);
            bad |= !fin;
            if (i < q1 && fin) {
                bool near;
                int k = lut[ring_bin((v[j].x - c.x) * inv.x, (v[j].y - c.y) * inv.y, near)];
                if (near) k = wedge_of(ray, nr, c, k, v[j].x, v[j].y, ctr);
                a.wid[i] = (uint16_t)k;  // (0xffff: c itself, in no wedge)
                if (k >= 0) atomicAdd(&cnt[k], 1);
            }
        }
    }
    if (__ballot(bad) && lane_id() == 0) s_bad = 1;
    __syncthreads();
    if (t < kRays) a.off[b * kRays + t] = cnt[t];
    if (t == 0 && s_bad) atomicOr(&ctl->err, kErrNonFinite);
    ctr_flush(ctl->ctr, ctr, csum);
}

// The counts' prefixes over the nb workgroups: 64 rays to a workgroup.
__global__ __launch_bounds__(1024) void k_ring_scan(RingArgs a, int nb)
{
    __shared__ int part[16][64];
    RingCtl* ctl = a.ctl;
    if (gate_shut(a)) return;
    if (call_ended(&ctl->err, &ctl->left)) return;
    const int lane = lane_id(), w = (int)(threadIdx.x >> 6), k = (int)blockIdx.x * 64 + lane;
    const int per = (nb + 15) / 16, b0 = min(w * per, nb), b1 = min(b0 + per, nb);
    int sum = 0;
    for (int b = b0; b < b1; ++b) sum += gld(a.off + b * kRays + k);
    part[w][lane] = sum;
    __syncthreads();
    int run = 0, all = 0;
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        const int v = part[u][lane];
        run += u < w ? v : 0;
        all += v;
    }
    for (int b = b0; b < b1; ++b) {
        const int v = gld(a.off + b * kRays + k);
        gst(a.off + b * kRays + k, run);
        run += v;
    }
    if (w == 0) {
        ctl->tot[k] = all;
        if (all > wedge_most(a.n)) ctl->left = 1;
    }
}

__global__ __launch_bounds__(1024) void k_ring_scatter(RingArgs a)
{
    constexpr int U = 4;
    __shared__ int cur[kRays], red[16];
    RingCtl* ctl = a.ctl;
    if (gate_shut(a)) return;
    if (ctl->left | ctl->err) return;
    const int t = (int)threadIdx.x, b = (int)blockIdx.x;
    int all;
    const int base = block_prefix<1024>(t < kRays ? ctl->tot[t] : 0, red, &all);
    if (t < kRays) cur[t] = base + a.off[b * kRays + t];
    if (b == 0 && t < kRays) {
        ctl->wedge[t].off = base;
        ctl->wedge[t].len = ctl->tot[t];
    }
    __syncthreads();
    int q0, q1;
    ring_share(a.n, b, (int)gridDim.x, q0, q1);
    for (int q = q0; q < q1; q += 1024 * U) {
        float2 v[U];
        int k[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int i = min(q + t + 1024 * j, q1 - 1);
            v[j] = gld(a.xy + i);
            k[j] = a.wid[i];
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int i = q + t + 1024 * j;
            if (i < q1 && k[j] < kRays)
                gst(a.slots + atomicAdd(&cur[k[j]], 1),
                    make_float4(v[j].x, v[j].y, __int_as_float(a.ids ? gld(a.ids + i) : i), 0.0f));
        }
    }
}

// Whether p is at or after the ray from c along d, both less than half a turn
// apart, exactly; bad if that takes more than float64 differences.
__device__ __forceinline__ bool after_ray(double dx, double dy, float2 c, float px, float py, bool& bad)
{
    double x, y, ex, ey;
    two_sum((double)px, -(double)c.x, x, ex);
    two_sum((double)py, -(double)c.y, y, ey);
    const double P = dx * y, Q = dy * x;
    if (fabs(P - Q) > (fabs(P) + fabs(Q)) * 0x1p-50) return P > Q;
    bad |= ex != 0.0 || ey != 0.0;
    const double t[4] = {P, -Q, fma(dx, y, -P), -fma(dy, x, -Q)};
    return expansion_sign(t) >= 0;
}

__global__ __launch_bounds__(1024) void k_ring_cut(RingArgs a)
{
    __shared__ uint16_t lut[kSubBins];
    __shared__ int hist[kSubBins], cnt[kSubRays], cur[kSubRays], start[kSubRays + 1], red[16], s_p0, s_bad;
    RingCtl* ctl = a.ctl;
    if (gate_shut(a)) return;
    const int t = (int)threadIdx.x, w = (int)blockIdx.x;
    if (call_ended(&ctl->err, &ctl->left) || w >= ctl->nr) return;
    const int off = ctl->wedge[w].off, len = ctl->wedge[w].len;
    const float2 c = ctl->c, A = gld(ctl->ray + w), B = gld(ctl->ray + w + 1);
    const int want = min(max(len / kPocketTarget, 1), kSubRays);
    const float4* src = a.slots + off;
    hist[t] = 0;
    if (t < kSubRays) cnt[t] = 0;
    if (t == 0) s_bad = 0;
    __syncthreads();
    // a point's bin: its ray's share of the chord from A to B, in float64
    // (float32 cannot tell neighbours of a dense wedge apart); bin j starts at
    // the ray along dir(j)
    const double ax = (double)A.x - c.x, ay = (double)A.y - c.y, bx = (double)B.x - c.x, by = (double)B.y - c.y;
    auto dir_x = [&](int j) { return ax + (double)j * (1.0 / kSubBins) * (bx - ax); };
    auto dir_y = [&](int j) { return ay + (double)j * (1.0 / kSubBins) * (by - ay); };
    bool bad = false;
    for (int i = t; i < len; i += 1024) {
        const float4 p = gld(src + i);
        const double x = (double)p.x - c.x, y = (double)p.y - c.y;
        const double u = ax * y - ay * x, v = x * by - y * bx;
        const float s = (float)(u + v), f = (float)u * __builtin_amdgcn_rcpf(s) * (float)kSubBins;
        int j = min(max((int)f, 0), kSubBins - 1);
        const float r = f - (float)j;
        // (the rounding of f is less than half of kRingNear)
        if (!((int)(r >= kRingNear) & (int)(r <= 1.0f - kRingNear))) {
            if (r < 0.5f) j -= j > 0 && !after_ray(dir_x(j), dir_y(j), c, p.x, p.y, bad);
            else j += j + 1 < kSubBins && after_ray(dir_x(j + 1), dir_y(j + 1), c, p.x, p.y, bad);
        }
        bad |= !(s > 0x1p-100f);
        atomicAdd(&hist[j], 1);
        a.wid[off + i] = (uint16_t)j;
    }
    if (bad) s_bad = 1;
    __syncthreads();
    if (s_bad) {
        if (t == 0) ctl->left = 1;
        return;
    }
    // a ray at the bin's start where a share ends
    int all, K;
    const int h = hist[t], at = block_prefix<1024>(h, red, &all);
    const int was = t > 0 ? hist[t - 1] : 0;
    const bool on = t == 0 || (at < all && (long long)at * want / all != (long long)(at - was) * want / all);
    const int k0 = block_prefix<1024>(on ? 1 : 0, red, &K) + (on ? 1 : 0) - 1;  // (K <= want)
    lut[t] = (uint16_t)k0;
    if (on) {
        start[k0] = t;
        cur[k0] = at;
    }
    if (h) atomicAdd(&cnt[k0], h);
    if (t == 0) {
        start[K] = kSubBins;
        s_p0 = atomicAdd(&ctl->n_pocket, K);
        ctl->wedge[w].first = s_p0;
        ctl->wedge[w].cnt = K;
        if (s_p0 + K > a.pocket_cap) { s_bad = 1; ctl->left = 1; }
    }
    __syncthreads();
    const bool heap = t < K && cnt[t] > pocket_most(len, want);
    if (__syncthreads_or(heap)) {
        if (t == 0) ctl->left = 1;
        return;
    }
    if (s_bad) return;
    if (t < K) {
        RingPocket p;
        p.ax = (float)(c.x + dir_x(start[t])); p.ay = (float)(c.y + dir_y(start[t]));
        p.bx = (float)(c.x + dir_x(start[t + 1])); p.by = (float)(c.y + dir_y(start[t + 1]));
        p.off = off + cur[t]; p.len = cnt[t]; p.pad[0] = p.pad[1] = 0;
        gst(a.pockets + s_p0 + t, p);
    }
    __syncthreads();
    for (int i = t; i < len; i += 1024)
        gst(a.slots2 + off + atomicAdd(&cur[lut[a.wid[off + i]]], 1), gld(src + i));
}

constexpr int kRingWaves = 4;
__global__ __launch_bounds__(64 * kRingWaves) void k_ring_pocket(RingArgs a)
{
    constexpr int R = kWavePts / 64;
    __shared__ WaveLds Ws[kRingWaves];
    __shared__ uint32_t csum[3];
    RingCtl* ctl = a.ctl;
    if (gate_shut(a)) return;
    if (call_ended(&ctl->err, &ctl->left)) return;
    const int lane = lane_id(), w = (int)(threadIdx.x >> 6), np = ctl->n_pocket;
    const float2 c = ctl->c;
    WaveLds& W = Ws[w];
    if (threadIdx.x < 3) csum[threadIdx.x] = 0u;
    __syncthreads();
    Counters ctr = {0u, 0u, 0u};
    for (int j = (int)blockIdx.x * kRingWaves + w; j < np; j += (int)gridDim.x * kRingWaves) {
        const RingPocket p = gld(a.pockets + j);
        float4* slot = a.slots2 + p.off;
        const float2 A = make_float2(p.ax, p.ay), B = make_float2(p.bx, p.by);
        // up to kWavePts points at a time: those left of the ones before and
        // the next ones
        int m = 0, next = 0, f;
        for (;;) {
            const int take = min(p.len - next, kWavePts - m);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int q = lane + 64 * r;
                if (q < take) {
                    const float4 v = gld(slot + next + q);
                    W.xy[0][m + q] = make_float2(v.x, v.y);
                    W.id[m + q] = __float_as_int(v.z);
                }
            }
            wave_sync();
            next += take;
            m = wave_chain<true>(W, m + take, c, A, B, f, ctr);
            if (next == p.len || m == kWavePts) break;
            // back to the first buffer, in order
            for (int q = lane; q < m; q += 64) W.xy[f ^ 1][q] = make_float2(__int_as_float(W.id[W.at[f][q]]), 0.0f);
            wave_sync();
            for (int q = lane; q < m; q += 64) W.id[q] = __float_as_int(W.xy[f ^ 1][q].x);
            wave_sync();
            if (f == 1) {
                for (int q = lane; q < m; q += 64) W.xy[0][q] = W.xy[1][q];
                wave_sync();
            }
        }
        if (next < p.len) {  // (full: too many of its points are left)
            if (lane == 0) ctl->left = 1;
            wave_sync();
            continue;
        }
        for (int q = lane; q < m; q += 64)
            gst(slot + q, make_float4(W.xy[f][q].x, W.xy[f][q].y, __int_as_float(W.id[W.at[f][q]]), 0.0f));
        if (lane == 0) gst(&a.pockets[j].len, m);
        wave_sync();
    }
    ctr_flush(ctl->ctr, ctr, csum);
}

// Two lists of nodes.
struct NodesGlobal {
    float4* b[2];
    __device__ __forceinline__ float4 get(int f, int i) const { return gld(b[f] + i); }
    __device__ __forceinline__ void put(int f, int i, float4 v) const { gst(b[f] + i, v); }
};
template <int P>
struct NodesLds {
    float4 (*b)[P];
    __device__ __forceinline__ float4 get(int f, int i) const { return b[f][i]; }
    __device__ __forceinline__ void put(int f, int i, float4 v) const { b[f][i] = v; }
};

// The removal rounds over the m nodes of buf's first list, by a workgroup of T threads: as a
// ring (RING), or as a chain whose two ends stay. Returns how many are left, in
// list f. red: T / 64 words.
// Where two arcs meet at a reflex node, a round takes two nodes: after 8 rounds
// every other one tests a node against those m / 4, m / 8, .. places away (any
// two nodes around it will do as long as they are less than half a turn apart),
// which takes such a stretch at once (two circles of 1M points side by side:
// 20 ms of rounds without). SWEEP: no round before needs to take a node, as in
// a list whose pieces went through their own rounds; the places apart go from
// m / 4 to 1 and round again, until neighbours agree (five lobes of a star, 3M
// points: 1.5 ms of the join without).
template <int T, bool RING, bool SWEEP = false, typename Buf>
__device__ __forceinline__ int ring_rounds(const Buf& buf, int m, float2 c, int& f, int* red, Counters& ctr)
{
    constexpr int W = T / 64, kRows = 32;
    const int lane = lane_id(), w = (int)(threadIdx.x >> 6);
    f = 0;
    int far = 0;
    for (int round = 0;; ++round) {
        int step = 1;
        if (SWEEP) {
            far = far < 2 ? m >> 2 : min(far >> 1, m >> 2);
            step = max(far, 1);
        } else if (round >= 8 && (round & 1)) {
            far = min(far < 2 ? m : far >> 1, m >> 2);
            step = max(far, 1);
        }
        // each wave takes a contiguous run of whole rows, kRows at a time
        int out = 0;  // nodes kept before the block of rows
        for (int q0 = 0; q0 < m; q0 += T * kRows) {
            const int mb = min(m - q0, T * kRows);
            const int per = (((mb + W - 1) / W) + 63) & ~63;
            const int wb = q0 + min(w * per, mb), we = q0 + min(w * per + per, mb);
            uint32_t keep = 0u;
            int cnt = 0;
            for (int r = 0; wb + 64 * r < we; ++r) {
                const int q = wb + 64 * r + lane;
                bool kp = false;
                if (q < we) {
                    const int qo = q - step, qe = q + step;
                    const float4 p = buf.get(f, q), o = buf.get(f, qo >= 0 ? qo : (RING ? qo + m : 0)),
                                 e = buf.get(f, qe < m ? qe : (RING ? qe - m : m - 1));
                    const float2 op = make_float2(o.x, o.y), ep = make_float2(e.x, e.y);
                    kp = (!RING && (q == 0 || q == m - 1)) || orient_of(op, make_float2(p.x, p.y), ep, ctr) > 0 ||
                         (RING && step > 1 && orient_of(c, op, ep, ctr) <= 0);
                }
                keep |= (uint32_t)kp << r;
                cnt += (int)__popcll(__ballot(kp));
            }
            __syncthreads();
            if (lane == 0) red[w] = cnt;
            __syncthreads();
            int at = out;
#pragma unroll
            for (int u = 0; u < W; ++u) {
                at += u < w ? red[u] : 0;
                out += red[u];
            }
            for (int r = 0; wb + 64 * r < we; ++r) {
                const bool kp = (keep >> r) & 1u;
                const uint64_t M = __ballot(kp);
                if (kp) buf.put(f ^ 1, at + bits_below(M), buf.get(f, wb + 64 * r + lane));
                at += (int)__popcll(M);
            }
        }
        __syncthreads();
        f ^= 1;
        if (out == m && step == 1) return m;  // (uniform)
        m = out;
    }
}

__device__ __forceinline__ uint64_t lex_key(const float4& p)
{
    return ((uint64_t)order_key(p.x + 0.0f) << 32) | order_key(p.y + 0.0f);
}

// The rounds over a wedge's nodes (its two ends stay).
constexpr int kWedgeT = 256, kWedgeLds = 1024;
__global__ __launch_bounds__(kWedgeT) void k_ring_wedge(RingArgs a)
{
    __shared__ int s_at[kSubRays + 1], s_off[kSubRays], red[kWedgeT / 64];
    __shared__ unsigned long long s_min;
    __shared__ float4 s_list[2][kWedgeLds];
    __shared__ uint32_t csum[3];
    RingCtl* ctl = a.ctl;
    if (gate_shut(a)) return;
    const int t = (int)threadIdx.x, w = (int)blockIdx.x;
    if ((ctl->left | ctl->err) || w >= ctl->nr) return;
    const int first = ctl->wedge[w].first, K = ctl->wedge[w].cnt, off = ctl->wedge[w].off;
    Counters ctr = {0u, 0u, 0u};
    int run = 0;
    for (int k0 = 0; k0 < K; k0 += kWedgeT) {
        const int k = k0 + t, c = k < K ? gld(&a.pockets[first + k].len) : 0;
        int all;
        const int pre = block_prefix<kWedgeT>(c, red, &all);
        if (k < K) {
            s_at[k] = run + pre;
            s_off[k] = gld(&a.pockets[first + k].off);
        }
        run += all;
    }
    if (t == 0) s_at[K] = run;
    if (t < 3) csum[t] = 0u;
    __syncthreads();
    int m = run;
    // the pockets' nodes as one list (m <= the wedge's points), in LDS if it fits
    uint64_t lo = ~0ull;
    int lo_at = 0;
    bool bad = false;
    auto solve = [&](const auto& list) {
        for (int i = t; i < m; i += kWedgeT) {
            int l = 0, u = K;
            while (u - l > 1) {
                const int mid = (l + u) >> 1;
                if (s_at[mid] <= i) l = mid;
                else u = mid;
            }
            list.put(0, i, gld(a.slots2 + s_off[l] + (i - s_at[l])));
        }
        __syncthreads();
        int f;
        m = ring_rounds<kWedgeT, false>(list, m, ctl->c, f, red, ctr);
        // back to `slots`; its lexicographic minimum; every edge has to turn
        // about c (the first one may lie on a ray: the join sees to it)
        for (int i = t; i < m; i += kWedgeT) {
            const float4 p = list.get(f, i);
            if (i + 1 < m) {
                const float4 q = list.get(f, i + 1);
                const int o = orient_of(ctl->c, make_float2(p.x, p.y), make_float2(q.x, q.y), ctr);
                bad |= o < 0 || (o == 0 && i > 0);
            }
            gst(a.slots + off + i, p);
            const uint64_t v = lex_key(p);
            lo_at = v < lo ? i : lo_at;
            lo = v < lo ? v : lo;
        }
    };
    if (m <= kWedgeLds) solve(NodesLds<kWedgeLds>{s_list});
    else solve(NodesGlobal{{a.slots + off, a.slots2 + off}});
    if (t == 0) s_min = ~0ull;
    if (__ballot(bad) && lane_id() == 0) atomicOr(&ctl->bad, 1);
    __syncthreads();
    const uint64_t wl = wave_min_u64(lo);
    if (lane_id() == 63) atomicMin(&s_min, (unsigned long long)wl);
    __syncthreads();
    if (lo == s_min && m > 0 && t < m) ctl->low_at[w] = lo_at;  // (one node: the positions differ)
    if (t == 0) {
        ctl->low[w] = s_min;
        ctl->wedge[w].len = m;
    }
    ctr_flush(ctl->ctr, ctr, csum);
}

// The wedges' nodes joined into the hull. Seam k joins piece k - 1's last
// nodes and piece k's first ones: nodes that are not strictly convex between
// their neighbours go, from both sides of the seam, until those left are.
// Neighbouring seams share a piece and take turns; a piece that would empty is
// left to the removal rounds over the whole ring (rare).
// The nodes are the hull if the ring of them turns about c: each is strictly
// convex, they are in order by angle, wedge by wedge, and every edge takes less
// than half a turn, so all of them together take one. The edges inside a wedge
// were checked there (removing nodes at its ends adds none); left are each
// piece's first edge and the ones across the seams. Nothing is written for a
// set that fails.
constexpr int kEnds = 4;
__global__ __launch_bounds__(1024) void k_ring_join(RingArgs a)
{
    __shared__ int pre[kRays], suf[kRays], off[kRays], at[kRays], low_at[kRays], red[16];
    __shared__ int len[kRays];
    __shared__ float2 ends[kRays][2 * kEnds];
    __shared__ int s_chg, s_seq, s_start;
    __shared__ unsigned long long s_min;
    __shared__ uint32_t csum[3];
    RingCtl* ctl = a.ctl;
    if (gate_shut(a)) return;
    const int t = (int)threadIdx.x, lane = lane_id(), w = t >> 6;
    if (ctl->left | ctl->err) return;
    int K;
    uint64_t low = ~0ull;
    // the pieces that hold nodes, in order
    {
        const int cnt = t < ctl->nr ? ctl->wedge[t].len : 0;
        const int j = block_prefix<1024>(cnt > 0 ? 1 : 0, red, &K);
        if (cnt > 0) {
            pre[j] = 0;
            suf[j] = cnt;
            off[j] = ctl->wedge[t].off;
            low_at[j] = ctl->low_at[t];
            low = ctl->low[t];
        }
        if (t == 0) { s_seq = 0; s_chg = 0; s_start = 0; s_min = ~0ull; }
        if (t < 3) csum[t] = 0u;
        __syncthreads();
        const uint64_t wl = wave_min_u64(low);
        if (lane == 63) atomicMin(&s_min, (unsigned long long)wl);
        __syncthreads();
        if (cnt > 0 && low == s_min) s_start = j;  // its piece, for now
    }
    __syncthreads();
    const float2 c = ctl->c;
    Counters ctr = {0u, 0u, 0u};
    // (a piece's first and last nodes are in LDS: the seams' chain of reads)
    for (int i = t; i < K * 2 * kEnds; i += 1024) {
        const int k = i / (2 * kEnds), e = i % (2 * kEnds), n = suf[k], j = e < kEnds ? e : n - 2 * kEnds + e;
        if (j >= 0 && j < n) {
            const float4 v = gld(a.slots + off[k] + j);
            ends[k][e] = make_float2(v.x, v.y);
            len[k] = n;
        }
    }
    __syncthreads();
    auto node = [&](int k, int j) {
        const int n = len[k];
        if (j < kEnds) return ends[k][j];
        if (j >= n - kEnds) return ends[k][j - n + 2 * kEnds];
        const float4 v = gld(a.slots + off[k] + j);
        return make_float2(v.x, v.y);
    };
    auto dec = [&](int k) { return k > 0 ? k - 1 : K - 1; };
    auto inc = [&](int k) { return k + 1 < K ? k + 1 : 0; };
    auto seam = [&](int k) -> bool {
        bool changed = false;
        for (;;) {
            const int ka = dec(k), kb = k;
            const int ja = suf[ka] - 1, jb = pre[kb];  // the last node before the seam, the first after it
            int kp = ka, jp = ja - 1, kn = kb, jn = jb + 1;  // their outer neighbours
            if (jp < pre[ka]) {
                kp = dec(ka);
                jp = suf[kp] - 1;
            }
            if (jn >= suf[kb]) {
                kn = inc(kb);
                jn = pre[kn];
            }
            const float2 A = node(ka, ja), B = node(kb, jb);
            if (orient_of(node(kp, jp), A, B, ctr) <= 0) {
                if (ja == pre[ka]) { s_seq = 1; return changed; }
                suf[ka] = ja;
            } else if (orient_of(A, B, node(kn, jn), ctr) <= 0) {
                if (jb + 1 == suf[kb]) { s_seq = 1; return changed; }
                pre[kb] = jb + 1;
            } else {
                return changed;
            }
            changed = true;
        }
    };
    if (K >= 4) {
        for (;;) {
            bool changed = false;
            for (int color = 0; color < 3; ++color) {
                const int mine = (t == K - 1 && (K & 1)) ? 2 : (t & 1);
                if (t < K && mine == color) changed |= seam(t);
                __syncthreads();
            }
            if (changed) s_chg = 1;
            __syncthreads();
            const bool again = s_chg != 0 && s_seq == 0;
            __syncthreads();
            if (t == 0) s_chg = 0;
            if (!again) break;
            __syncthreads();
        }
    } else if (t == 0) {
        s_seq = 1;
    }
    __syncthreads();
    int h, start, buf = 0;
    bool bad = false;
    if (s_seq) {
        const int n = t < K ? suf[t] - pre[t] : 0;
        const int p = block_prefix<1024>(n, red, &h);
        if (t < K) at[t] = p;
        __syncthreads();
        for (int k = w; k < K; k += 16)
            for (int j = lane; j < suf[k] - pre[k]; j += 64) gst(a.slots2 + at[k] + j, gld(a.slots + off[k] + pre[k] + j));
        __syncthreads();
        const NodesGlobal list = {{a.slots2, a.slots}};
        int f;
        h = ring_rounds<1024, true, true>(list, h, c, f, red, ctr);
        buf = f ^ 1;
        for (int j = t; j < h; j += 1024) {
            const float4 p = list.get(f, j), q = list.get(f, j + 1 < h ? j + 1 : 0);
            bad |= orient_of(c, make_float2(p.x, p.y), make_float2(q.x, q.y), ctr) <= 0;
        }
        for (int j = t; j < h; j += 1024)
            if (lex_key(list.get(f, j)) == s_min) s_start = j;  // (one node: the ring's positions differ)
        __syncthreads();
        start = s_start;
        const int per = (h + kRays - 1) / kRays;
        K = per ? (h + per - 1) / per : 0;
        if (t < K) {
            ctl->off[t] = t * per;
            ctl->at[t] = t * per;
        }
    } else {
        const int n = t < K ? suf[t] - pre[t] : 0;
        const int p = block_prefix<1024>(n, red, &h);
        if (t < K) {
            ctl->off[t] = off[t] + pre[t];
            ctl->at[t] = p;
            at[t] = p;
            const int k = inc(t);
            const float2 A = node(t, pre[t]), Z = node(t, suf[t] - 1);
            bad |= orient_of(c, Z, node(k, pre[k]), ctr) <= 0;
            if (n > 1) bad |= orient_of(c, A, node(t, pre[t] + 1), ctr) <= 0;
        }
        __syncthreads();
        start = at[s_start] + low_at[s_start] - pre[s_start];
    }
    bad |= h < 3;
    if (__ballot(bad) && lane == 0) atomicOr(&ctl->bad, 1);
    if (t == 0) {
        ctl->at[K] = h;
        ctl->pieces = K;
        ctl->h = h;
        ctl->start = min(max(start, 0), max(h - 1, 0));
        ctl->buf = buf;
    }
    ctr_flush(ctl->ctr, ctr, csum);
}

// The hull from its lexicographic minimum, if the nodes are one, and the status.
constexpr int kRingEmitT = 256;
__global__ __launch_bounds__(kRingEmitT) void k_ring_emit(RingArgs a)
{
    __shared__ int at[kRays + 1], off[kRays];
    const RingCtl* ctl = a.ctl;
    if (gate_shut(a)) return;
    LocalStatus* st = a.status;
    const int t = (int)threadIdx.x, b = (int)blockIdx.x, nb = (int)gridDim.x;
    const int err = ctl->err;
    const bool good = !(ctl->left | err) && ctl->bad == 0;
    const int h = good ? ctl->h : 0;
    if (b == 0) {
        if (t < kLocalStatPasses) { st->pass_v[t] = 0; st->pass_s[t] = 0; }
        if (t == 0) {
            st->h = h;
            st->err = err;
            st->left = (good || err) ? 0 : 1;
            if (a.gate) {
                *a.h_dev = h;
                *a.bad_dev = err != 0;
            }
            st->passes = 0;
            st->first_v = a.n;
            st->line = a.line;
            st->orient = ctr_total(ctl->ctr, 0);
            st->orient_exact = ctr_total(ctl->ctr, 1);
            st->cmp_exact = ctr_total(ctl->ctr, 2);
            st->t0 = ctl->t0;
        }
    }
    if (good) {
        const int K = ctl->pieces, start = ctl->start;
        const float4* nodes = ctl->buf ? a.slots2 : a.slots;
        for (int k = t; k <= K; k += kRingEmitT) at[k] = ctl->at[k];
        for (int k = t; k < K; k += kRingEmitT) off[k] = ctl->off[k];
        __syncthreads();
        for (int e = b * kRingEmitT + t; e < h; e += nb * kRingEmitT) {
            int l = 0, u = K;
            while (u - l > 1) {
                const int m = (l + u) >> 1;
                if (at[m] <= e) l = m;
                else u = m;
            }
            const float4 p = gld(nodes + off[l] + (e - at[l]));
            const int r = e >= start ? e - start : e - start + h;
            if (r < a.cap) gst(a.out + r, __float_as_int(p.z));
        }
    }
    if (b == 0 && t == 0) st->t1 = wall_clock64();
}

}  // namespace sqh
