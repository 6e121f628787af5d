// Rings of points (device code, gfx950): sets of which a large part are hull
// vertices, so that no polygon sieves them.
//
// K vertices v_0 .. v_{K-1} of the sample's hull, evenly spaced along it, cut
// the plane into K wedges seen from a centre c strictly inside their polygon.
// A point of wedge k belongs to pocket k if it is strictly right of v_k ->
// v_{k+1}; the others lie in the triangle c v_k v_{k+1}, and are no hull
// vertices unless they are copies of v_k (whose lowest index is kept).
//
// Most of a ring's points survive most passes of QuickHull, so a pocket is
// solved by the sort-then-remove of the paper's section 3 instead: a wave
// sorts its points by angle about c, exactly, and then removes, in rounds and
// all at once, every point that is not strictly convex between its current
// neighbours. Such a point lies in the triangle of c and the two neighbours,
// points of the set, so it is no hull vertex whatever else goes in the same
// round (copies are removed first). The pockets' chains in order form a
// polygon that is star-shaped about c; the same rounds over all of it leave a
// star-shaped polygon with only strictly convex nodes, which is convex: the
// hull. 150 points take a wave about 1000 instructions, the passes 6000.
#pragma once
#include "sqh_solve.hpp"

namespace sqh {

constexpr int kDenseMaxK = 1024;   // pockets of one set
constexpr int kDenseTarget = 150;  // points per pocket aimed at: most pockets fit a wave's 254 (larger ones go to larger solvers)

// One pocket: its points are slots [off, off + len) of the pocket array
// (16 bytes each: x, y, index, nothing); once solved, the first len of them are its
// nodes, v_k first.
struct Pocket {
    float ax, ay, bx, by;    // v_k, v_{k+1}
    int aid, off, len, ring;  // index of v_k; its ring
};
// A ring of pockets [t0, t0 + k).
struct DenseSet {
    int set, t0, k, pad;
    float cx, cy;  // the centre
    int pad2[2];
};

constexpr int kRingBins = 4096;        // bins of the angle
constexpr float kRingNear = 0x1p-10f;  // (a share of a bin)

// The bin of a direction: 1024 to a quadrant, by the share of |y| in |x| + |y|
// (turning counter-clockwise). near: closer to a bin's border than the rounding
// of x, y (scaled by the extents) and of this may have moved it, or the border:
// together less than half of kRingNear where the centre is within 1024 extents of 0.
__device__ __forceinline__ int ring_bin(float x, float y, bool& near)
{
    constexpr int Q = kRingBins / 4;
    const float a = fabsf(x), b = fabsf(y), s = a + b;
    const bool l = x < 0.0f, d = y < 0.0f;
    const float f = (l == d ? b : a) * __builtin_amdgcn_rcpf(s) * (float)Q;
    const int j = min(max((int)f, 0), Q - 1);
    const float r = f - (float)j;
    near = !((int)(r >= kRingNear) & (int)(r <= 1.0f - kRingNear) & (int)(s > 0x1p-100f));
    return (d ? (l ? 2 : 3) : (l ? 1 : 0)) * Q + j;
}

struct DenseLds {
    float2 v[kDenseMaxK];  // the vertices
    int id[kDenseMaxK];
    int cnt[kDenseMaxK], cur[kDenseMaxK];
    uint16_t lut[kRingBins];  // the last vertex at or before a bin's start, but for rounding
    float2 c, inv;  // the centre; 1 / half extents
    unsigned int lo[2], hi[2];
    int bad;
};

// Chooses the vertices and the centre from the ring L.ring[0 .. h) of a
// sample (h >= 2 K >= 8). D may overlap everything of L but L.bad.
// Returns false if the centre is not certified inside (then nothing is usable).
template <int T, int P>
__device__ __forceinline__ bool dense_build(const SolveLds<P>& L, int h, int K, DenseLds& D)
{
    constexpr int E = kDenseMaxK / T;
    const int t = (int)threadIdx.x;
    float2 v[E];
    int id[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int k = t + T * e;
        if (k < K) {
            const int r = L.ring[(int)((long long)k * h / K)];
            v[e] = L.xy[r];
            id[e] = L.id[r];
        }
    }
    const float2 p = L.xy[L.ring[0]], q = L.xy[L.ring[h / 3]], r = L.xy[L.ring[2 * h / 3]];
    lds_barrier();
    if (t == 0) {
        D.c.x = (float)(((double)p.x + (double)q.x + (double)r.x) / 3.0);
        D.c.y = (float)(((double)p.y + (double)q.y + (double)r.y) / 3.0);
        D.bad = 0;
    }
    if (t < 2) { D.lo[t] = ~0u; D.hi[t] = 0u; }
    for (int b = t; b < kRingBins; b += T) D.lut[b] = 0;
    lds_barrier();
    uint32_t box[4] = {~0u, ~0u, 0u, 0u};
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int k = t + T * e;
        if (k < K) {
            D.v[k] = v[e];
            D.id[k] = id[e];
            D.cnt[k] = 0;
            const uint32_t x = order_key(v[e].x), y = order_key(v[e].y);
            box[0] = min(box[0], x); box[1] = min(box[1], y);
            box[2] = max(box[2], x); box[3] = max(box[3], y);
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const uint64_t mn = wave_min_u64(box[i]), mx = wave_max_u64(box[2 + i]);
        if (lane_id() == 63) {
            atomicMin(&D.lo[i], (unsigned int)mn);
            atomicMax(&D.hi[i], (unsigned int)mx);
        }
    }
    lds_barrier();
    auto back = [](uint32_t u) { return __uint_as_float((u & 0x80000000u) ? u ^ 0x80000000u : ~u); };
    const float ex = back(D.hi[0]) - back(D.lo[0]), ey = back(D.hi[1]) - back(D.lo[1]);
    const float2 c = D.c, inv = make_float2((ex > 0.0f && ex < INFINITY) ? 2.0f / ex : 1.0f, (ey > 0.0f && ey < INFINITY) ? 2.0f / ey : 1.0f);
    if (t == 0) D.inv = inv;
    for (int k = t; k < K; k += T) {
        const float2 a = D.v[k], b = D.v[k + 1 < K ? k + 1 : 0];
        if (orient_exact(a.x, a.y, b.x, b.y, c.x, c.y) <= 0) D.bad = 1;
        bool near;
        const int i = ring_bin((a.x - c.x) * inv.x, (a.y - c.y) * inv.y, near);
        const int n = (ring_bin((b.x - c.x) * inv.x, (b.y - c.y) * inv.y, near) - i) & (kRingBins - 1);
        // (a wedge is less than half a turn; more is a rounded step back)
        if (n <= kRingBins / 2 + 1)
            for (int j = 1; j <= n; ++j) D.lut[(i + j) & (kRingBins - 1)] = (uint16_t)k;
    }
    lds_barrier();
    return D.bad == 0;
}

// The wedge of p, but for rounding: from the bin's first vertex by bisection
// among the bin's (of 1024 even wedges a bin holds one in four, and ten steps
// of bisection over all of them took half of the cut's time).
__device__ __forceinline__ int wedge_guess(const DenseLds& D, int K, float px, float py)
{
    const float2 c = D.c, inv = D.inv;
    const float x = px - c.x, y = py - c.y;
    bool near;
    const int b = ring_bin(x * inv.x, y * inv.y, near);
    int k = D.lut[b], span = (int)D.lut[(b + 1) & (kRingBins - 1)] - k;
    span = span < 0 ? span + K : span;  // vertices in the bin
    while (span > 0) {
        const int half = (span + 1) >> 1;
        int m = k + half;
        m = m >= K ? m - K : m;
        const float2 v = D.v[m];
        const bool after = (v.x - c.x) * y - (v.y - c.y) * x >= 0.0f;
        k = after ? m : k;
        span = after ? span - half : half - 1;
    }
    return k;
}

// Pocket of p: k if p is strictly right of v_k -> v_{k+1} in wedge k, else -1.
// `id` joins v_k's copies if p is one.
__device__ __forceinline__ int pocket_of(DenseLds& D, int K, float px, float py, int id, Counters& ctr)
{
    int k = wedge_guess(D, K, px, py);
    const float2 c = D.c;
    int n = k + 1 < K ? k + 1 : 0;
    float2 v = D.v[k], w = D.v[n];
    const Orient32 o0 = orient32p(c.x, c.y, v.x, v.y, px, py), o1 = orient32p(c.x, c.y, w.x, w.y, px, py);
    const Orient32 oe = orient32p(v.x, v.y, w.x, w.y, px, py);
    const bool sure = (o0.d > o0.es) & (o1.d < -o1.es) & (fabsf(oe.d) > oe.es);
    int s = oe.d < 0.0f ? k : -1;
    ctr.orient += 3;
    if (__ballot(!sure)) {
        if (!sure) {
            // the exact wedge: at or after ray k, before ray k + 1 (the guess
            // is at most a few wedges off; p = c belongs to none)
            ctr.orient_exact += 3;
            int tries = 0;
            bool in = false;
            for (; tries <= K; ++tries) {
                v = D.v[k];
                n = k + 1 < K ? k + 1 : 0;
                w = D.v[n];
                const int a = orient_exact(c.x, c.y, v.x, v.y, px, py), b = orient_exact(c.x, c.y, w.x, w.y, px, py);
                in = a >= 0 && b < 0;
                if (in) break;
                // (a wedge is less than half a turn wide: c is strictly inside the polygon)
                if (a < 0) k = k > 0 ? k - 1 : K - 1;
                else k = n;
            }
            s = -1;
            if (in) {
                if (px == v.x && py == v.y) atomicMin(&D.id[k], id);
                else if (orient_exact(v.x, v.y, w.x, w.y, px, py) < 0) s = k;
            }
        }
    }
    return s;
}

// Exact order about c of two points of one wedge: -1 if p comes before q. On
// one ray the nearer point comes first, copies by index.
__device__ __forceinline__ int around(float2 c, float2 p, int pid, float2 q, int qid)
{
    const int o = orient_exact(c.x, c.y, p.x, p.y, q.x, q.y);
    if (o != 0) return o > 0 ? -1 : 1;
    if (p.x != q.x) return (fabs((double)p.x - (double)c.x) < fabs((double)q.x - (double)c.x)) ? -1 : 1;
    if (p.y != q.y) return (fabs((double)p.y - (double)c.y) < fabs((double)q.y - (double)c.y)) ? -1 : 1;
    return pid < qid ? -1 : 1;
}

__device__ __forceinline__ int orient_of(float2 o, float2 e, float2 p, Counters& ctr)
{
    const Orient32 v = orient32p(o.x, o.y, e.x, e.y, p.x, p.y);
    ++ctr.orient;
    if (fabsf(v.d) > v.es) return v.d > 0.0f ? 1 : -1;
    ++ctr.orient_exact;
    return orient_exact(o.x, o.y, e.x, e.y, p.x, p.y);
}

// x of lane ^ D, without the LDS crossbar: row permutes up to 8, the row and half
// swaps above.
template <int D>
__device__ __forceinline__ uint32_t lane_xor(uint32_t x)
{
    constexpr int kQuad1 = 0xb1, kQuad2 = 0x4e, kQuad3 = 0x1b, kRor8 = 0x128, kHalfMirror = 0x141;
    const int v = (int)x;
    if (D == 1) return (uint32_t)__builtin_amdgcn_update_dpp(0, v, kQuad1, 0xf, 0xf, true);
    if (D == 2) return (uint32_t)__builtin_amdgcn_update_dpp(0, v, kQuad2, 0xf, 0xf, true);
    if (D == 4)
        return (uint32_t)__builtin_amdgcn_update_dpp(0, __builtin_amdgcn_update_dpp(0, v, kHalfMirror, 0xf, 0xf, true), kQuad3, 0xf,
                                                     0xf, true);
    if (D == 8) return (uint32_t)__builtin_amdgcn_update_dpp(0, v, kRor8, 0xf, 0xf, true);
    if (D == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        return (lane_id() & 16) ? r[0] : r[1];
    }
    const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return (lane_id() & 32) ? r[0] : r[1];
}

// One step of the sort below: elements D apart, in runs of SIZE.
template <int R, int SIZE, int D>
__device__ __forceinline__ void wave_sort_step(uint32_t (&k)[R])
{
    const int lane = lane_id();
    if constexpr (D >= R) {
        constexpr int LD = D / R;
        // (every register of a lane sorts the same way here)
        const bool up = ((lane * R) & SIZE) == 0, low = (lane & LD) == 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t o = lane_xor<LD>(k[r]);
            k[r] = (up == low) ? min(k[r], o) : max(k[r], o);
        }
    } else {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (r & D) continue;
            const bool up = ((lane * R + r) & SIZE) == 0;
            const uint32_t a = k[r], b = k[r + D], lo = min(a, b), hi = max(a, b);
            k[r] = up ? lo : hi;
            k[r + D] = up ? hi : lo;
        }
    }
    if constexpr (D > 1) wave_sort_step<R, SIZE, D / 2>(k);
}
// Sorts 64 R keys over the wave, element lane * R + r ascending (bitonic).
template <int R, int SIZE = 2>
__device__ __forceinline__ void wave_sort(uint32_t (&k)[R])
{
    wave_sort_step<R, SIZE, SIZE / 2>(k);
    if constexpr (SIZE < 64 * R) wave_sort<R, SIZE * 2>(k);
}

constexpr int kWavePts = 256;  // points of a wave's pocket
struct WaveLds {
    float2 xy[2][kWavePts];
    uint8_t at[2][kWavePts];  // each one's place among the pocket's points as loaded
    int id[kWavePts];
};

// Whether p comes before q about c, certainly: the float64 cross product beyond
// its rounding (differences and products: less than 2^-51 of the products' sum).
__device__ __forceinline__ bool before_sure(float2 c, float2 p, float2 q)
{
    const double P = ((double)p.x - c.x) * ((double)q.y - c.y), Q = ((double)p.y - c.y) * ((double)q.x - c.x);
    return P - Q > (fabs(P) + fabs(Q)) * 0x1p-50;
}

template <int R>
__device__ __forceinline__ void wave_order(WaveLds& W, int n, float2 c, float2 A, float2 B)
{
    const int lane = lane_id();
    const double ax = (double)A.x - c.x, ay = (double)A.y - c.y, bx = (double)B.x - c.x, by = (double)B.y - c.y;
    uint32_t key[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = lane + 64 * r;
        key[r] = 0xffffff00u | (uint32_t)(i & 255);
        if (i < n) {
            // 0 at A, 1 at B, increasing with the angle (in float64: a
            // narrow pocket's points look alike to float32)
            const float2 p = W.xy[0][i];
            const double x = (double)p.x - c.x, y = (double)p.y - c.y;
            const double u = ax * y - ay * x, v = x * by - y * bx;
            const float g = (float)u * __builtin_amdgcn_rcpf((float)(u + v));
            const float f = fminf(fmaxf(g, 0.0f), 1.0f);  // (NaN becomes 0: any order will do here)
            key[r] = (min((uint32_t)(f * 16777216.0f), 0xfffffeu) << 8) | (uint32_t)i;
        }
    }
    wave_sort<R>(key);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int e = lane * R + r, q = (int)(key[r] & 255u);
        if (e < n) {
            W.xy[1][e] = W.xy[0][q];
            W.at[1][e] = (uint8_t)q;
        }
    }
}

// One wave: the n <= 256 points W.xy[0], W.id in order about c and without
// those that are not strictly convex from A to B (points of the set), or, OPEN,
// between the first and the last of them (A and B only lie on rays around
// them). Returns how many are left and in which buffer (f).
template <bool OPEN>
__device__ __forceinline__ int wave_chain(WaveLds& W, int n, float2 c, float2 A, float2 B, int& f, Counters& ctr)
{
    const int lane = lane_id();
    if (n <= 64) wave_order<1>(W, n, c, A, B);
    else if (n <= 128) wave_order<2>(W, n, c, A, B);
    else wave_order<4>(W, n, c, A, B);
    wave_sync();
    // the rounded keys may have misplaced neighbours: exact sweeps until the
    // order holds
    bool unsure = false;
    for (int i = lane; i + 1 < n; i += 64) {
        const float2 p = W.xy[1][i], q = W.xy[1][i + 1];
        unsure |= !before_sure(c, p, q);
    }
    if (__ballot(unsure)) {
        for (int sweep = 0, still = 0; still < 2 && sweep < 2 * kWavePts + 2; ++sweep) {
            bool swapped = false;
            for (int i = 2 * lane + (sweep & 1); i + 1 < n; i += 128) {
                const float2 p = W.xy[1][i], q = W.xy[1][i + 1];
                if (before_sure(c, p, q)) continue;
                const uint8_t pa = W.at[1][i], qa = W.at[1][i + 1];
                ++ctr.orient_exact;
                if (around(c, p, W.id[pa], q, W.id[qa]) > 0) {
                    W.xy[1][i] = q; W.xy[1][i + 1] = p;
                    W.at[1][i] = qa; W.at[1][i + 1] = pa;
                    swapped = true;
                }
            }
            wave_sync();
            still = __ballot(swapped) ? 0 : still + 1;
        }
    }
    f = 1;
    for (;;) {
        int m = 0;
        for (int i0 = 0; i0 < n; i0 += 64) {
            const int i = i0 + lane;
            bool keep = false;
            float2 p = A;
            if (i < n) {
                p = W.xy[f][i];
                const float2 o = i > 0 ? W.xy[f][i - 1] : A, q = i + 1 < n ? W.xy[f][i + 1] : B;
                // a copy goes; the first of some copies waits for them to go
                const bool copy = (!OPEN || i > 0) && p.x == o.x && p.y == o.y;
                const bool twin = (!OPEN || i + 1 < n) && p.x == q.x && p.y == q.y;
                const bool end = OPEN && (i == 0 || i == n - 1);
                keep = !copy && (twin || end || orient_of(o, p, q, ctr) > 0);
            }
            const uint64_t M = __ballot(keep);
            if (keep) {
                const int d = m + bits_below(M);
                W.xy[f ^ 1][d] = p;
                W.at[f ^ 1][d] = W.at[f][i];
            }
            m += (int)__popcll(M);
        }
        wave_sync();
        f ^= 1;
        if (m == n) return m;
        n = m;
    }
}

}  // namespace sqh
