// Sieve of a point set by a polygon of its own points (device code, gfx950).
//
// The paper's first mode (section 4.2) drops the points inside a polygon of
// extreme points before the first split. Here the polygon is the hull of a
// strided sample, and its interior is tabulated as vertical slabs: slab b
// covers the x that map to b and holds a y interval such that every point of
// the slab with y strictly inside it lies in the polygon and is none of its
// vertices' positions, hence is no hull vertex of the set (a strict hull
// vertex inside the polygon is at a vertex of it, and copies of a polygon
// vertex stay: they decide the lowest index). A point costs one subtraction,
// one product, a conversion, one 8-byte LDS read and two comparisons.
#pragma once
#include "sqh_solve.hpp"

namespace sqh {

constexpr int kSetDense = -1;  // solve_set: too many vertices for one workgroup's LDS
constexpr int kSetBad = -2;    // ... a non-finite coordinate

struct Slabs {
    float x0, scale;  // slab of x: (x - x0) * scale, truncated, at most last
    uint32_t last;
};

__device__ __forceinline__ bool slab_inside(const Slabs& s, const float2* bins, float x, float y)
{
    const float f = (x - s.x0) * s.scale;
    // (the conversion takes negative values and NaN to 0, large ones to the top)
    const uint32_t b = min(__float2uint_rz(f), s.last);
    const float2 v = bins[b];
    return (y > v.x) & (y < v.y);
}

// largest float <= v / smallest float >= v
__device__ __forceinline__ float down32(double v)
{
    const float f = (float)v;
    return (double)f > v ? nextafterf(f, -INFINITY) : f;
}
__device__ __forceinline__ float up32(double v)
{
    const float f = (float)v;
    return (double)f < v ? nextafterf(f, INFINITY) : f;
}

// Slabs of the convex polygon v[0 .. h) (LDS, counter-clockwise from its
// lexicographic minimum; h < 3 gives empty slabs) into bins[0 .. NB). *kb (an
// LDS word) receives the place of its maximum. Starts and ends with a barrier.
//
// Slabs 0 and NB - 1 reach past the polygon's x range and stay empty; they
// cover almost none of it (2^-6 of a slab's width). The x of slab b lie in
// [x0 + b w (1 - 2^-20), x0 + (b + 1) w (1 + 2^-20)], w = 1 / scale (two
// float32 roundings move the quotient by less than 2^-22), widened by the
// rounding of the evaluation here (2^-48 |x0|). The lower chain is convex
// and the upper one concave, so their values at the two ends bound them on
// the slab; the evaluation in float64 errs by less than 2^-49 max |y|, and
// the interval is narrowed by 2^-40 max |y| before it is rounded inwards.
template <int T>
__device__ __forceinline__ Slabs build_slabs(const float2* v, int h, float2* bins, int NB, int* kb)
{
    const int t = (int)threadIdx.x;
    lds_barrier();
    if (t == 0 && h < 3) *kb = 0;
    if (h >= 3) {
        for (int r = t; r < h; r += T) {
            const float2 p = v[r], q = v[r + 1 < h ? r + 1 : 0], o = v[r > 0 ? r - 1 : h - 1];
            const bool after = (p.x > q.x || (p.x == q.x && p.y > q.y)) && (p.x > o.x || (p.x == o.x && p.y > o.y));
            if (after) *kb = r;  // the lexicographic maximum (one local maximum on a convex ring)
        }
    }
    lds_barrier();
    const int kB = *kb;
    auto pt = [&](int r) { return v[r >= h ? r - h : r]; };
    const float xa = h >= 3 ? v[0].x : 0.0f, xb = h >= 3 ? v[kB].x : 0.0f;
    const float ext = xb - xa;
    Slabs s;
    s.last = (uint32_t)(NB - 1);
    s.scale = ((float)(NB - 2) + 0x1p-5f) / ext;
    const bool ok = ext > 0x1p-100f && ext < 0x1p126f;
    if (!ok) {
        s.scale = 0.0f;
        s.x0 = 0.0f;
    } else {
        s.x0 = (float)((double)xa - (1.0 - 0x1p-6) / (double)s.scale);
    }
    const double w = ok ? 1.0 / (double)s.scale : 0.0, x0 = (double)s.x0, ex = fabs(x0) * 0x1p-48;
    for (int b = t; b < NB; b += T) {
        float2 iv = make_float2(INFINITY, -INFINITY);
        const double xl = x0 + (double)b * w * (1.0 - 0x1p-20) - ex, xr = x0 + (double)(b + 1) * w * (1.0 + 0x1p-20) + ex;
        if (ok && xl >= (double)xa && xr < (double)xb) {
            // the last node of the lower chain (0 .. kB) at or left of xl and
            // of xr, the last node of the upper chain (kB .. h) at or right of
            // them: four binary searches in step, their LDS reads together
            int l[4] = {0, 0, kB, kB}, u[4] = {kB, kB, h, h};
            for (int k = max(kB, h - kB); k > 1; k = (k + 1) >> 1) {
                float mx[4];
                int m[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) m[e] = (l[e] + u[e]) >> 1;
#pragma unroll
                for (int e = 0; e < 4; ++e) mx[e] = pt(m[e]).x;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const double x = (e & 1) ? xr : xl;
                    const bool go = (e < 2) ? ((double)mx[e] <= x) : ((double)mx[e] >= x);
                    const bool more = u[e] - l[e] > 1;
                    l[e] = (more & go) ? m[e] : l[e];
                    u[e] = (more & !go) ? m[e] : u[e];
                }
            }
            double lo = -INFINITY, hi = INFINITY, my = 0.0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float2 p = pt(l[e]), q = pt(l[e] + 1);
                const double x = (e & 1) ? xr : xl, dx = (double)q.x - (double)p.x;
                const double y = dx == 0.0 ? (double)p.y
                                           : (double)p.y + (x - (double)p.x) * ((double)q.y - (double)p.y) / dx;
                my = fmax(my, fmax(fabs((double)p.y), fabs((double)q.y)));
                if (e < 2) lo = fmax(lo, y);
                else hi = fmin(hi, y);
            }
            const double m = my * 0x1p-40 + 0x1p-160;
            iv.x = up32(lo + m);
            iv.y = down32(hi - m);
        }
        bins[b] = iv;
    }
    lds_barrier();
    return s;
}

// A polygon as two x-sorted chains: the last node of 0 .. kB - 1 at or left of x
// (l0), and of kB .. h - 1 at or right of it (l1).
__device__ __forceinline__ void chain_edges(const float2* v, int h, int kB, float x, int& l0, int& l1)
{
    int u0 = kB, u1 = h;
    l0 = 0;
    l1 = kB;
    for (int k = max(kB, h - kB); k > 1; k = (k + 1) >> 1) {
        const int m0 = (l0 + u0) >> 1, m1 = (l1 + u1) >> 1;
        const float x0 = v[m0].x, x1 = v[m1].x;
        const bool g0 = x0 <= x, g1 = x1 >= x, o0 = u0 - l0 > 1, o1 = u1 - l1 > 1;
        l0 = (o0 & g0) ? m0 : l0;
        u0 = (o0 & !g0) ? m0 : u0;
        l1 = (o1 & g1) ? m1 : l1;
        u1 = (o1 & !g1) ? m1 : u1;
    }
}

// Whether p is at a vertex of the polygon: at an end of its edges over p's x.
__device__ __forceinline__ bool chain_copy(const float2* v, int h, int kB, float x, float y)
{
    if (!(x >= v[0].x && x <= v[kB].x)) return false;
    int l0, l1;
    chain_edges(v, h, kB, x, l0, l1);
    const float2 q[4] = {v[l0], v[l0 + 1], v[l1], v[l1 + 1 < h ? l1 + 1 : 0]};
    bool at = false;
#pragma unroll
    for (int i = 0; i < 4; ++i) at |= q[i].x == x && q[i].y == y;
    return at;
}

// The same, exactly: true if p is in the closed polygon and at none of its
// vertices (so that it is no hull vertex; a copy of a vertex stays). The lower and the upper edge over its x are certified by
// the static line filter where it applies (line), else by the semi-static one;
// the points neither certifies, long collinear runs on the border among them,
// are settled exactly.
__device__ __forceinline__ bool chain_inside(const float2* v, int h, int kB, bool line, float Mx, float My, float x,
                                             float y, uint32_t& n_exact)
{
    const float2 A = v[0], B = v[kB];
    if (!(x >= A.x && x <= B.x)) return false;
    int l0, l1;
    chain_edges(v, h, kB, x, l0, l1);
    const float2 o[2] = {v[l0], v[l1]}, e[2] = {v[l0 + 1], v[l1 + 1 < h ? l1 + 1 : 0]};
    bool sure = x > A.x && x < B.x, out = false;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const float dx = e[k].x - o[k].x, dy = e[k].y - o[k].y;
        float d, m;
        if (line) {
            const float c = dy * o[k].x - dx * o[k].y;
            m = (fabsf(dx) * My + fabsf(dy) * Mx) * 0x1p-19f + kFilterTau;
            d = fmaf(-dy, x, fmaf(dx, y, c));
            if (!(fabsf(y) <= My)) d = 0.0f;  // (past the polygon's extent: not certified)
        } else {
            const Orient32 w = orient32p(o[k].x, o[k].y, e[k].x, e[k].y, x, y);
            d = w.d; m = w.es;
        }
        out |= d < -m;
        sure &= d > m;
    }
    if (out || sure) return sure && !out;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        ++n_exact;
        if (orient_exact(o[k].x, o[k].y, e[k].x, e[k].y, x, y) < 0) return false;
        if (o[k].x == e[k].x && !(y >= fminf(o[k].y, e[k].y) && y <= fmaxf(o[k].y, e[k].y))) return false;
        if ((x == o[k].x && y == o[k].y) || (x == e[k].x && y == e[k].y)) return false;
    }
    return true;
}

// Points i * n / m, i = 0 .. m - 1 (m <= P; all of them if m == n) into
// positions 0 .. m - 1. Sets L.bad on a non-finite coordinate. Returns m.
template <int T, int P>
__device__ __forceinline__ int load_points(SolveLds<P>& L, const float2* xy, int n, int m, const int* ids = nullptr)
{
    bool bad = false;
#pragma unroll
    for (int r = 0; r < P / T; ++r) {
        const int i = (int)threadIdx.x + T * r;
        if (i < m) {
            const int q = m == n ? i : (int)((long long)i * n / m);
            const float2 v = gld(xy + q);
            bad |= !((int)isfinite(v.x) & (int)isfinite(v.y));
            L.xy[i] = v;
            L.id[i] = ids ? gld(ids + q) : q;
        }
    }
    if (__ballot(bad) && lane_id() == 0) L.bad = 1;
    lds_barrier();
    return m;
}

// The hull of a set of n points: its ring in L.ring[0 .. h) (positions; L.id
// gives the indices). Returns h, kSetDense (more than a quarter of the sample,
// or more than P / 2 collected points, are vertices of their hull, or the sieve
// thins the set so little that it would be solved P points at a time: nothing
// is written) or kSetBad.
//
// Up to P points are solved as they are. A larger set is streamed past the
// slabs of its sample's hull; the points left are collected in LDS. Should
// they not fit, the collected points are replaced by their hull, whose slabs
// then sieve the rest.
// On kSetDense for the first reason, with nothing streamed yet, *sample is the
// ring size of the sample's hull (still in L); else 0.
template <int T, int P>
__device__ __forceinline__ int solve_set(SolveLds<P>& L, const float2* xy, int n, bool f64, Counters& ctr,
                                         SolveStats* st, int* sample)
{
    constexpr int U = 8;  // points per thread and step of the stream
    __shared__ int s_kb;
    __shared__ int s_tot[3];
    const int t = (int)threadIdx.x;
    if (n == 0) return 0;
    // the sample: a sixteenth of the set, at least T points (a larger one
    // sieves better but its own hull takes longer)
    int cnt = load_points<T, P>(L, xy, n, n <= P ? n : min(P, max(T, n >> 4)));
    bool fin = n <= P, first = true;
    int pos = 0;
    for (;;) {
        if (L.bad) return kSetBad;
        const int h = solve<T, P, true>(L, cnt, 0, 0, f64, ctr, fin ? st : nullptr);
        if (fin) return h;
        // about h / cnt of the points would pass the sieve: a set that keeps
        // more than a quarter (a ring of points) is not for it
        if (4 * h > cnt && (first || h > P / 2)) {
            *sample = first ? h : 0;
            return kSetDense;
        }
        // (the ring's coordinates past the slabs, in order)
        static_assert(T + P / 2 <= P, "slabs and ring share the keys' space");
        for (int r = t; r < h; r += T) L.bins[T + r] = L.xy[L.ring[r]];
        const Slabs sl = build_slabs<T>(L.bins + T, h, L.bins, T, &s_kb);
        if (first) {
            // the sample's vertices come back with the stream
            first = false;
            cnt = 0;
        } else {
            float2 v[P / 2 / T];
            int id[P / 2 / T];
#pragma unroll
            for (int r = 0; r < P / 2 / T; ++r) {
                const int i = t + T * r;
                if (i < h) { v[r] = L.xy[L.ring[i]]; id[r] = L.id[L.ring[i]]; }
            }
            lds_barrier();
#pragma unroll
            for (int r = 0; r < P / 2 / T; ++r) {
                const int i = t + T * r;
                if (i < h) { L.xy[i] = v[r]; L.id[i] = id[r]; }
            }
            cnt = h;
        }
        if (t < 3) s_tot[t] = 0;
        lds_barrier();
        int k = 0;
        bool small = false, bad = false;
        float2 nv[U];  // the next step's points, loaded a step ahead
        auto fetch = [&](int at) {
            if (at + T * U <= n) {
                // one uniform base per row, the same lane offset
#pragma unroll
                for (int j = 0; j < U; ++j) nv[j] = gld(xy + at + T * j + t);
            } else {
#pragma unroll
                for (int j = 0; j < U; ++j) nv[j] = gld(xy + min(at + t + T * j, n - 1));
            }
        };
        const int from = pos;
        fetch(pos);
        while (pos < n) {
            // one step: U rows of T points, or one row where U might not fit
            const int u = small ? 1 : U;
            float2 v[U];
            uint32_t keep = 0u;
#pragma unroll
            for (int j = 0; j < U; ++j) v[j] = nv[j];
            fetch(min(pos + T * u, n - 1));
            int wc = 0;
#pragma unroll
            for (int j = 0; j < U; ++j) keep |= (uint32_t)!slab_inside(sl, L.bins, v[j].x, v[j].y) << j;
            if (small || pos + T * U > n) {
#pragma unroll
                for (int j = 0; j < U; ++j)
                    if (j >= u || pos + t + T * j >= n) keep &= ~(1u << j);
            }
            if (__ballot(keep != 0u)) {
#pragma unroll
                for (int j = 0; j < U; ++j) {
                    const bool kp = (keep >> j) & 1u;
                    // (a non-finite coordinate is inside no slab)
                    bad |= kp & !((int)isfinite(v[j].x) & (int)isfinite(v[j].y));
                    wc += __popcll(__ballot(kp));
                }
            }
            int base = 0;
            if (lane_id() == 0 && wc) base = atomicAdd(&s_tot[k], wc);
            base = __builtin_amdgcn_readfirstlane(base);
            lds_barrier();
            const int tot = s_tot[k];
            if (t == 0) s_tot[k == 0 ? 2 : k - 1] = 0;  // (last read before this barrier, next used after the next one)
            k = k == 2 ? 0 : k + 1;
            if (cnt + tot > P) {  // (uniform)
                if (small) break;
                small = true;
                fetch(pos);
                continue;
            }
            int w = cnt + base;
            if (wc) {
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const bool kp = (keep >> j) & 1u;
                const uint64_t M = __ballot(kp);
                if (kp) {
                    const int d = w + bits_below(M);
                    L.xy[d] = v[j];
                    L.id[d] = pos + t + T * j;
                }
                w += (int)__popcll(M);
            }
            }
            cnt += tot;
            pos += T * u;
        }
        if (__ballot(bad) && lane_id() == 0) L.bad = 1;
        fin = pos >= n;
        lds_barrier();
        // (copies, or points on a line: 16 solves of 4096 of them take 0.25 ms,
        // and a million 4 ms; other paths drop them at the first split)
        if ((n - pos) / 16 > pos - from) {  // (uniform)
            *sample = 0;
            return L.bad ? kSetBad : kSetDense;
        }
    }
}

}  // namespace sqh
