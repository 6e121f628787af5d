// The pre-filter of single hulls: its extremes and its test (device code,
// gfx950).
//
// The paper's first mode (section 4.2) drops the points inside the
// quadrilateral of the extreme points in x and y before the first split;
// the octagon adds the extremes of x + y and x - y.
//
// Corner k is, among the points whose projection on direction k is extreme,
// the one of lowest index; the diagonal projections are the float32 sums
// fl(x + y) and fl(x - y), and -0 counts as +0. Directions, counter-clockwise
// from -x:
//   0 min x   1 min x + y   2 min y   3 max x - y
//   4 max x   5 max x + y   6 max y   7 min x - y
// Neither the rounding nor the tie rule matters for the hull. The corners
// are input points; a point strictly left of every edge of the closed
// polygon through them sees each edge turn by a positive angle, so its
// winding number is positive and it lies in the interior of the corners'
// convex hull, hence of the input's: it is no hull vertex. A point at a
// corner's position is on an edge that starts there, so it is never
// certified inside; if all corners coincide there is no edge and every
// point is kept. The subset (points not certified inside, with their input
// indices) therefore holds every hull vertex and every copy of one, and its
// hull, tie rules included, is the input's. "Strictly left" is certified by
// the float32 orientation filter; an overflow in it makes the bound
// infinite or NaN, which certifies nothing.
#pragma once
#include "sqh_pred.hpp"

namespace sqh {

// order-preserving map of a float32 onto uint32 (for non-NaN values)
__device__ __forceinline__ uint32_t ord32(float f)
{
    const uint32_t u = __float_as_uint(f);
    return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}

// Directions 3, 4, 5, 6 take the largest projection, the others the
// smallest. Across lanes and workgroups an extreme is carried as one 64-bit
// key: high word the projection's order, low word the index (smallest-key
// directions) or its complement (largest-key directions), so that the
// extreme key names the lowest index among the extreme projections.
constexpr uint32_t kExtMax = 0x78u;

__device__ __forceinline__ bool ext_is_max(int k) { return (kExtMax >> k) & 1u; }
__device__ __forceinline__ uint64_t ext_none(int k) { return ext_is_max(k) ? 0ull : ~0ull; }
__device__ __forceinline__ uint64_t ext_key(int k, float v, int id)
{
    if (id < 0) return ext_none(k);
    const uint32_t o = ord32(v + 0.0f);  // -0 -> +0
    return ((uint64_t)o << 32) | (ext_is_max(k) ? ~(uint32_t)id : (uint32_t)id);
}
__device__ __forceinline__ uint64_t ext_pick(int k, uint64_t a, uint64_t b)
{
    return ext_is_max(k) ? (a > b ? a : b) : (a < b ? a : b);
}
// (0 if all projections overflowed: any point will do for a corner)
__device__ __forceinline__ int ext_index(int k, uint64_t key)
{
    const uint32_t lo = (uint32_t)key;
    return max((int)(ext_is_max(k) ? ~lo : lo), 0);
}

// One lane's extremes: its points come in increasing index order, so a
// strict comparison keeps the lowest index among equal projections.
struct ExtLane {
    float v[8];
    int id[8];
    __device__ __forceinline__ void init()
    {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            v[k] = ext_is_max(k) ? -INFINITY : INFINITY;
            id[k] = -1;
        }
    }
    __device__ __forceinline__ void add(float x, float y, int q)
    {
        const float s = x + y, d = x - y;
        const float pr[8] = {x, s, y, d, x, s, y, d};
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const bool t = ext_is_max(k) ? (pr[k] > v[k]) : (pr[k] < v[k]);
            v[k] = t ? pr[k] : v[k];
            id[k] = t ? q : id[k];
        }
    }
};

__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int m)
{
    const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)v, m);
    const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(v >> 32), m);
    return ((uint64_t)hi << 32) | lo;
}

__device__ __forceinline__ float rfl_f(float v)
{
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// The polygon's non-degenerate edges, wave-uniform (n = 0: all corners
// coincide, every point is kept).
//
// Line test (|coordinates| <= 2^60): edge o -> o + (dx, dy) (dx, dy rounded)
// as t = fma(nx, px, fma(ny, py, c)), nx = -dy, ny = dx, c = fl(fl(dy ox) -
// fl(dx oy)). With D = |dx| My + |dy| Mx, where Mx, My bound |x|, |y| over
// the input (the extremes in x and y), the rounding of the differences, of
// c and of both fma's moves t from the exact orientation of (o, e, p) by at
// most 9 u D (1 + 10 u) plus 5 * 2^-150 in the subnormal range (u = 2^-24),
// so t > m = 2^-19 D + 2^-140 (32 u D) proves the orientation positive. The
// bound on the coordinates keeps every term below 2^123 (no overflow).
// Larger coordinates use the float32 orientation filter, whose overflow
// gives an infinite or NaN bound and certifies nothing.
constexpr float kLineCoordMax = 0x1p60f;
constexpr float kLineRel = 0x1p-19f;

struct KeepEdges {
    float nx[8], ny[8], c[8], m[8];
    int n;
    bool line;  // the line test applies (else the orientation filter)
};

// edges in LDS for the orientation filter: ox, oy, dx, dy per edge
struct KeepLds {
    float e[4][8];
};

// corners cx, cy in direction order (the quadrilateral uses the even ones)
__device__ __forceinline__ void keep_build(KeepEdges& E, KeepLds& L, const float (&cx)[8], const float (&cy)[8],
                                           bool quad)
{
    const float Mx = fmaxf(fabsf(cx[0]), fabsf(cx[4]));  // min x, max x
    const float My = fmaxf(fabsf(cy[2]), fabsf(cy[6]));  // min y, max y
    E.line = fmaxf(Mx, My) <= kLineCoordMax;
    E.n = 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) E.nx[i] = E.ny[i] = E.c[i] = E.m[i] = 0.0f;
    const bool w0 = threadIdx.x == 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        if (quad && (i & 1)) continue;
        const int j = quad ? ((i + 2) & 7) : ((i + 1) & 7);
        if (cx[i] == cx[j] && cy[i] == cy[j]) continue;  // zero-length edge
        const float dx = cx[j] - cx[i], dy = cy[j] - cy[i];
        const float cc = dy * cx[i] - dx * cy[i];
        const float mm = (fabsf(dx) * My + fabsf(dy) * Mx) * kLineRel + kFilterTau;
        // (placed with selects so that the arrays stay in registers)
#pragma unroll
        for (int t = 0; t < 8; ++t) {
            if (t == E.n) {
                E.nx[t] = -dy;
                E.ny[t] = dx;
                E.c[t] = cc;
                E.m[t] = mm;
                if (w0) {
                    L.e[0][t] = cx[i];
                    L.e[1][t] = cy[i];
                    L.e[2][t] = dx;
                    L.e[3][t] = dy;
                }
            }
        }
        ++E.n;
    }
}

// keep p: not certified strictly left of every edge
__device__ __forceinline__ bool keep_point(const KeepEdges& E, const KeepLds& L, float px, float py, Counters& ctr)
{
    if (E.n == 0) return true;
    bool in = true;
    if (E.line) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (i < E.n) in = in && fmaf(E.nx[i], px, fmaf(E.ny[i], py, E.c[i])) > E.m[i];
        }
    } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if (i < E.n) {
                const float P = L.e[2][i] * (py - L.e[1][i]);
                const float Q = L.e[3][i] * (px - L.e[0][i]);
                const float d = P - Q;
                const float es = (fabsf(P) + fabsf(Q)) * kFilterScale + kFilterTau;
                in = in && d > es;
            }
        }
    }
    ctr.orient += (uint32_t)E.n;
    return !in;
}

}  // namespace sqh
