// The hull of one small point set, or the chain of one segment, by one
// workgroup with everything in LDS (device code, gfx950).
//
// QuickHull of sections 4.3 - 4.4 without moving coordinates: a pass
// classifies the live points, a packed list of positions, against A->C and
// C->B of their segment (section 4.4.3), finds the farthest point of every
// child (section 4.4.1) with one 64-bit LDS maximum per point, appends the
// points kept to the next pass's list, and replaces the segment table by its
// children (sections 4.4.2, 4.4.4). The ring is a linked list (next vertex of
// each vertex), put in order at the end by pointer jumping. The set's first
// split is the same step on one pseudo segment A -> B -> A.
//
// What bounds it: one compute unit's instruction issue while many points are
// live (about 100 instructions a point and pass), then latency: a pass has
// three barriers and a chain of six dependent LDS reads.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sqh_pred.hpp"
#include "sqh_chunk.hpp"

namespace sqh {

// ---- small helpers ----

// float -> unsigned with the same order (no NaN)
__device__ __forceinline__ uint32_t order_key(float f)
{
    const uint32_t u = __float_as_uint(f);
    return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}

__device__ __forceinline__ uint64_t dpp_u64(uint64_t v, uint64_t ident, const int step)
{
    // lanes without a source take `ident` (the reduction's identity)
    const int il = (int)(uint32_t)ident, ih = (int)(uint32_t)(ident >> 32);
    const int l = (int)(uint32_t)v, h = (int)(uint32_t)(v >> 32);
    int rl, rh;
    switch (step) {
    case 0: rl = __builtin_amdgcn_update_dpp(il, l, 0x111, 0xf, 0xf, false);
            rh = __builtin_amdgcn_update_dpp(ih, h, 0x111, 0xf, 0xf, false); break;  // row_shr:1
    case 1: rl = __builtin_amdgcn_update_dpp(il, l, 0x112, 0xf, 0xf, false);
            rh = __builtin_amdgcn_update_dpp(ih, h, 0x112, 0xf, 0xf, false); break;  // row_shr:2
    case 2: rl = __builtin_amdgcn_update_dpp(il, l, 0x114, 0xf, 0xf, false);
            rh = __builtin_amdgcn_update_dpp(ih, h, 0x114, 0xf, 0xf, false); break;  // row_shr:4
    case 3: rl = __builtin_amdgcn_update_dpp(il, l, 0x118, 0xf, 0xf, false);
            rh = __builtin_amdgcn_update_dpp(ih, h, 0x118, 0xf, 0xf, false); break;  // row_shr:8
    case 4: rl = __builtin_amdgcn_update_dpp(il, l, 0x142, 0xa, 0xf, false);
            rh = __builtin_amdgcn_update_dpp(ih, h, 0x142, 0xa, 0xf, false); break;  // row_bcast:15
    default: rl = __builtin_amdgcn_update_dpp(il, l, 0x143, 0xc, 0xf, false);
             rh = __builtin_amdgcn_update_dpp(ih, h, 0x143, 0xc, 0xf, false); break;  // row_bcast:31
    }
    return ((uint64_t)(uint32_t)rh << 32) | (uint32_t)rl;
}
// The wave's smallest / largest value, in lane 63 (every lane active).
__device__ __forceinline__ uint64_t wave_min_u64(uint64_t v)
{
#pragma unroll
    for (int s = 0; s < 6; ++s) {
        const uint64_t o = dpp_u64(v, ~0ull, s);
        v = o < v ? o : v;
    }
    return v;
}
__device__ __forceinline__ uint64_t wave_max_u64(uint64_t v)
{
#pragma unroll
    for (int s = 0; s < 6; ++s) {
        const uint64_t o = dpp_u64(v, 0ull, s);
        v = o > v ? o : v;
    }
    return v;
}

// A workgroup barrier that orders LDS accesses only: global stores in flight
// need not complete first.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Orders a wave's own LDS accesses across its lanes (they execute in order).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ int bits_below(uint64_t M)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(M >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)M, 0u));
}

// Whether an earlier kernel of the call ended it (err | left), alike on every
// wave of the workgroup: one thread reads the words, because a kernel whose
// workgroups also set them may have set them between two waves' own reads, and
// a workgroup that goes on without some of its waves works on LDS they never
// wrote. Every thread calls it; it holds a barrier. (A word that the kernel does
// not set can be read by each wave: BatchCtl::stop.)
__device__ __forceinline__ bool call_ended(const int* err, const int* left)
{
    __shared__ int s_ended;
    if (threadIdx.x == 0)
        s_ended = __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) |
                  __hip_atomic_load(left, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    return s_ended != 0;
}

// Exact order of two distinct candidates for the edge o -> e (section 4.4.1;
// ties: the point earliest along the edge, then the lower index).
__device__ __forceinline__ bool farther_exact(float2 o, float2 e, float2 p, int pid, float2 q, int qid)
{
    if (p.x == q.x && p.y == q.y) return pid < qid;
    const int s = area_cmp_exact(o.x, o.y, e.x, e.y, p.x, p.y, q.x, q.y);
    if (s != 0) return s > 0;
    const bool fwd = (e.x > o.x) || (e.x == o.x && e.y > o.y);
    const bool p_first = (p.x < q.x) || (p.x == q.x && p.y < q.y);
    return fwd ? p_first : !p_first;
}

// ---- the solver ----

constexpr int kSolvePasses = 64;  // passes whose sizes are noted
// Coordinates beyond this make a set's areas be bounded by the high words of
// float64 intervals (a point's products may overflow in float32, and with no
// bounds every point challenges its child's leader exactly: 35K points scaled
// by 1e34 took a batch 25 ms).
// So are sets whose coordinates all stay below kFineFrom: their areas come near
// the bounds' underflow margin of 2^-140 (742K points scaled by 1e-23: 8.4 ms).
constexpr float kWideFrom = 0x1p62f, kFineFrom = 0x1p-56f;
// The bounds: the smaller one in the low word. Out of line, so that the float32
// form keeps its registers (inlined it cost k_batch_big 4 %).
__device__ __noinline__ uint64_t area_bounds64(float ox, float oy, float ex, float ey, float px, float py)
{
    double m;
    const double d = -orient64(ox, oy, ex, ey, px, py, m);
    return ((uint64_t)((uint32_t)__double2hiint(d + m) + 1u) << 32) | (uint32_t)__double2hiint(fmax(d - m, 0.0));
}
constexpr uint16_t kNoNext = 0xffffu;

struct LSegIdx {
    uint16_t a, c, b, pad;  // positions of A, the farthest point C and B
};

// P points. At every pass S <= P / 2: every active segment is an edge of the
// ring found so far, whose vertices are no longer live, and holds a live
// point, so 2 S <= P.
template <int P>
struct SolveLds {
    float2 xy[P];
    int id[P];
    uint16_t next[P];
    union {
        uint64_t key[P];   // per child: largest lower bound of the area, ~position
        float2 bins[P];    // between solves: the sieve's slabs
    };
    union {
        LSegIdx seg[2][P / 2];
        struct { uint16_t jn[2][P], jd[2][P]; };  // ordering: pointer, distance
    };
    union {
        uint16_t map[P];   // child -> segment of the next pass; flags while a leader is settled
        uint16_t ring[P];  // after the solve: vertex positions in ring order
    };
    uint16_t list[2][P];   // live positions of the pass and of the next one
    uint16_t chd[P];       // per live position: its child in the pass before
    uint64_t kmin, kmax, imin, imax;
    int ns[2], any[2], beat[2];
    int live[2];           // lengths of the lists
    int bad;
    int wide, fine;        // a coordinate is so large that float32 products may overflow; one is no tiny number
};

// What a call adds up over the sets one workgroup solves.
struct SolveStats {
    int passes;                                  // passes after the first compaction (the largest of them)
    int pass_v[kSolvePasses], pass_s[kSolvePasses];
};

template <int P>
__device__ __forceinline__ void note_scale(SolveLds<P>& L, float top)
{
    const bool w = __ballot(top > kWideFrom) != 0ull, f = __ballot(top >= kFineFrom) != 0ull;
    if (lane_id() == 0) {
        if (w) L.wide = 1;
        if (f) L.fine = 1;
    }
}

// Solves the points 0 .. cnt-1 of L (cnt >= 1; WHOLE) or the chain from A at
// position ia to B at ib (both below cnt) over every other position, all of
// them strictly right of A -> B. Returns the number of list nodes: the ring's
// vertices, or A and the chain's vertices; L.ring[r] is the position of node
// r (A is node 0). Every thread of the T-thread workgroup calls it; L.xy and
// L.id must be visible.
template <int T, int P, bool WHOLE>
__device__ __forceinline__ int solve(SolveLds<P>& L, int cnt, int ia, int ib, bool f64, Counters& ctr,
                                     SolveStats* st)
{
    constexpr int R = P / T, kPair = R > 1 ? 2 : 1;
    static_assert(R % kPair == 0, "points go in pairs");
    static_assert(P % T == 0 && P <= 0xfff0, "positions are 16-bit");
    const int t = (int)threadIdx.x, lane = lane_id();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = t + T * r;
        if (i < cnt) {
            L.next[i] = kNoNext;
            L.list[0][i] = (uint16_t)i;
            L.chd[i] = 0;
        }
        L.key[i] = 0ull;
    }
    if (t == 0) {
        L.kmin = ~0ull; L.kmax = 0ull;
        L.imin = ~0ull; L.imax = ~0ull;
        L.ns[0] = 1; L.ns[1] = 0;
        L.any[0] = 0; L.any[1] = 0;
        L.beat[0] = 0; L.beat[1] = 0;
        L.live[0] = cnt; L.live[1] = 0;
        L.map[0] = 0;
        L.wide = 0; L.fine = 0;
    }
    lds_barrier();
    float top_abs = 0.0f;
    // the first segment's "farthest point" is B itself: its children are the
    // sides of A -> B and, for a set, of B -> A
    int ic = ib;
    if constexpr (WHOLE) {
        // A and B: the lexicographic extremes, the lowest index among copies
        uint64_t k[R], lo = ~0ull, hi = 0ull;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = t + T * r;
            const float2 p = i < cnt ? L.xy[i] : make_float2(0.0f, 0.0f);
            top_abs = fmaxf(top_abs, fmaxf(fabsf(p.x), fabsf(p.y)));
            // (+ 0.0f: -0 counts as +0)
            k[r] = ((uint64_t)order_key(p.x + 0.0f) << 32) | order_key(p.y + 0.0f);
            if (i < cnt) {
                lo = k[r] < lo ? k[r] : lo;
                hi = k[r] > hi ? k[r] : hi;
            }
        }
        note_scale(L, top_abs);
        lo = wave_min_u64(lo);
        hi = wave_max_u64(hi);
        if (lane == 63) {
            atomicMin((unsigned long long*)&L.kmin, (unsigned long long)lo);
            atomicMax((unsigned long long*)&L.kmax, (unsigned long long)hi);
        }
        lds_barrier();
        const uint64_t kmin = L.kmin, kmax = L.kmax;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (t + T * r < cnt && (k[r] == kmin || k[r] == kmax)) {
                const uint64_t v = ((uint64_t)(uint32_t)L.id[t + T * r] << 32) | (uint32_t)(t + T * r);
                if (k[r] == kmin) atomicMin((unsigned long long*)&L.imin, (unsigned long long)v);
                if (k[r] == kmax) atomicMin((unsigned long long*)&L.imax, (unsigned long long)v);
            }
        }
        lds_barrier();
        ia = (int)(uint32_t)L.imin;
        ib = (int)(uint32_t)L.imax;
        if (kmin == kmax) {  // one position: its lowest index
            if (t == 0) L.ring[0] = (uint16_t)ia;
            lds_barrier();
            return 1;
        }
        ic = ib;
        ib = ia;
    } else {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = t + T * r;
            if (i < cnt) top_abs = fmaxf(top_abs, fmaxf(fabsf(L.xy[i].x), fabsf(L.xy[i].y)));
        }
        note_scale(L, top_abs);
    }
    if (t == 0) {
        LSegIdx g;
        g.a = (uint16_t)ia; g.c = (uint16_t)ic; g.b = (uint16_t)ib; g.pad = 0;
        L.seg[0][0] = g;
    }
    lds_barrier();
    // the bounds of areas in float64, where float32 has none (or may not be asked)
    const bool wide = f64 || L.wide != 0 || L.fine == 0;
    int nodes = WHOLE ? 1 : 0;  // (pass 0 adds B to a ring, or counts A)
    int pass = 0;
    for (;; ++pass) {
        const int c = pass & 1, S = L.ns[c];
        if (S == 0) break;  // (uniform)
        const int sp = WHOLE ? pass - 2 : pass - 1;  // (a set's passes 0 and 1 are the split and the first compaction)
        if (st && t == 0 && sp >= 0 && sp < kSolvePasses) st->pass_s[sp] += S;
        // 1. each live point: its child and the child's largest lower bound.
        // Points go two at a time without branches, so that their LDS reads
        // are in flight together.
        const int V = L.live[c];
        float2 p[R];
        int pos[R], ch[R];
        uint32_t lok[R], hik[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            ch[r] = -1;
            pos[r] = 0;
            lok[r] = 0u; hik[r] = 0u;
            p[r] = make_float2(0.0f, 0.0f);
        }
#pragma unroll
        for (int r0 = 0; r0 < R; r0 += kPair) {
            if (T * r0 + (t & ~63) >= V) continue;  // (uniform in a wave)
            LSegIdx g[kPair];
            float2 A[kPair], C[kPair], B[kPair];
            int lab[kPair];
#pragma unroll
            for (int k = 0; k < kPair; ++k) pos[r0 + k] = (int)L.list[c][min(t + T * (r0 + k), V - 1)];
#pragma unroll
            for (int k = 0; k < kPair; ++k) { lab[k] = L.chd[pos[r0 + k]]; p[r0 + k] = L.xy[pos[r0 + k]]; }
#pragma unroll
            for (int k = 0; k < kPair; ++k) lab[k] = L.map[lab[k]];
#pragma unroll
            for (int k = 0; k < kPair; ++k) g[k] = L.seg[c][lab[k]];
#pragma unroll
            for (int k = 0; k < kPair; ++k) { A[k] = L.xy[g[k].a]; C[k] = L.xy[g[k].c]; B[k] = L.xy[g[k].b]; }
            Orient32 o1[kPair], o2[kPair];
            int s1[kPair], s2[kPair];
            bool lv[kPair], und = false;
#pragma unroll
            for (int k = 0; k < kPair; ++k) {
                const int r = r0 + k, i = pos[r];
                // A, B and C themselves leave (their copies are settled exactly)
                lv[k] = (t + T * r < V) & (i != g[k].a) & (i != g[k].c) & (i != g[k].b);
                o1[k] = orient32p(A[k].x, A[k].y, C[k].x, C[k].y, p[r].x, p[r].y);
                o2[k] = orient32p(C[k].x, C[k].y, B[k].x, B[k].y, p[r].x, p[r].y);
                const bool ok1 = !f64 & (fabsf(o1[k].d) > o1[k].es), ok2 = !f64 & (fabsf(o2[k].d) > o2[k].es);
                s1[k] = ok1 ? (o1[k].d > 0.0f ? 1 : -1) : 0;
                s2[k] = ok2 ? (o2[k].d > 0.0f ? 1 : -1) : 0;
                und |= lv[k] & ((s1[k] == 0) | ((s1[k] > 0) & (s2[k] == 0)));
                ctr.orient += lv[k] ? 2u : 0u;
            }
            if (__ballot(und)) {
#pragma unroll
                for (int k = 0; k < kPair; ++k) {
                    const float2 q = p[r0 + k];
                    settle_p(s1[k], lv[k] && s1[k] == 0, A[k].x, A[k].y, C[k].x, C[k].y, q.x, q.y, ctr.orient_exact);
                    settle_p(s2[k], lv[k] && s1[k] >= 0 && s2[k] == 0, C[k].x, C[k].y, B[k].x, B[k].y, q.x, q.y,
                             ctr.orient_exact);
                }
            }
            uint64_t key[kPair], top[kPair];
#pragma unroll
            for (int k = 0; k < kPair; ++k) {
                const int r = r0 + k;
                const bool in0 = s1[k] < 0, in1 = !in0 & (s2[k] < 0), in = lv[k] & (in0 | in1);
                const float a = -(in0 ? o1[k].d : o2[k].d), w = 2.0f * (in0 ? o1[k].es : o2[k].es);
                // the area is positive, so the bounds order as their bits;
                // a NaN (overflow) leaves the whole range
                lok[r] = __float_as_uint(fmaxf(a - w, 0.0f));
                hik[r] = __float_as_uint(fminf(a + w, INFINITY));
                ch[r] = in ? 2 * lab[k] + (in0 ? 0 : 1) : -1;
            }
            if (wide) {  // (uniform)
#pragma unroll
                for (int k = 0; k < kPair; ++k) {
                    const int r = r0 + k;
                    const bool in0 = s1[k] < 0;
                    const float2 o = in0 ? A[k] : C[k], e = in0 ? C[k] : B[k];
                    const uint64_t b = area_bounds64(o.x, o.y, e.x, e.y, p[r].x, p[r].y);
                    lok[r] = (uint32_t)b;
                    hik[r] = (uint32_t)(b >> 32);
                }
            }
#pragma unroll
            for (int k = 0; k < kPair; ++k) {
                const int r = r0 + k;
                key[k] = ((uint64_t)lok[r] << 32) | (uint32_t)~pos[r];
                top[k] = L.key[max(ch[r], 0)];
            }
#pragma unroll
            for (int k = 0; k < kPair; ++k) {
                const int r = r0 + k;
                const uint64_t M = __ballot(ch[r] >= 0);
                int at = 0;
                if (lane == 0 && M) at = atomicAdd(&L.live[c ^ 1], (int)__popcll(M));
                at = __builtin_amdgcn_readfirstlane(at);
                if (ch[r] >= 0) {
                    if (key[k] > top[k])
                        atomicMax((unsigned long long*)&L.key[ch[r]], (unsigned long long)key[k]);
                    L.list[c ^ 1][at + bits_below(M)] = (uint16_t)pos[r];
                    L.chd[pos[r]] = (uint16_t)ch[r];
                }
            }
        }
        if (t == 0) {
            L.ns[c ^ 1] = 0;   // (last read at the top of the pass before)
            L.any[c ^ 1] = 0;
        }
        lds_barrier();
        // 2. points whose interval reaches the leader's lower bound
        uint32_t cand = 0u;
        {
            uint64_t top[R];
#pragma unroll
            for (int r = 0; r < R; ++r) top[r] = L.key[max(ch[r], 0)];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const bool m = (ch[r] >= 0) & ((int)~(uint32_t)top[r] != pos[r]) &
                               (hik[r] >= (uint32_t)(top[r] >> 32));
                cand |= (uint32_t)m << r;
            }
        }
        if (__ballot(cand != 0u) && lane == 0) L.any[c] = 1;
        lds_barrier();
        if (L.any[c]) {  // (uniform)
            // settle them exactly against the leader; a beaten leader steps
            // down and its challengers elect the one of lowest index among them
            // (copies of one point agree at once: by position they took seven
            // rounds for 178 copies, and 53 chunks of them 1.5 ms)
            for (int u = t; u < 2 * S; u += T) L.map[u] = 0;
            lds_barrier();
            for (int round = 0;; ++round) {
                const int fb = round & 1;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    if ((cand >> r) & 1u) {
                        const int u = ch[r], l = (int)~(uint32_t)L.key[u];
                        const LSegIdx g = L.seg[c][u >> 1];
                        const float2 o = (u & 1) ? L.xy[g.c] : L.xy[g.a], e = (u & 1) ? L.xy[g.b] : L.xy[g.c];
                        ++ctr.cmp_exact;
                        if (farther_exact(o, e, p[r], L.id[pos[r]], L.xy[l], L.id[l])) {
                            L.map[u] = 1;
                            L.beat[fb] = 1;
                        } else {
                            cand &= ~(1u << r);
                        }
                    }
                }
                lds_barrier();
                if (!L.beat[fb]) break;  // (uniform)
                for (int u = t; u < 2 * S; u += T)
                    if (L.map[u]) L.key[u] = 0ull;
                if (t == 0) L.beat[fb ^ 1] = 0;
                lds_barrier();
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    // (a candidate left here beat its child's old leader)
                    if ((cand >> r) & 1u)
                        atomicMax((unsigned long long*)&L.key[ch[r]],
                                  (unsigned long long)(((uint64_t)~(uint32_t)L.id[pos[r]] << 32) | (uint32_t)~pos[r]));
                }
                for (int u = t; u < 2 * S; u += T) L.map[u] = 0;
                lds_barrier();
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (((cand >> r) & 1u) && (int)~(uint32_t)L.key[ch[r]] == pos[r]) cand &= ~(1u << r);
            }
            if (t == 0) { L.beat[0] = 0; L.beat[1] = 0; }
        }
        // 3. C joins the ring; the children replace the segments
        const int nl = L.live[c ^ 1];
        if (st && t == 0 && sp + 1 >= 0 && sp + 1 < kSolvePasses) st->pass_v[sp + 1] += nl;
        for (int s0 = 0; s0 < S; s0 += T) {
            const int s = s0 + t;
            uint64_t k0 = 0ull, k1 = 0ull;
            LSegIdx g = {};
            if (s < S) {
                k0 = L.key[2 * s];
                k1 = L.key[2 * s + 1];
                L.key[2 * s] = 0ull;
                L.key[2 * s + 1] = 0ull;
                g = L.seg[c][s];
                L.next[g.a] = g.c;
                L.next[g.c] = g.b;
            }
            const uint64_t M0 = __ballot(k0 != 0ull), M1 = __ballot(k1 != 0ull);
            int b0 = 0;
            if (lane == 0 && (M0 | M1)) b0 = atomicAdd(&L.ns[c ^ 1], (int)(__popcll(M0) + __popcll(M1)));
            b0 = __builtin_amdgcn_readfirstlane(b0);
            if (k0) {
                const int j = b0 + bits_below(M0);
                LSegIdx q;
                q.a = g.a; q.c = (uint16_t)~(uint32_t)k0; q.b = g.c; q.pad = 0;
                L.seg[c ^ 1][j] = q;
                L.map[2 * s] = (uint16_t)j;
            }
            if (k1) {
                const int j = b0 + (int)__popcll(M0) + bits_below(M1);
                LSegIdx q;
                q.a = g.c; q.c = (uint16_t)~(uint32_t)k1; q.b = g.b; q.pad = 0;
                L.seg[c ^ 1][j] = q;
                L.map[2 * s + 1] = (uint16_t)j;
            }
        }
        if (t == 0) L.live[c] = 0;  // (read at the top of this pass; filled by the next)
        nodes += S;
        lds_barrier();
    }
    if (st && t == 0) {
        const int np = WHOLE ? (pass > 2 ? pass - 2 : 0) : pass - 1;
        st->passes = np > st->passes ? np : st->passes;
    }
    // ---- ring order: the nodes packed into a list, then each one's distance
    // to the last node by pointer jumping (a wave alone needs no barriers)
    const int end = ib;  // (the last node points here: A of a ring, B of a chain)
    if (t == 0) L.live[0] = 0;
    lds_barrier();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int i = t + T * r;
        const int nx = (i < cnt && (WHOLE || i != ib)) ? (int)L.next[i] : (int)kNoNext;
        const uint64_t M = __ballot(nx != kNoNext);
        if (!M) continue;
        int at = 0;
        if (lane == 0) at = atomicAdd(&L.live[0], (int)__popcll(M));
        at = __builtin_amdgcn_readfirstlane(at);
        if (nx != kNoNext) {
            L.list[0][at + bits_below(M)] = (uint16_t)i;
            L.jn[0][i] = (uint16_t)(nx == end ? i : nx);
            L.jd[0][i] = (uint16_t)(nx == end ? 0 : 1);
        }
    }
    lds_barrier();
    if (nodes <= 64) {
        if (t < 64) {
            const bool on = lane < nodes;
            const int i = L.list[0][on ? lane : 0];
            int n = L.jn[0][i], d = L.jd[0][i];
            for (int span = 1; span < nodes - 1; span <<= 1) {
                const int d2 = L.jd[0][n], n2 = L.jn[0][n];
                d += d2;
                n = n2;
                wave_sync();
                if (on) {
                    L.jd[0][i] = (uint16_t)d;
                    L.jn[0][i] = (uint16_t)n;
                }
                wave_sync();
            }
            if (on) L.ring[nodes - 1 - d] = (uint16_t)i;
        }
        lds_barrier();
        return nodes;
    }
    int node[R], f = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) node[r] = L.list[0][min(t + T * r, nodes - 1)];
    const bool mine = (t & ~63) < nodes;  // (a wave without a node skips the rounds)
    for (int span = 1; span < nodes - 1; span <<= 1) {
        if (mine) {
            int n1[R], d1[R], n2[R], d2[R];
#pragma unroll
            for (int r = 0; r < R; ++r) { n1[r] = L.jn[f][node[r]]; d1[r] = L.jd[f][node[r]]; }
#pragma unroll
            for (int r = 0; r < R; ++r) { n2[r] = L.jn[f][n1[r]]; d2[r] = L.jd[f][n1[r]]; }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                // (threads past the last node repeat it: the same values)
                L.jn[f ^ 1][node[r]] = (uint16_t)n2[r];
                L.jd[f ^ 1][node[r]] = (uint16_t)(d1[r] + d2[r]);
            }
        }
        f ^= 1;
        lds_barrier();
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (t + T * r < nodes) L.ring[nodes - 1 - L.jd[f][node[r]]] = (uint16_t)node[r];
    lds_barrier();
    return nodes;
}

}  // namespace sqh
