// Resumable closest-hit walks, shared by the kernels that keep one per lane:
// the bounce loop and the specular refinement.
#pragma once

#include "common.h"

namespace pcrt {

// Resumable closest-hit walk of one lane: nearest hit among the disks != excl
// with t in (t_lo, inf), near child first, with the tie rule: t* = min t; among
// hits with t <= t* + eps_tie the smallest (d2, id) wins. Hits within the
// current window are kept in a short list that is pruned whenever t* shrinks;
// if the list overflows, a second, exact pass over the final window decides.
// The state is kept across the iterations of the loop that steps the walk;
// park holds a leaf reached but not yet tested.
struct Walk {
    f3 inv, oi;
    int ref, sp, park;
    float tmin;         // nearest hit so far; in the second pass the end of its window
    bool spill, pass2;  // candidate list overflowed; second (exact) pass running
};

// The walks' tie lists, in LDS: entry q of a lane is (t, d2, id) in rows
// 3q .. 3q + 2 of its column; id < 0 is a free entry. In the second pass entry
// 0 is the best hit of the window so far. A walk touches its list only where a
// disk is hit, and the registers this leaves free are worth more to the
// node steps and to the code between the walks.
// Three entries: no bounce of the office overflows them (as with four); one
// entry sends 1 % of its bounces to the second pass.
constexpr int kTieList = 3;
constexpr int kTieRows = 3 * kTieList;
struct Ties {
    float *col;  // this lane's column: row r at col[r * kWave]
    __device__ __forceinline__ float &t(int q) const { return col[(3 * q) * kWave]; }
    __device__ __forceinline__ float &d2(int q) const { return col[(3 * q + 1) * kWave]; }
    __device__ __forceinline__ int id(int q) const { return __float_as_int(col[(3 * q + 2) * kWave]); }
    __device__ __forceinline__ void set_id(int q, int v) const { col[(3 * q + 2) * kWave] = __int_as_float(v); }
};

__device__ __forceinline__ void walk_start(Walk &w, const Ties &c, int root, f3 o, f3 d) {
    w.inv = safe_inv(d);
    w.oi = times(o, w.inv);
    w.ref = root;
    w.sp = 0;
    w.park = kNoRef;
    w.tmin = INFINITY;
#pragma unroll
    for (int q = 0; q < kTieList; ++q) c.set_id(q, -1);
    w.spill = w.pass2 = false;
}

// The disks of the parked leaf against the walk.
__device__ __forceinline__ void walk_leaf(const DevScene &S, Walk &w, const Ties &c, f3 o, f3 d, int excl, float t_lo,
                                          float eps_tie, Stack &stk) {
    const int v = -1 - w.park;
    const int first = v >> 3, cnt = (v & 7) + 1;
    stk.test(cnt);
    for (int i = 0; i < cnt; ++i) {
        const float4 dp = ld4(S.disk, (uint32_t)(first + i) * 32u);
        const float4 dn = ld4(S.disk, (uint32_t)(first + i) * 32u + 16u);
        const int id = __float_as_int(dp.w);
        float t, d2;
        if (!(disk_hit(o, d, xyz(dp), xyz(dn), S.r2, t, d2) & (id != excl) & (t > t_lo))) continue;
        if (w.pass2) {
            if (t <= w.tmin && (d2 < c.d2(0) || (d2 == c.d2(0) && id < c.id(0)))) {
                c.t(0) = t;
                c.d2(0) = d2;
                c.set_id(0, id);
            }
            continue;
        }
        if (t > w.tmin + eps_tie) continue;
        if (t < w.tmin) {
            w.tmin = t;
            const float lim = t + eps_tie;
#pragma unroll
            for (int q = 0; q < kTieList; ++q)
                if (c.id(q) >= 0 && c.t(q) > lim) c.set_id(q, -1);
        }
        bool placed = false;
#pragma unroll
        for (int q = 0; q < kTieList; ++q)
            if (!placed && c.id(q) < 0) {
                c.t(q) = t;
                c.d2(q) = d2;
                c.set_id(q, id);
                placed = true;
            }
        if (!placed) w.spill = true;
    }
    w.park = kNoRef;
}

// One node of the walk: true if a child was entered (ref is then that child,
// the other entered children are on the stack).
template <int W>
__device__ __forceinline__ bool node_step(const DevScene &S, Walk &w, float t_lo, float tc, Stack &stk) {
    if constexpr (W > 2) {
        return wide_step<W>(S, w.ref, w.sp, w.inv, w.oi, t_lo, tc, stk);
    } else {
        const uint32_t nb = (uint32_t)w.ref * 64u;
        const float4 a = ld4(S.node, nb), b = ld4(S.node, nb + 16u), e = ld4(S.node, nb + 32u), r = ld4(S.node, nb + 48u);
        float n0, n1;
        const bool h0 = box_hit(a.x, a.y, a.z, a.w, b.x, b.y, w.inv, w.oi, t_lo, tc, n0);
        const bool h1 = box_hit(b.z, b.w, e.x, e.y, e.z, e.w, w.inv, w.oi, t_lo, tc, n1);
        const int r0 = __float_as_int(r.x), r1 = __float_as_int(r.y);
        if (h0 && h1) {
            const bool f0 = n0 <= n1;
            stk.put(w.sp++, f0 ? r1 : r0);
            w.ref = f0 ? r0 : r1;
            return true;
        }
        if (h0 | h1) {
            w.ref = h0 ? r0 : r1;
            return true;
        }
        return false;
    }
}


// Steps the walking lanes of a wavefront: node steps run until half of the
// walking lanes hold a leaf (parked), then the parked leaves are tested
// together. Returns once at most n_busy >> shift lanes still walk; a lane
// whose walk has ended is no longer walking (walking = false).
template <int W>
__device__ __forceinline__ void walk_round(const DevScene &S, Walk &w, const Ties &c, bool &walking, uint32_t n_busy,
                                           int shift, f3 o, f3 d, int excl, float eps_self, float eps_tie, Stack &stk) {
    for (;;) {
        for (;;) {
            if (walking && w.ref < 0 && w.ref != kNoRef && w.park == kNoRef) {
                w.park = w.ref;
                w.ref = w.sp > 0 ? stk.get(--w.sp) : kNoRef;
            }
            const uint32_t n_walk = (uint32_t)__popcll(__ballot(walking));
            const uint32_t n_park = (uint32_t)__popcll(__ballot(walking && w.park != kNoRef));
            if (!__ballot(walking && w.ref >= 0) || 2 * n_park >= n_walk) break;
            if (walking && w.ref >= 0) {
                stk.visit();
                const float tc = w.pass2 ? w.tmin : w.tmin + eps_tie;
                if (!node_step<W>(S, w, eps_self, tc, stk)) w.ref = w.sp > 0 ? stk.get(--w.sp) : kNoRef;
            }
        }
        if (walking && w.park != kNoRef) walk_leaf(S, w, c, o, d, excl, eps_self, eps_tie, stk);
        if (walking && w.ref == kNoRef) walking = false;
        const uint32_t n_walk = (uint32_t)__popcll(__ballot(walking));
        if (n_walk == 0 || (n_walk << shift) <= n_busy) break;
    }
}

// An ended walk whose candidate list overflowed: starts the second, exact
// pass over the final tie window; false if the walk's answer stands.
__device__ __forceinline__ bool walk_second_pass(Walk &w, const Ties &c, int root, float eps_tie) {
    if (!(w.spill && !w.pass2 && w.tmin < INFINITY)) return false;
    w.pass2 = true;
    w.tmin += eps_tie;
    c.t(0) = c.d2(0) = INFINITY;
    c.set_id(0, 0x7fffffff);
    w.ref = root;
    w.sp = 0;
    w.park = kNoRef;
    return true;
}

// The disk an ended walk found (-1: none) and its distance.
__device__ __forceinline__ int walk_hit(const Walk &w, const Ties &c, float &t) {
    t = INFINITY;
    if (!(w.tmin < INFINITY)) return -1;
    float bd2 = INFINITY;
    int bid = 0x7fffffff;
#pragma unroll
    for (int q = 0; q < kTieList; ++q) {
        const int id = c.id(q);
        const float d2 = c.d2(q);
        if ((q == 0 || !w.pass2) && id >= 0 && (d2 < bd2 || (d2 == bd2 && id < bid))) {
            bd2 = d2;
            bid = id;
            t = c.t(q);
        }
    }
    return bid;
}

}  // namespace pcrt
