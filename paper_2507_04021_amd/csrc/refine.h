// The specular refinement kernel (Sec. II-B.2): image-method minimiser,
// validation passes with plane replacements, final occlusion test and the
// path field. A template shared by the translation units that instantiate
// it: specular.hip (the scalar TE/TM field) and specular_pol.hip (the
// polarised field), compiled in parallel.
#pragma once

#include "common.h"
#include "internal.h"
#include "walk.h"

namespace pcrt {

// Image method on k planes (exact minimiser of Eq. (1) restricted to them):
// images I_m of the TX, back-trace from the RX; every segment must cross its
// plane strictly inside, and both neighbours of x_m must lie strictly on the
// same side of plane m, farther than eps_self (a reflection, not a
// transmission).
template <int KM>
__device__ __forceinline__ bool refine_planes(int k, f3 tx, f3 rx, const f3 *pp, const f3 *pn, float eps_self,
                                              f3 *x) {
    f3 img[KM + 1];
    img[0] = tx;
#pragma unroll
    for (int m = 1; m <= KM; ++m)
        if (m <= k) img[m] = img[m - 1] - (2.f * dot(img[m - 1] - pp[m - 1], pn[m - 1])) * pn[m - 1];
    x[0] = tx;
    f3 cur = rx;
#pragma unroll
    for (int m = KM; m >= 1; --m) {
        if (m > k) continue;
        f3 seg = img[m] - cur;
        float den = dot(seg, pn[m - 1]);
        if (den == 0.f) return false;
        float s = dot(pp[m - 1] - cur, pn[m - 1]) / den;
        if (!(s > 0.f && s < 1.f)) return false;
        cur = cur + s * seg;
        x[m] = cur;
    }
#pragma unroll
    for (int m = 1; m <= KM; ++m) {
        if (m > k) continue;
        f3 nb = (m == k) ? rx : x[m + 1];
        float da = dot(x[m - 1] - pp[m - 1], pn[m - 1]);
        float db = dot(nb - pp[m - 1], pn[m - 1]);
        if (!(da * db > 0.f && fabsf(da) > eps_self && fabsf(db) > eps_self)) return false;
    }
    return true;
}

// The same minimiser for the walks: only the points x_from and x_(from+1) are
// kept (from < k), the others stream through the tests, so the lanes' walk
// state stays in registers beside it.
template <int KM>
__device__ __forceinline__ bool refine_segment(int k, f3 tx, f3 rx, const f3 *pp, const f3 *pn, float eps_self,
                                               int from, f3 &a, f3 &b) {
    f3 img[KM + 1];
    img[0] = tx;
#pragma unroll
    for (int m = 1; m <= KM; ++m)
        if (m <= k) img[m] = img[m - 1] - (2.f * dot(img[m - 1] - pp[m - 1], pn[m - 1])) * pn[m - 1];
    f3 cur = rx, nb = rx;  // x_(m+1), x_(m+2), the receiver beyond x_k
    a = tx;
    b = tx;
    bool ok = true;
#pragma unroll
    for (int m = KM; m >= 0; --m) {
        if (m > k) continue;
        f3 xm = tx;
        if (m > 0) {
            f3 seg = img[m] - cur;
            float den = dot(seg, pn[m - 1]);
            float s = dot(pp[m - 1] - cur, pn[m - 1]) / den;
            ok = ok && den != 0.f && s > 0.f && s < 1.f;
            xm = cur + s * seg;
        }
        if (m < KM && m < k) {
            float da = dot(xm - pp[m], pn[m]);
            float db = dot(nb - pp[m], pn[m]);
            ok = ok && da * db > 0.f && fabsf(da) > eps_self && fabsf(db) > eps_self;
        }
        if (m == from) a = xm;
        if (m == from + 1) b = xm;
        nb = cur;
        cur = xm;
    }
    return ok;
}

struct PairOut {
    bool valid;
    float len;
    c32 te, tm;
};

// The representative's interaction planes of a key, rec being the record of its
// last interaction: its first k hit disks' planes, or with point-set averaging
// its first k averaged interactions (point and normal from the records).
template <int KM>
struct KeyPlanes {
    f3 pp[KM], pn[KM];
    int k;
};

template <int KM, bool AVG>
__device__ __forceinline__ void load_planes(const LaunchArgs &A, uint32_t rec, KeyPlanes<KM> &kp) {
    const uint32_t K = A.D.K;
    const uint32_t g = rec / K;
    kp.k = (int)(rec % K) + 1;
#pragma unroll
    for (int m = 0; m < KM; ++m)
        if (m < kp.k) {
            const size_t ri = (size_t)g * K + m;
            if (AVG) {
                kp.pp[m] = xyz(A.rb.xl[ri]);
                kp.pn[m] = xyz(A.rb.nk[ri]);
            } else {
                const int id = A.rb.id[ri];
                kp.pp[m] = xyz(A.S.pos[id]);
                kp.pn[m] = xyz(A.S.nrm[id]);
            }
        }
}

// The same with the planes that replaced some of them: ovr[j * kWave] is the
// disk whose plane replaced plane j, -1 if none (its averaged point and normal
// are then pl[2j], pl[2j + 1]).
template <int KM, bool AVG>
__device__ __forceinline__ void cur_planes(const LaunchArgs &A, uint32_t rec, const int *ovr, const float4 *pl,
                                           KeyPlanes<KM> &kp) {
    load_planes<KM, AVG>(A, rec, kp);
#pragma unroll
    for (int j = 0; j < KM; ++j)
        if (j < kp.k) {
            const int od = ovr[j * kWave];
            if (od >= 0) {
                kp.pp[j] = AVG ? xyz(pl[2 * j]) : xyz(A.S.pos[od]);
                kp.pn[j] = AVG ? xyz(pl[2 * j + 1]) : xyz(A.S.nrm[od]);
            }
        }
}

__device__ __forceinline__ f3 rx_point(const LaunchArgs &A, uint32_t r) {
    return mk(A.rx[3 * r], A.rx[3 * r + 1], A.rx[3 * r + 2]);
}

// The field of a validated path: points x[0] = TX, x[1..k], disks hid on planes
// kp; the last point sees the receiver.
template <int KM, bool POL>
__device__ __forceinline__ void path_field(const LaunchArgs &A, uint32_t q, uint32_t r, f3 rx, const f3 *x,
                                           const int *hid, const KeyPlanes<KM> &kp, PairOut &po) {
    const uint32_t K = A.D.K;
    const int k = kp.k;
    f3 xk = x[1];
#pragma unroll
    for (int m = 1; m <= KM; ++m)
        if (m == k) xk = x[m];
    float L = 0.f;
    c32 pte = {1.f, 0.f}, ptm = {1.f, 0.f};
    float csv[KM];
    constexpr bool pol = POL;
    cv3 ev = {};
    if (pol) ev = pol_launch(A.pol_tx, normalize(x[1] - x[0]));
#pragma unroll
    for (int m = 1; m <= KM; ++m) {
        if (m > k) continue;
        f3 seg = x[m] - x[m - 1];
        float sl = len(seg);
        L += sl;
        const f3 di = (1.0f / sl) * seg;
        float c = fabsf(dot(di, kp.pn[m - 1]));
        csv[m - 1] = c;
        uint32_t lab = __float_as_uint(A.S.nrm[hid[m - 1]].w);
        if (lab >= A.n_labels) lab = 0;
        float er = A.mats[3 * lab], sg = A.mats[3 * lab + 1], sc = A.mats[3 * lab + 2];
        c32 te, tm;
        fresnel(er, sg * A.fc.inv_we0, c, te, tm);
        float R = sqrtf(fmaxf(0.f, 1.f - sc * sc));
        if (pol) {
            const f3 nxt = m < k ? x[m < KM ? m + 1 : m] : rx;
            pol_reflect(ev, di, normalize(nxt - x[m]), kp.pn[m - 1], te, tm, R);
        } else {
            pte = cmul(pte, {R * te.re, R * te.im});
            ptm = cmul(ptm, {R * tm.re, R * tm.im});
        }
    }
    L += len(rx - xk);
    c32 ph = propagate(L, A.fc.inv_lam_hi, A.fc.inv_lam_lo);
    float a0 = A.fc.amp_iso / L;
    if (pol) pte = ptm = pol_receive(ev, A.pol_rx, normalize(rx - xk));
    po.te = cmul({a0 * pte.re, a0 * pte.im}, ph);
    po.tm = cmul({a0 * ptm.re, a0 * ptm.im}, ph);
    po.len = L;
    po.valid = true;
    if ((A.flags & 8) && q < A.D.rec_keys) {
        size_t p = (size_t)q * A.D.n_rx + r;
#pragma unroll
        for (int m = 0; m < KM; ++m)
            if (m < k) {
                A.sb.hit[p * K + m] = hid[m];
                A.sb.cs[p * K + m] = csv[m];
            }
    }
}

// Persistent single-wavefront blocks. A work unit is (key chunk, slice of up
// to kRefineRxSlice receivers, fewer where units are scarce); units are dealt
// where each wavefront has one, else handed out by an atomic counter (11 ns for each
// who asks), slice-minor so that consecutive units reuse a chunk's key planes.
//
// The wavefront deals a unit's (key, receiver) pairs to its lanes in tiles
// of 64 and solves the image method for each pair (cheap, no traversal);
// pairs with a solution join a queue in LDS, with the direction of their
// first segment. An idle lane takes a queued candidate and validates it: a ray
// from each image point to the next must hit a disk of the expected surface,
// close in angle (t_a) and plane distance (t_d). The first interaction that
// fails those two tests replaces its plane by the hit disk's and starts
// again from the transmitter with the new image points (kappa times at most);
// any other failure ends the candidate. If every interaction holds, the last
// point must see the receiver, and the path's field is evaluated. With
// point-set averaging the validation hit is averaged over its set first
// (Sec. II-C): its point and normal are tested, and become the new plane.
//
// What bounds it: the closest-hit walks (a few short ones per candidate, most
// of them first segments that end in a plane replacement), that is L2
// latency and the lanes that wait for longer walks. So the walks are those of
// the bounce loop: resumable, leaves parked, the wavefront steps them until at
// most an eighth of its busy lanes still walk, and the lanes whose walks ended
// then decide together (plane replacement, next segment or end) and walk on
// or take the next candidate. A lane keeps its candidate until it ends; what
// it needs besides the walk (key planes, replaced planes, image points) is
// loaded and computed again at each decision, which costs less than keeping
// it in registers through the walks.
//
// Sums: a path's amplitudes go to this block's result slots, indexed by the
// open unit and the pair within it, with a bit in LDS. When a unit is done,
// lane r adds the paths of receiver r in increasing key order and writes the
// unit's partial sum of receiver r0 + r for chunk c. The result does not
// depend on timing or on the order in which candidates ended. Up to two units
// are open at once: while the last candidates of one end, the tiles of the
// next feed the idle lanes.
//
// Measured on the 1M-point office (2^20 rays, K = 5, 64 receivers; one pass at
// a time for a whole batch before): 4.19 -> 3.06 ms; on its polarised solve
// (2^18 rays) 3.32 -> 2.15, with averaging 1.74 -> 1.32. Lanes decide once at
// most 1/2, 1/4 or 1/8 of the busy ones still walk: 3.30, 3.06, 3.05 ms (1.54,
// 1.37, 1.32 with averaging): a decision is a chain of dependent loads, worth
// waiting for company. When nothing is left to feed idle lanes, all busy lanes
// are waited for (a solve of 35 candidates 80 -> 66 us).
constexpr int kRefineOpen = 2;          // units open at once per wavefront
constexpr int kRefineRefillShift = 3;   // lanes decide once at most busy / 8 still walk

struct RefUnit {  // an open unit (wavefront-uniform)
    uint32_t c, part, r0, nr, q0, ne, t, pending;  // pending: candidates queued or held by a lane
    f3 tx;
    bool open;
};

// Global-memory writes of some lanes of a single-wavefront block are visible
// to its other lanes after this.
__device__ __forceinline__ void block_sync_global() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// POL: the polarised field (its own instances, so that the scalar ones keep
// their register allocation). Three wavefronts per SIMD up to K = 5 (168
// registers: up to 42 spilled up to K = 4, 111 to 141 at K = 5): at K = 5, two (none spilled) take 0.4 ms
// more of the office's 27.1, 0.1 of its polarised solve's 3.15, 0.06 of the averaged one's 2.53, though less where most
// candidates are paths (empty room, 3 000 receivers 2.23 -> 2.10); four took 3.2 ms of the office (247 spilled) where
// three took 3.06.
template <int KM, int W, bool AVG, bool POL>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(KM <= 5 ? 3 : 2, 8))) void k_refine(
    LaunchArgs A) {
    constexpr uint32_t kUnitPairs = kKeyChunk * kRefineRxSlice;
    static_assert(kRefineOpen == 2 && kRefineOpen * kUnitPairs == kRefineResPerBlock, "two open units");
    static_assert(kRefineOpen * kUnitPairs <= 0x10000, "a queue entry names its pair in 16 bits");
    __shared__ int lds_stack[kStackLds * kWave];
    __shared__ uint16_t queue[kRefineQueue];       // open-unit slot x kUnitPairs + pair
    __shared__ uint32_t queue_rec[kRefineQueue];   // record of its key's last interaction
    __shared__ float queue_u[3][kRefineQueue];     // direction of the candidate's first segment
    __shared__ int ovr[KM][kWave];                 // per lane and interaction: the disk whose plane replaced the key's
    __shared__ float tie_list[kTieRows * kWave];
    __shared__ uint32_t vbits[kRefineOpen][kUnitPairs / 32];  // pairs of an open unit that are paths
    const int lane = threadIdx.x;
    const uint32_t glane = blockIdx.x * kWave + lane;
    Stack stk{lds_stack + lane, A.S.spill + glane, A.S.spill_lanes};
    float4 *res = A.spec_res + (size_t)blockIdx.x * kRefineOpen * kUnitPairs;
    // the validated disks of this lane's candidate, interaction m at hid_g[m * kWave]
    int *hid_g = A.spec_hid + (size_t)blockIdx.x * kWave * KM + lane;
    // point-set averaging: the replaced planes of this lane's candidate, (point, normal) per interaction
    float4 *pl_g = AVG ? A.spec_ovr + (size_t)glane * KM * 2 : nullptr;
    const uint32_t n_rx = A.D.n_rx, n_items = A.D.n_items;
    const uint32_t n_chunks = A.chunk_off[n_items];
    const RefineShape shape = planned_refine(A);
    const uint32_t slice = shape.slice, parts = shape.parts, part_keys = kKeyChunk / parts;
    const uint32_t n_slices = (n_rx + slice - 1) / slice;
    const uint32_t n_units = n_chunks * n_slices * parts;
    if (blockIdx.x >= n_units) return;  // (3 072 wavefronts asking the counter for 36 units: 104 us, 29 so)
    const bool one_open = parts > 1;  // parts are few pairs: a second would only take them from another wavefront
    const bool rec = A.flags & 8;
    const float eps_self = A.thr.eps_self, eps_tie = A.thr.eps_tie;
    uint32_t n_cand = 0, n_valid = 0;
    RefUnit U[kRefineOpen];
#pragma unroll
    for (int k = 0; k < kRefineOpen; ++k) U[k] = RefUnit{0, 0, 0, 0, 0, 0, 0, 0, mk(0.f, 0.f, 0.f), false};
    bool exhausted = false;       // the unit counter has run out
    uint32_t head = 0, tail = 0;  // queue ring positions (wavefront-uniform)
    // this lane's candidate: entry of the queue, passes that ended in a plane
    // replacement, segment being walked (from image point seg - 1 to seg)
    bool busy = false, walking = false;
    uint32_t ent = 0, krec = 0;
    int retries = 0, seg = 1, excl = -1;
    f3 o = mk(0.f, 0.f, 0.f), d = mk(0.f, 0.f, 1.f);
    const Ties ties{tie_list + lane};
    Walk w;
    walk_start(w, ties, A.S.root, o, d);
    w.ref = kNoRef;
    for (;;) {
        // lanes whose walks ended: second pass, plane replacement, next segment or end
        bool ended = false;
        if (busy && !walking) {
            if (walk_second_pass(w, ties, A.S.root, eps_tie)) {
                walking = true;
            } else {
                const bool s1 = ent >= kUnitPairs;
                const uint32_t e = ent % kUnitPairs;
                const uint32_t nr = s1 ? U[1].nr : U[0].nr;
                const uint32_t q = (s1 ? U[1].q0 : U[0].q0) + e / nr;
                const uint32_t r = (s1 ? U[1].r0 : U[0].r0) + e % nr;
                // the plane and label of the interaction just walked to
                const int od = ovr[seg - 1][lane];
                const size_t ri = (size_t)(krec / A.D.K) * A.D.K + seg - 1;
                const int id0 = A.rb.id[ri];
                const int idp = od >= 0 ? od : id0;
                f3 pp, pn;
                if (AVG) {
                    pp = od >= 0 ? xyz(pl_g[2 * (seg - 1)]) : xyz(A.rb.xl[ri]);
                    pn = od >= 0 ? xyz(pl_g[2 * (seg - 1) + 1]) : xyz(A.rb.nk[ri]);
                } else {
                    pp = xyz(A.S.pos[idp]);
                    pn = xyz(A.S.nrm[idp]);
                }
                float t;
                const int h = walk_hit(w, ties, t);
                const float4 hp = A.S.pos[h < 0 ? 0 : h];
                // (a replaced plane's disk lies on the same surface)
                bool good = h >= 0 && __float_as_uint(hp.w) == __float_as_uint(A.S.pos[id0].w), again = false;
                if (good) {
                    f3 hn = xyz(A.S.nrm[h]);
                    if (AVG) dps_average(A.S, o, d, excl, eps_self, A.thr.lambda_d, h, t, hn);
                    const f3 qh = o + t * d;
                    const bool ang_ok = fabsf(dot(hn, pn)) >= A.thr.cos_ta;
                    const bool dist_ok = fabsf(dot(qh - pp, pn)) <= A.thr.t_d;
                    if (!(ang_ok && dist_ok)) {  // start again on the hit disk's plane
                        again = retries < A.thr.kappa;
                        good = again;
                        retries += 1;
                        if (again) {
                            ovr[seg - 1][lane] = h;
                            if (AVG) {
                                pl_g[2 * (seg - 1)] = make_float4(qh.x, qh.y, qh.z, 0.f);
                                pl_g[2 * (seg - 1) + 1] = make_float4(hn.x, hn.y, hn.z, 0.f);
                            }
                        }
                    }
                }
                PairOut po;
                po.valid = false;
                ended = true;
                if (good) {
                    if (!again) hid_g[(seg - 1) * kWave] = h;
                    excl = again ? -1 : h;
                    const int from = again ? 0 : seg;  // the next segment starts at image point from
                    KeyPlanes<KM> kp;
                    cur_planes<KM, AVG>(A, krec, &ovr[0][lane], pl_g, kp);
                    if (from < kp.k) {
                        f3 a, b;
                        if (refine_segment<KM>(kp.k, s1 ? U[1].tx : U[0].tx, rx_point(A, r), kp.pp, kp.pn, eps_self,
                                               from, a, b)) {
                            seg = from + 1;
                            o = a;
                            d = normalize(b - a);
                            walk_start(w, ties, A.S.root, o, d);
                            walking = true;
                            ended = false;
                        }
                    } else {  // every interaction holds: the last point must see the receiver
                        const f3 rx = rx_point(A, r);
                        f3 a, xk;
                        (void)refine_segment<KM>(kp.k, s1 ? U[1].tx : U[0].tx, rx, kp.pp, kp.pn, eps_self, kp.k - 1, a,
                                                 xk);
                        if (!occluded<W>(A.S, xk, rx, h, eps_self, stk)) {
                            __asm__ volatile("" ::: "memory");  // planes are loaded again, not kept through the walk
                            cur_planes<KM, AVG>(A, krec, &ovr[0][lane], pl_g, kp);
                            f3 x[KM + 1];
                            (void)refine_planes<KM>(kp.k, s1 ? U[1].tx : U[0].tx, rx, kp.pp, kp.pn, eps_self, x);
                            int hid[KM];
#pragma unroll
                            for (int m = 0; m < KM; ++m) hid[m] = m < kp.k ? hid_g[m * kWave] : 0;
                            path_field<KM, POL>(A, q, r, rx, x, hid, kp, po);
                        }
                    }
                }
                if (ended) {
                    if (rec && q < A.D.rec_keys) {
                        const size_t p = (size_t)q * n_rx + r;
                        A.sb.valid[p] = po.valid;
                        A.sb.len[p] = po.valid ? po.len : 0.f;
                        A.sb.amp[p] = po.valid ? make_float4(po.te.re, po.te.im, po.tm.re, po.tm.im)
                                               : make_float4(0.f, 0.f, 0.f, 0.f);
                    }
                    if (po.valid) {
                        ++n_valid;
                        res[ent] = make_float4(po.te.re, po.te.im, po.tm.re, po.tm.im);
                        atomicOr(&vbits[s1 ? 1 : 0][e >> 5], 1u << (e & 31));
                    }
                    busy = false;
                }
            }
        }
        U[0].pending -= (uint32_t)__popcll(__ballot(ended && ent < kUnitPairs));
        U[1].pending -= (uint32_t)__popcll(__ballot(ended && ent >= kUnitPairs));
        // close the units whose tiles are done and whose candidates have all ended
#pragma unroll
        for (int k = 0; k < kRefineOpen; ++k) {
            if (!(U[k].open && U[k].t * kWave >= U[k].ne && U[k].pending == 0)) continue;
            block_sync_global();  // result slots written by other lanes are visible
            if (parts > 1) {  // the paths and their bits; k_combine adds the chunk's
                const uint32_t v = U[k].c * n_rx + U[k].r0, j0 = U[k].part * part_keys, e = lane;
                if (e < U[k].ne && ((vbits[k][e >> 5] >> (e & 31)) & 1u))
                    A.spec_split[(size_t)v * kKeyChunk + j0 + e] = res[k * kUnitPairs + e];
                if (e < part_keys / 8)
                    A.spec_bits[(size_t)v * (kKeyChunk / 8) + j0 / 8 + e] = (uint8_t)(vbits[k][e >> 2] >> (8 * (e & 3)));
            } else if ((uint32_t)lane < U[k].nr) {
                double acc[5] = {0, 0, 0, 0, 0};
                for (uint32_t e = (uint32_t)lane; e < U[k].ne; e += U[k].nr)  // increasing key
                    if ((vbits[k][e >> 5] >> (e & 31)) & 1u) {
                        const float4 v = res[k * kUnitPairs + e];
                        const double tr = v.x, ti = v.y, mr = v.z, mi = v.w;
                        acc[0] += 0.5 * (tr * tr + ti * ti + mr * mr + mi * mi);
                        acc[1] += tr;
                        acc[2] += ti;
                        acc[3] += mr;
                        acc[4] += mi;
                    }
                double *out = A.spec_part + ((size_t)U[k].c * n_rx + U[k].r0 + lane) * 5;
                for (int a = 0; a < 5; ++a) out[a] = acc[a];
            }
            block_sync_global();  // sums read before the slot is reused
            U[k].open = false;
        }
        // feed the idle lanes: image-test tiles of an open unit, else of a newly opened one
        const uint64_t idle = __ballot(!busy);
        const uint32_t n_idle = (uint32_t)__popcll(idle);
        while (tail - head < n_idle) {
            int s = -1;
#pragma unroll
            for (int k = 0; k < kRefineOpen; ++k)
                if (s < 0 && U[k].open && U[k].t * kWave < U[k].ne) s = k;
            if (s < 0 && !exhausted) {
#pragma unroll
                for (int k = 0; k < kRefineOpen; ++k) {
                    if (s >= 0 || U[k].open || exhausted || (k && one_open)) continue;
                    uint32_t u = blockIdx.x;
                    if (n_units <= gridDim.x) {  // dealt
                        exhausted = true;
                    } else {
                        if (lane == 0) u = atomicAdd(&A.work[1], 1u);
                        u = __builtin_amdgcn_readfirstlane(u);
                        if (u >= n_units) {
                            exhausted = true;
                            continue;
                        }
                    }
                    const uint32_t part = u % parts, cs = u / parts, c = cs / n_slices;
                    int lo = 0, hi = (int)n_items - 1;  // item of this chunk
                    while (lo < hi) {
                        int mid = (lo + hi + 1) >> 1;
                        if (A.chunk_off[mid] <= c) lo = mid;
                        else hi = mid - 1;
                    }
                    const Item I = A.items[lo];
                    U[k].c = c;
                    U[k].part = part;
                    U[k].r0 = (cs % n_slices) * slice;
                    U[k].nr = min(slice, n_rx - U[k].r0);
                    U[k].q0 = A.key_off[lo] + (c - A.chunk_off[lo]) * kKeyChunk + part * part_keys;
                    const uint32_t q1 = max(U[k].q0, min(U[k].q0 + part_keys, A.key_off[lo + 1]));
                    U[k].ne = (q1 - U[k].q0) * U[k].nr;
                    U[k].t = 0;
                    U[k].pending = 0;
                    U[k].tx = mk(I.tx[0], I.tx[1], I.tx[2]);
                    U[k].open = true;
                    if ((uint32_t)lane < kUnitPairs / 32) vbits[k][lane] = 0u;
                    wave_sync();
                    s = k;
                }
            }
            if (s < 0) break;
            const bool t1 = s == 1;
            const uint32_t t0 = t1 ? U[1].t : U[0].t, ne = t1 ? U[1].ne : U[0].ne, nr = t1 ? U[1].nr : U[0].nr;
            const uint32_t e = t0 * kWave + lane;
            bool cand = false;
            uint32_t qrec = 0;
            f3 u = mk(0.f, 0.f, 1.f);
            if (e < ne) {
                const uint32_t q = (t1 ? U[1].q0 : U[0].q0) + e / nr, r = (t1 ? U[1].r0 : U[0].r0) + e % nr;
                KeyPlanes<KM> kp;
                qrec = A.keylist[q];
                load_planes<KM, AVG>(A, qrec, kp);
                f3 a, b;
                cand = refine_segment<KM>(kp.k, t1 ? U[1].tx : U[0].tx, rx_point(A, r), kp.pp, kp.pn, eps_self, 0, a, b);
                // launch at the reception points: only where the receiver sees the reception
                // point of the set the representative ray ends in (the visibility matrix)
                if (cand && A.dps_vis)
                    cand = A.dps_vis[(size_t)r * A.S.n_sets + A.S.dps_of[A.rb.id[qrec]]] != 0;
                if (cand) u = normalize(b - a);
                if (rec) {
                    if (q >= A.D.rec_keys) {
                        atomicOr((unsigned long long *)&A.counters[6], 4ull);  // tape capacity exceeded
                    } else if (!cand) {
                        const size_t p = (size_t)q * n_rx + r;
                        A.sb.valid[p] = 0;
                        A.sb.len[p] = 0.f;
                        A.sb.amp[p] = make_float4(0.f, 0.f, 0.f, 0.f);
                    }
                }
            }
            n_cand += cand;
            const uint64_t m = __ballot(cand);
            if (cand) {
                const uint32_t at = (tail + mbcnt(m)) % kRefineQueue;
                queue[at] = (uint16_t)(s * kUnitPairs + e);
                queue_rec[at] = qrec;
                queue_u[0][at] = u.x;
                queue_u[1][at] = u.y;
                queue_u[2][at] = u.z;
            }
            const uint32_t n_new = (uint32_t)__popcll(m);
            tail += n_new;
            U[0].pending += t1 ? 0u : n_new;
            U[1].pending += t1 ? n_new : 0u;
            U[0].t += t1 ? 0u : 1u;
            U[1].t += t1 ? 1u : 0u;
            wave_sync();
        }
        const uint32_t avail = min(tail - head, n_idle);
        if (!busy && mbcnt(idle) < avail) {
            const uint32_t at = (head + mbcnt(idle)) % kRefineQueue;
            ent = queue[at];
            krec = queue_rec[at];
            retries = 0;
            seg = 1;
            excl = -1;
#pragma unroll
            for (int j = 0; j < KM; ++j) ovr[j][lane] = -1;
            o = ent >= kUnitPairs ? U[1].tx : U[0].tx;
            d = mk(queue_u[0][at], queue_u[1][at], queue_u[2][at]);
            walk_start(w, ties, A.S.root, o, d);
            busy = walking = true;
        }
        head += avail;
        wave_sync();  // taken entries are read before their ring slots are reused
        const uint32_t n_busy = (uint32_t)__popcll(__ballot(busy));
        // nothing is left that could feed an idle lane
        const bool dry = (exhausted || one_open) && tail == head && !(U[0].open && U[0].t * kWave < U[0].ne) &&
                         !(U[1].open && U[1].t * kWave < U[1].ne);
        if (n_busy == 0) {
            if (!U[0].open && !U[1].open) break;  // no unit left to open, every unit closed
            continue;
        }
        walk_round<W>(A.S, w, ties, walking, n_busy, dry ? 6 : kRefineRefillShift, o, d, excl, eps_self, eps_tie, stk);
    }
    flush_visits(stk, A.counters, 11);
    n_cand = warp_sum_u(n_cand);
    n_valid = warp_sum_u(n_valid);
    if (lane == 0) {
        add_to(n_cand, &A.counters[7]);
        add_to(n_valid, &A.counters[4]);
    }
}


template <int W, bool AVG, bool POL>
void launch_refine_wa(const LaunchArgs &A, dim3 grid, hipStream_t s) {
    switch (A.D.K) {
        case 1: hipLaunchKernelGGL((k_refine<1, W, AVG, POL>), grid, dim3(kWave), 0, s, A); break;
        case 2: hipLaunchKernelGGL((k_refine<2, W, AVG, POL>), grid, dim3(kWave), 0, s, A); break;
        case 3: hipLaunchKernelGGL((k_refine<3, W, AVG, POL>), grid, dim3(kWave), 0, s, A); break;
        case 4: hipLaunchKernelGGL((k_refine<4, W, AVG, POL>), grid, dim3(kWave), 0, s, A); break;
        case 5: hipLaunchKernelGGL((k_refine<5, W, AVG, POL>), grid, dim3(kWave), 0, s, A); break;
        case 6: hipLaunchKernelGGL((k_refine<6, W, AVG, POL>), grid, dim3(kWave), 0, s, A); break;
        case 7: hipLaunchKernelGGL((k_refine<7, W, AVG, POL>), grid, dim3(kWave), 0, s, A); break;
        default: hipLaunchKernelGGL((k_refine<8, W, AVG, POL>), grid, dim3(kWave), 0, s, A); break;
    }
}

}  // namespace pcrt
