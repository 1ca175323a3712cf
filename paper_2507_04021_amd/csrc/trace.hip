// Ray launch and the constant-count bounce loop (Sec. II-B): every ray keeps
// bouncing specularly for up to K interactions; each interaction is recorded,
// its specular prefix key (surface-label sequence, Sec. II-B.4) is inserted
// into a per-transmitter hash set, and -- for diffuse scattering -- the
// Fresnel-weighted coefficient of the chain up to this point is stored.
//
// Persistent grid of one-wave blocks; each wave reserves wave_rays
// consecutive ray slots per atomic fetch and hands them to its idle lanes.
#include "common.h"
#include "internal.h"
#include "walk.h"

namespace pcrt {

__device__ __forceinline__ uint32_t key_insert(const HashBufs &hb, uint32_t base, uint64_t enc, uint32_t j,
                                               uint64_t *status) {
    const uint32_t mask = hb.cap - 1;
    uint32_t slot = (uint32_t)mix64(enc) & mask;
    for (uint32_t probe = 0; probe < hb.cap; ++probe) {
        unsigned long long *kp = hb.key + base + slot;
        uint32_t *rp = hb.rep + base + slot;
        unsigned long long cur = __hip_atomic_load(kp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // (read along with the key: a representative only falls, so one read too early costs an atomic at most)
        const uint32_t rep = __hip_atomic_load(rp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (cur == 0ull) cur = atomicCAS(kp, 0ull, (unsigned long long)enc);
        if (cur == 0ull || cur == enc) {
            if (rep > j) atomicMin(rp, j);
            return slot;
        }
        slot = (slot + 1) & mask;
    }
    atomicOr((unsigned long long *)status, 1ull);
    return 0xffffffffu;
}

// The bounce loop (Sec. II-B) with ballot-compacted ray refill. Every lane
// keeps one ray's state -- its bounce, origin, direction, unfolded length,
// chain coefficients and key -- and the state of its current closest-hit
// walk, which resumes from one iteration to the next. The wavefront steps
// its walking lanes until at most a quarter of its busy lanes are still walking;
// the lanes whose walks ended then finish their bounce together (record the
// interaction, reflect) and start the next bounce's walk, and lanes whose
// rays ended are refilled, compacted in lane order by a ballot, from the ray
// slots the wavefront reserved (wave_rays per atomic fetch). Within the
// walking, a lane that reaches a leaf parks it and keeps taking node steps
// (the next stack entry) until half of the walking lanes hold a leaf; the
// parked leaves are then tested together, so node and leaf steps rarely
// share an iteration. A lane never waits for the wavefront's longest walk.
// Parking only delays when a leaf's disks are tested; the nearest hit and its
// tie rule do not depend on the visiting order, so the results are those of
// an unbroken walk (bitwise, tested). Measured on the 1M-point office (4-wide
// tree, leaf 2): 3.11 ms -> 2.46 ms; without parking the refill alone gave
// 3.26 ms (node and leaf steps in the same iterations).
//
// What bounds it: L2 misses of the node and disk loads, so wavefronts in
// flight. With the tie lists in LDS (8 KiB per wavefront with the stack) the
// loop fits five wavefronts per SIMD; with four / five, and refill at half:
// office 2.23 / 2.25 ms, 64 poses in a room (36M rays) 10.4 / 10.1 ms; refill
// at a quarter: 2.27 / 2.29 ms and 10.0 / 9.8 ms, the reception-point launch
// 0.97 -> 0.93 ms. Four wavefronts with the lists in registers and refill at
// half: 2.34, 10.9 and 1.02 ms.
constexpr int kTraceRefillShift = 2;  // refill once at most busy / 4 lanes still walk

template <int W>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(W == 8 ? 3 : 5, 8))) void k_trace(
    LaunchArgs A) {
    __shared__ int lds_stack[kStackLds * kWave];
    __shared__ float tie_list[kTieRows * kWave];
    const int lane = threadIdx.x;
    const uint32_t glane = blockIdx.x * kWave + lane;
    Stack stk{lds_stack + lane, A.S.spill + glane, A.S.spill_lanes};
    const uint32_t T = A.D.T, K = A.D.K;
    const bool want_diff = A.flags & 4, want_spec = A.flags & 2;
    const bool want_geom = A.flags & (4 | 8 | 32);  // points/lengths/cosines: diffuse, tape, averaged planes
    const bool avg = A.flags & 32;                  // weighted-average intersection over point sets
    const float eps_self = A.thr.eps_self, eps_tie = A.thr.eps_tie;
    const uint32_t n_lanes = A.trace_lanes, take = A.wave_rays;
    bool busy = false, walking = false;  // this lane has a ray; its walk has not ended
    uint32_t g = 0, j = 0, k = 0;
    int it = 0, excl = -1;
    f3 o = mk(0.f, 0.f, 0.f), d = mk(0.f, 0.f, 1.f);
    float L = 0.f;
    c32 pte = {1.f, 0.f}, ptm = {1.f, 0.f};
    uint64_t enc = 0;
    const Ties ties{tie_list + lane};
    Walk w;
    walk_start(w, ties, A.S.root, o, d);
    // This wavefront's reserved ray slots [q_next, q_end): the first are dealt (all wavefronts start together, and an
    // atomic on one word costs 11 ns whoever issues it), further ones come from a counter.
    const uint32_t dealt = gridDim.x * take;
    uint32_t q_next = min(blockIdx.x * take, T), q_end = min(q_next + take, T);
    bool q_dry = false;
    uint32_t n_int = 0, n_ray = 0, n_spill = 0;
    for (;;) {
        // refill idle lanes, in lane order, from the reserved slots
        for (;;) {
            const uint64_t idle = __ballot(!busy && (uint32_t)lane < n_lanes);
            if (!idle || q_dry) break;
            if (q_next >= q_end) {
                uint32_t base = T;
                if (lane == 0 && dealt < T) base = dealt + atomicAdd(&A.work[0], take);
                base = __builtin_amdgcn_readfirstlane(base);
                if (base >= T) {
                    q_dry = true;
                    break;
                }
                q_next = base;
                q_end = min(base + take, T);
            }
            const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(idle >> 32),
                                                           __builtin_amdgcn_mbcnt_lo((uint32_t)idle, 0u));
            const uint32_t avail = q_end - q_next;
            if (!busy && (uint32_t)lane < n_lanes && rank < avail) {
                g = q_next + rank;
                it = find_item(A.items, A.D.n_items, g);
                const Item &I = A.items[it];
                const uint32_t local = g - I.ray_off;
                const size_t rb = (size_t)g * K;
                if (local >= I.n_rays) {  // padding slot of the item
                    for (uint32_t kk = 0; kk < K; ++kk) A.rb.id[rb + kk] = -1;
                } else {
                    j = A.subset ? A.subset[local] : local;
                    bool live = true;
                    if (A.flags & 64) {  // towards reception point j (Sec. II-B): FP64 direction, rounded to FP32
                        if (j >= A.S.n_sets) {
                            for (uint32_t kk = 0; kk < K; ++kk) A.rb.id[rb + kk] = -1;
                            n_ray += 1;
                            live = false;
                        } else {
                            d = normalize(aim_dir(I.tx, A.S.dps_recv[j]));
                        }
                    } else {
                        d = normalize(fib_dir(j, I.budget));
                    }
                    if (live) {
                        o = mk(I.tx[0], I.tx[1], I.tx[2]);
                        L = 0.f;
                        excl = -1;
                        pte = ptm = {1.f, 0.f};
                        enc = 0;
                        k = 0;
                        walk_start(w, ties, A.S.root, o, d);
                        busy = walking = true;
                    }
                }
            }
            q_next += min((uint32_t)__popcll(idle), avail);
        }
        const uint32_t n_busy = (uint32_t)__popcll(__ballot(busy));
        if (n_busy == 0) break;  // the slots are used up and every ray has ended
        walk_round<W>(A.S, w, ties, walking, n_busy, kTraceRefillShift, o, d, excl, eps_self, eps_tie, stk);
        if (walking || !busy) continue;
        // this lane's walk ended: the second, exact pass if the tie list overflowed, else the bounce
        if (walk_second_pass(w, ties, A.S.root, eps_tie)) {
            n_spill += 1;
            walking = true;
            continue;
        }
        float t;
        const int h = walk_hit(w, ties, t);
        const size_t rb = (size_t)g * K;
        if (h < 0) {  // the ray leaves the scene
            for (uint32_t kk = k; kk < K; ++kk) A.rb.id[rb + kk] = -1;
            n_int += k;
            n_ray += 1;
            busy = false;
            continue;
        }
        const float4 pn = A.S.nrm[h];
        f3 n = xyz(pn);
        if (avg) {  // the point set's weighted average replaces the disk's point and normal
            dps_average(A.S, o, d, excl, eps_self, A.thr.lambda_d, h, t, n);
            A.rb.nk[rb + k] = make_float4(n.x, n.y, n.z, 0.f);
        }
        const float dn = dot(d, n);
        const float sgn = dn > 0.f ? -1.f : 1.f;
        const float cosi = fabsf(dn);
        const f3 q = fma3(t, d, o);
        L += t;
        A.rb.id[rb + k] = h;
        if (want_geom) {
            A.rb.xl[rb + k] = make_float4(q.x, q.y, q.z, L);
            A.rb.cs[rb + k] = sgn * cosi;
        }
        if (want_diff) {
            uint32_t lab = __float_as_uint(pn.w);
            if (lab >= A.n_labels) {
                atomicOr((unsigned long long *)&A.counters[6], 2ull);
                lab = 0;
            }
            const float er = A.mats[3 * lab], sg = A.mats[3 * lab + 1], sc = A.mats[3 * lab + 2];
            c32 te, tm;
            fresnel(er, sg * A.fc.inv_we0, cosi, te, tm);
            const c32 cte = cmul(pte, te), ctm = cmul(ptm, tm);
            const float wgt = A.fc.amp_iso * sc;
            A.rb.coef[rb + k] = make_float4(wgt * cte.re, wgt * cte.im, wgt * ctm.re, wgt * ctm.im);
            const float R = sqrtf(fmaxf(0.f, 1.f - sc * sc));
            pte = {R * cte.re, R * cte.im};
            ptm = {R * ctm.re, R * ctm.im};
        }
        if (A.rb.dslot) {  // voxel diffuse key: labels before this interaction, then this point set
            const uint64_t encd = enc * (uint64_t)A.S.n_sets + (uint64_t)A.S.dps_of[h] + 1ull;
            A.rb.dslot[rb + k] = key_insert(A.dhb, 0u, encd, j, A.counters + 6);
        }
        if (want_spec || A.rb.dslot) {
            const uint32_t su = __float_as_uint(A.S.pos[h].w);
            enc = enc * (uint64_t)A.n_surf1 + (uint64_t)(su + 1);
            if (want_spec) A.rb.slot[rb + k] = key_insert(A.hb, (uint32_t)it * A.hb.cap, enc, j, A.counters + 6);
        }
        d = normalize(fma3(-2.f * dn, n, d));
        o = q;
        excl = h;
        k += 1;
        if (k == K) {
            n_int += K;
            n_ray += 1;
            busy = false;
        } else {
            walk_start(w, ties, A.S.root, o, d);
            walking = true;
        }
    }
    flush_visits(stk, A.counters, 9);
    n_int = warp_sum_u(n_int);
    n_ray = warp_sum_u(n_ray);
    n_spill = warp_sum_u(n_spill);
    if (lane == 0) {
        add_to(n_int, &A.counters[0]);
        add_to(n_ray, &A.counters[1]);
        add_to(n_spill, &A.counters[8]);
    }
}

uint32_t compute_units() {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
        (void)hipGetLastError();
        return 256;  // no device to ask
    }
    return (uint32_t)std::max(cus, 1);
}

uint32_t resident_blocks(const void *kernel, int block_threads) {
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, block_threads, 0) != hipSuccess) {
        (void)hipGetLastError();
        return 2048;  // no device to ask: an upper bound for 256 compute units
    }
    return (uint32_t)std::max(per_cu, 1) * compute_units();
}

template <int W>
uint32_t trace_cap() {
    static const uint32_t cap = resident_blocks((const void *)k_trace<W>, kWave);
    return cap;
}

uint32_t trace_cap_w(uint32_t width) {
    return width == 8 ? trace_cap<8>() : width == 4 ? trace_cap<4>() : trace_cap<2>();
}

// Lanes of a wavefront that take rays, where the caller leaves the fetch open. A wavefront of few rays steps faster (a
// node step costs its lanes' separate cache lines, and it waits for its longest
// walk), so a launch too small to give every SIMD a wavefront of 64 rays is
// spread over one wavefront per SIMD, of 4 rays at least. 2 000 rays, K = 2:
// 88 us with 64 lanes, 72 / 67 / 62 / 98 with 16 / 8 / 4 / 1; but 65 537 rays,
// K = 3 (already a wavefront of 64 per SIMD): 0.295 ms, 0.304 / 0.366 with 32 / 16.
static uint32_t trace_lanes(const SolveDims &D) {
    static const uint32_t simds = 4 * compute_units();
    uint32_t lanes = 4;
    while (lanes < (uint32_t)kWave && (D.T + lanes - 1) / lanes > simds) lanes <<= 1;
    return lanes;
}

// Rays per work fetch where the caller leaves it open. A fetch is an atomic on one
// word (11 ns each, whoever issues it): 36M rays in fetches of 64 are 562 000 of them, 6 ms one after another. From 16
// fetches of 256 per wavefront on the last ones no longer matter for the balance. 64 poses, 36M rays: 9.73 ms with 64,
// 9.38 / 9.27 / 9.28 / 9.51 with 128 / 256 / 512 / 1 024; but a million rays: 27.1 / 27.2 / 27.1 / 28.3 / 31.3 ms,
// 65 537 rays: 2.1 / 2.3 / 2.7 / 3.4 / 4.9 ms (whole solves).
static uint32_t default_wave_rays(const SolveDims &D) {
    const uint64_t large = 4 * kWave;
    return D.T >= 16 * large * trace_cap_w(D.width) ? (uint32_t)large : (uint32_t)kWave;
}

// A value that the caller gives is taken at every size, by whole wavefronts.
TraceShape trace_shape(const SolveDims &D, uint32_t wave_rays) {
    if (wave_rays) return {(uint32_t)kWave, wave_rays};
    const uint32_t lanes = trace_lanes(D);
    return {lanes, lanes < (uint32_t)kWave ? lanes : default_wave_rays(D)};
}

uint32_t trace_grid(const SolveDims &D, uint32_t take) {
    const uint32_t units = (D.T + take - 1) / take;
    return std::max<uint32_t>(1, std::min(trace_cap_w(D.width), units));
}

void launch_trace(const LaunchArgs &A, hipStream_t s) {
    const uint32_t grid = trace_grid(A.D, A.wave_rays);
    switch (A.D.width) {
        case 8: hipLaunchKernelGGL(k_trace<8>, dim3(grid), dim3(kWave), 0, s, A); break;
        case 4: hipLaunchKernelGGL(k_trace<4>, dim3(grid), dim3(kWave), 0, s, A); break;
        default: hipLaunchKernelGGL(k_trace<2>, dim3(grid), dim3(kWave), 0, s, A); break;
    }
}

__global__ void k_raygen(uint32_t n_budget, const uint32_t *ids, uint32_t n, float *out) {
    uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    f3 d = fib_dir(ids ? ids[i] : i, n_budget);
    out[3 * i] = d.x;
    out[3 * i + 1] = d.y;
    out[3 * i + 2] = d.z;
}

void launch_raygen(uint32_t n_budget, const uint32_t *ids, uint32_t n, float *out, hipStream_t s) {
    hipLaunchKernelGGL(k_raygen, dim3((n + 255) / 256), dim3(256), 0, s, n_budget, ids, n, out);
}

}  // namespace pcrt
