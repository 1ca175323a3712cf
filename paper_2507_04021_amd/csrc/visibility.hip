// Visibility matrix (Sec. II-A, II-B): whether each receiver sees each point
// set's reception point. Receiver r sees reception point j when the open
// segment between them meets no disk outside set j farther than eps_self
// from both ends (the set's own disks surround its reception point).
//
// Mapping, as for the diffuse connections: a wavefront takes a chunk of
// kVisChunk consecutive sets (voxel-key order, so neighbouring voxels)
// against one receiver, and every lane walks from the receiver, so walks
// started together share their start and their path through the upper tree.
// Walks are resumable with ballot-compacted refill, as in the diffuse
// connections: the wavefront steps its walking lanes until at most a quarter
// of its busy lanes still walk, then hands the idle lanes the next sets in
// lane order, from the next unit when one is handed out (every lane has its
// own receiver, so a wavefront is never drained between units). Each output
// byte is written by the lane that decided it, so the result does not depend
// on the schedule. Persistent single-wavefront blocks; the blocks of XCD x
// take the x-th eighth of the (set chunk, receiver) units, receiver-minor, so
// one XCD's L2 serves one region of the scene, each unit from a counter per
// group, a quarter of an XCD's blocks (`taken`): walks of one unit take several times as long as another's,
// and dealt in advance, with a drain at the end of each of its one or two units,
// the slowest wavefront set the time. On the office's 64 x 181 523 matrix: 2.65 ms
// with one 64-set batch per unit and no refill, 2.2 ms with refill over
// 1024-set units dealt in advance, 1.63 ms so, 1.52 with 20 stack entries in LDS.
// An atomic on one line costs 11 ns, so short walks wait for their counter: 10 671 sets x 500 receivers of the
// empty room 119 us with one counter per XCD, 69 with four (68 with eight). Up to two units per wavefront are dealt, with no
// counter and no launch to clear it: 10 sets x 10 000 receivers 36 -> 16 us, one receiver of 10 671 sets 20 -> 15,
// and 500 of 2 502 sets of the office, 1.6 units per wavefront, 209 -> 192.
#include "common.h"
#include "internal.h"

namespace pcrt {

constexpr uint32_t kVisChunk = 128;  // sets per work unit (office, scene build included: 64 / 128 / 256 / 512 / 1024 ->
                                     // 3.67 / 3.68 / 3.72 / 3.80 / 4.03 ms)
constexpr int kVisRefillShift = 2;    // refill once at most busy / 4 lanes still walk

template <int W>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(W == 8 ? 4 : 6, 8))) void k_visibility(
    DevScene S, const float *__restrict__ rx, uint32_t n_rx, const float4 *__restrict__ recv, uint32_t n_sets,
    float eps_self, uint8_t *__restrict__ out, uint32_t share, uint32_t *__restrict__ taken) {
    __shared__ int lds_stack[kStackLdsVisibility * kWave];
    const int lane = threadIdx.x;
    const uint32_t glane = blockIdx.x * kWave + lane;
    StackOf<kStackLdsVisibility> stk{lds_stack + lane, S.spill + glane, S.spill_lanes};
    const uint32_t n_units = (n_sets + kVisChunk - 1) / kVisChunk * n_rx;
    // group g's range is the one of XCD g / (groups per XCD)
    const uint32_t i = blockIdx.x % kVisGroups, g = i % kXcds * (kVisGroups / kXcds) + i / kXcds, nb = gridDim.x / kVisGroups;
    const uint32_t u0 = g * share, end = n_units > u0 ? min(share, n_units - u0) : 0;  // units of this group
    uint32_t t = blockIdx.x / kVisGroups - nb;   // lane 0: the unit to take next, less nb (the first of each wavefront are dealt)
    uint32_t next = 0, j1 = 0, r = 0;       // the current unit's next and last set, its receiver (wave-uniform)
    bool walking = false, hit = false;
    f3 a = mk(0.f, 0.f, 0.f);
    size_t o = 0;
    uint32_t j = 0;
    int ref = kNoRef, sp = 0, park = kNoRef;  // kNoRef / kNoRef whenever the lane is not walking
    f3 d = mk(0.f, 0.f, 1.f), inv = mk(1.f, 1.f, 1.f), oi = mk(0.f, 0.f, 0.f);
    float t_hi = 0.f;
    Octant oq = octant<W>(inv);
    for (;;) {
        for (uint64_t idle = __ballot(!walking); idle; idle = __ballot(!walking)) {
            if (next >= j1) {  // the unit is handed out: the next one
                const uint32_t k = nb + __builtin_amdgcn_readfirstlane(t);
                if (k >= end) break;
                const uint32_t u = u0 + k, c = u / n_rx;
                r = u % n_rx;
                next = c * kVisChunk;
                j1 = min(n_sets, next + kVisChunk);
                if (lane == 0) t = taken ? atomicAdd(&taken[32 * g], 1u) : t + nb;  // (used at the next unit: no wait here)
            }
            const uint32_t avail = min(j1 - next, (uint32_t)__popcll(idle));
            if (!walking && mbcnt(idle) < avail) {
                j = next + mbcnt(idle);
                o = (size_t)r * n_sets + j;
                a = mk(rx[3 * r], rx[3 * r + 1], rx[3 * r + 2]);
                // the set-up of occluded(a, recv[j]), walked from the receiver
                const f3 dv = xyz(recv[j]) - a;
                const float L = len(dv);
                d = (1.0f / L) * dv;
                inv = safe_inv(d);
                oi = times(a, inv);
                oq = octant<W>(inv);
                t_hi = L - eps_self;
                ref = t_hi > eps_self ? S.root : kNoRef;
                sp = 0;
                park = kNoRef;
                hit = false;
                walking = true;
            }
            next += avail;
        }
        const uint32_t n_busy = (uint32_t)__popcll(__ballot(walking));
        if (n_busy == 0) break;  // nothing left
        uint32_t n_walk = n_busy;
        for (;;) {
            for (;;) {
                if (ref < 0 && ref != kNoRef && park == kNoRef) {
                    park = ref;
                    ref = sp > 0 ? stk.get(--sp) : kNoRef;
                }
                const uint32_t n_park = (uint32_t)__popcll(__ballot(park != kNoRef));
                if (!__ballot(ref >= 0) || 2 * n_park >= n_walk) break;
                if (ref >= 0) {
                    stk.visit();
                    if (!step_any<W>(S, ref, sp, oq, inv, oi, eps_self, t_hi, stk))
                        ref = sp > 0 ? stk.get(--sp) : kNoRef;
                }
            }
            if (park != kNoRef) {
                const int v = -1 - park;
                const int first = v >> 3, cnt = (v & 7) + 1;
                stk.test(cnt);
                for (int q = 0; q < cnt; ++q) {
                    const float4 dp = ld4(S.disk, (uint32_t)(first + q) * 32u);
                    const float4 dn = ld4(S.disk, (uint32_t)(first + q) * 32u + 16u);
                    float th, d2;
                    const bool h = disk_hit(a, d, xyz(dp), xyz(dn), S.r2, th, d2);
                    if (h & (__float_as_int(dn.w) != (int)j) & (th > eps_self) & (th < t_hi)) {
                        hit = true;
                        break;
                    }
                }
                park = kNoRef;
                if (hit) ref = kNoRef;
            }
            const bool done = walking && ref == kNoRef && park == kNoRef;
            if (done) {
                out[o] = hit ? 0 : 1;
                walking = false;
            }
            n_walk = (uint32_t)__popcll(__ballot(walking));
            if (n_walk == 0 || (n_walk << kVisRefillShift) <= n_busy) break;
        }
    }
}

template <int W>
uint32_t visibility_cap() {
    static const uint32_t cap = resident_blocks((const void *)k_visibility<W>, kWave);
    return cap;
}

uint32_t visibility_grid(uint32_t width) {
    const uint32_t cap = width == 8 ? visibility_cap<8>() : width == 4 ? visibility_cap<4>() : visibility_cap<2>();
    return std::max<uint32_t>(kVisGroups, cap / kVisGroups * kVisGroups);
}

void launch_visibility(const DevScene &S, const float *rx, uint32_t n_rx, const float4 *recv, uint32_t n_sets,
                       float eps_self, uint8_t *out, uint32_t *taken, hipStream_t s) {
    const uint32_t grid = visibility_grid((uint32_t)S.width);
    const uint32_t n_units = (n_sets + kVisChunk - 1) / kVisChunk * n_rx;
    const uint32_t share = (n_units + kVisGroups - 1) / kVisGroups;
    if (share <= 2 * (grid / kVisGroups)) taken = nullptr;  // one or two units per wavefront: dealt
    else fill_u32(taken, 0, 32 * kVisGroups, s);
    switch (S.width) {
        case 8: hipLaunchKernelGGL(k_visibility<8>, dim3(grid), dim3(kWave), 0, s, S, rx, n_rx, recv, n_sets, eps_self,
                                   out, share, taken); break;
        case 4: hipLaunchKernelGGL(k_visibility<4>, dim3(grid), dim3(kWave), 0, s, S, rx, n_rx, recv, n_sets, eps_self,
                                   out, share, taken); break;
        default: hipLaunchKernelGGL(k_visibility<2>, dim3(grid), dim3(kWave), 0, s, S, rx, n_rx, recv, n_sets,
                                    eps_self, out, share, taken); break;
    }
}

__global__ void k_recv_copy(const float4 *__restrict__ recv, uint32_t n, float *__restrict__ out) {
    for (uint32_t j = blockIdx.x * blockDim.x + threadIdx.x; j < n; j += gridDim.x * blockDim.x) {
        const float4 c = recv[j];
        out[3 * (size_t)j] = c.x;
        out[3 * (size_t)j + 1] = c.y;
        out[3 * (size_t)j + 2] = c.z;
    }
}

void launch_recv_copy(const float4 *recv, uint32_t n, float *out, hipStream_t s) {
    hipLaunchKernelGGL(k_recv_copy, dim3(std::min<uint32_t>((n + 255) / 256, 8192)), dim3(256), 0, s, recv, n, out);
}

}  // namespace pcrt
