// Device-wide exclusive scan and LSD radix sort (64-bit keys, 32-bit
// payload), shared by the hierarchy build and the diffuse-record ordering.
#include "common.h"
#include "internal.h"

namespace pcrt {

// LSD, 8-bit digits, 64-bit keys with 32-bit payload. Per pass: tile
// histograms, one exclusive scan in digit-major order, stable scatter with a
// wavefront multisplit (8 ballots per key) for the in-tile rank.
constexpr int kRsBlock = 256;
constexpr int kRsRounds = 8;
constexpr int kRsTile = kRsBlock * kRsRounds;

__global__ void k_rs_hist(const uint64_t *__restrict__ key, uint32_t n, int shift, uint32_t *__restrict__ hist,
                          uint32_t tiles) {
    __shared__ uint32_t h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    uint32_t base = blockIdx.x * kRsTile;
    for (int r = 0; r < kRsRounds; ++r) {
        uint32_t i = base + r * kRsBlock + threadIdx.x;
        if (i < n) atomicAdd(&h[(key[i] >> shift) & 255], 1u);
    }
    __syncthreads();
    hist[threadIdx.x * tiles + blockIdx.x] = h[threadIdx.x];
}

__global__ void k_rs_scatter(const uint64_t *__restrict__ kin, const uint32_t *__restrict__ vin,
                             uint64_t *__restrict__ kout, uint32_t *__restrict__ vout, uint32_t n, int shift,
                             const uint32_t *__restrict__ hist, uint32_t tiles) {
    __shared__ uint32_t base[256], run[256];
    __shared__ uint32_t wcnt[kRsBlock / kWave][256];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    base[threadIdx.x] = hist[threadIdx.x * tiles + blockIdx.x];
    run[threadIdx.x] = 0;
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    for (int r = 0; r < kRsRounds; ++r) {
        for (int w = 0; w < kRsBlock / kWave; ++w) wcnt[w][threadIdx.x] = 0;
        __syncthreads();
        uint32_t i = blockIdx.x * kRsTile + r * kRsBlock + threadIdx.x;
        bool ok = i < n;
        uint64_t k = ok ? kin[i] : 0;
        uint32_t dg = (uint32_t)(k >> shift) & 255;
        uint64_t peers = __ballot(ok);
        for (int b = 0; b < 8; ++b) {
            bool bit = (dg >> b) & 1;
            uint64_t m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        uint32_t rank = __popcll(peers & lt);
        if (ok && rank == 0) wcnt[wave][dg] = __popcll(peers);
        __syncthreads();
        if (ok) {
            uint32_t before = 0;
            for (int w = 0; w < wave; ++w) before += wcnt[w][dg];
            uint32_t dst = base[dg] + run[dg] + before + rank;
            kout[dst] = k;
            vout[dst] = vin[i];
        }
        __syncthreads();
        uint32_t tot = 0;
        for (int w = 0; w < kRsBlock / kWave; ++w) tot += wcnt[w][threadIdx.x];
        run[threadIdx.x] += tot;
        __syncthreads();
    }
}


// Exclusive scan. Two launches, reduce then scan: tile sums, then every tile
// adds up the sums before its own (a few hundred to a few thousand words out
// of L2) and scans itself. Nothing has to be cleared beforehand and no block
// waits for another. Arrays of one tile take one launch. What bounds it is
// the launches (a solve has ten or so scans of a few thousand words), then
// the array's two reads and one write. Against block scans, a one-block scan
// of their sums and an add pass: 43 200-disk room, nine scans of 4 096 words
// 86 -> 20 us; 72 M marks of a 64-pose batch 650 -> 230 us.
constexpr uint32_t kScanOne = 16;  // words per thread of a scan in one block

__device__ __forceinline__ uint32_t wave_scan_u(uint32_t v) {  // inclusive
    const int lane = threadIdx.x & (kWave - 1);
    for (int o = 1; o < kWave; o <<= 1) {
        const uint32_t t = __shfl_up(v, o, kWave);
        if (lane >= o) v += t;
    }
    return v;
}

// Exclusive sum of v over a block of 1024 threads; part: 16 words of LDS.
__device__ __forceinline__ uint32_t block_scan_u(uint32_t v, uint32_t *part, uint32_t &total) {
    const uint32_t w = threadIdx.x / kWave;
    const uint32_t in = wave_scan_u(v);
    if ((threadIdx.x & (kWave - 1)) == kWave - 1) part[w] = in;
    __syncthreads();
    uint32_t before = 0, all = 0;
    for (uint32_t i = 0; i < 16; ++i) {
        const uint32_t p = part[i];
        before += i < w ? p : 0u;
        all += p;
    }
    __syncthreads();
    total = all;
    return before + in - v;
}

// IPT words per thread, four at a time at index 4 t + 4096 k of the tile.
template <uint32_t IPT>
__global__ __launch_bounds__(1024) void k_scan_sums(const uint32_t *__restrict__ a, uint32_t n,
                                                    uint32_t *__restrict__ blk) {
    __shared__ uint32_t part[16];
    const uint64_t base = (uint64_t)blockIdx.x * (1024u * IPT);
    uint32_t s = 0;
    for (uint32_t k = 0; k < IPT / 4; ++k) {
        const uint64_t i = base + k * 4096u + threadIdx.x * 4u;
        if (i + 4 <= n) {
            const uint4 v = *(const uint4 *)(a + i);
            s += v.x + v.y + v.z + v.w;
        } else {
            for (uint64_t j = i; j < n && j < i + 4; ++j) s += a[j];
        }
    }
    uint32_t total;
    (void)block_scan_u(s, part, total);
    if (threadIdx.x == 0) blk[blockIdx.x] = total;
}

// blk: the tile sums; the array's total goes to blk[total_at] (beyond them).
template <uint32_t IPT>
__global__ __launch_bounds__(1024) void k_scan_tiles(uint32_t *__restrict__ a, uint32_t n, uint32_t *blk,
                                                     uint32_t total_at) {
    __shared__ uint32_t part[16];
    uint32_t before = 0, run, all;
    if (gridDim.x > 1) {
        uint32_t s = 0;
        for (uint32_t i = threadIdx.x; i < blockIdx.x; i += 1024) s += blk[i];
        (void)block_scan_u(s, part, before);
    }
    const uint64_t base = (uint64_t)blockIdx.x * (1024u * IPT);
    run = before;
    for (uint32_t k = 0; k < IPT / 4; ++k) {
        const uint64_t i = base + k * 4096u + threadIdx.x * 4u;
        if (base + k * 4096u >= n) break;  // block-uniform
        uint32_t v[4] = {0, 0, 0, 0};
        if (i + 4 <= n) {
            const uint4 q = *(const uint4 *)(a + i);
            v[0] = q.x;
            v[1] = q.y;
            v[2] = q.z;
            v[3] = q.w;
        } else {
            for (uint32_t j = 0; j < 4; ++j) v[j] = i + j < n ? a[i + j] : 0u;
        }
        const uint32_t e0 = run + block_scan_u(v[0] + v[1] + v[2] + v[3], part, all);
        const uint32_t e1 = e0 + v[0], e2 = e1 + v[1], e3 = e2 + v[2];
        if (i + 4 <= n) {
            *(uint4 *)(a + i) = make_uint4(e0, e1, e2, e3);
        } else {
            const uint32_t e[4] = {e0, e1, e2, e3};
            for (uint32_t j = 0; j < 4; ++j)
                if (i + j < n) a[i + j] = e[j];
        }
        run += all;
    }
    if (blockIdx.x + 1 == gridDim.x && threadIdx.x == 0) blk[total_at] = run;
}

// Sort of up to kRsSmall keys in one block: all digit passes in LDS, with the
// same stable multisplit (a wavefront owns 256 consecutive positions, four
// rounds of 64). One launch instead of five per digit: the 4 096 records of a
// small solve 87 -> 30 us with the passes before and after it.
constexpr uint32_t kRsSmall = 4096;
constexpr uint32_t kRsSmallRounds = kRsSmall / 1024;

__global__ __launch_bounds__(1024) void k_rs_small(uint64_t *key, uint32_t *val, uint32_t n, int bit_lo, int bit_hi) {
    __shared__ uint64_t k_s[kRsSmall];
    __shared__ uint32_t v_s[kRsSmall];
    __shared__ uint16_t cnt[16][256];  // per wavefront and digit: keys so far, then the digit's start
    __shared__ uint32_t part[16];
    const uint32_t lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    uint64_t k[kRsSmallRounds];
    uint32_t v[kRsSmallRounds], rank[kRsSmallRounds];
    for (uint32_t r = 0; r < kRsSmallRounds; ++r) {
        const uint32_t i = wave * (kRsSmall / 16) + r * kWave + lane;
        k[r] = i < n ? key[i] : ~0ull;
        v[r] = i < n ? val[i] : 0u;
    }
    for (int shift = bit_lo; shift < bit_hi; shift += 8) {
        for (uint32_t i = threadIdx.x; i < 16u * 256u; i += 1024u) (&cnt[0][0])[i] = 0;
        __syncthreads();
        for (uint32_t r = 0; r < kRsSmallRounds; ++r) {
            const uint32_t i = wave * (kRsSmall / 16) + r * kWave + lane;
            const bool ok = i < n;
            const uint32_t dg = (uint32_t)(k[r] >> shift) & 255u;
            uint64_t peers = __ballot(ok);
            for (int b = 0; b < 8; ++b) {
                const bool bit = (dg >> b) & 1u;
                const uint64_t m = __ballot(bit);
                peers &= bit ? m : ~m;
            }
            const uint32_t below = mbcnt(peers);
            rank[r] = ok ? cnt[wave][dg] + below : 0u;
            wave_sync();
            if (ok && below == 0) cnt[wave][dg] = (uint16_t)(cnt[wave][dg] + __popcll(peers));
            wave_sync();
        }
        __syncthreads();
        // thread t: digit t / 4, wavefronts 4 (t % 4) .. + 3, in digit-major order
        const uint32_t d0 = threadIdx.x / 4, w0 = 4 * (threadIdx.x % 4);
        uint32_t c[4], s = 0;
        for (int j = 0; j < 4; ++j) {
            c[j] = cnt[w0 + j][d0];
            s += c[j];
        }
        uint32_t all, run = block_scan_u(s, part, all);
        for (int j = 0; j < 4; ++j) {
            cnt[w0 + j][d0] = (uint16_t)run;
            run += c[j];
        }
        __syncthreads();
        for (uint32_t r = 0; r < kRsSmallRounds; ++r) {
            const uint32_t i = wave * (kRsSmall / 16) + r * kWave + lane;
            if (i < n) {
                const uint32_t to = cnt[wave][(uint32_t)(k[r] >> shift) & 255u] + rank[r];
                k_s[to] = k[r];
                v_s[to] = v[r];
            }
        }
        __syncthreads();
        for (uint32_t r = 0; r < kRsSmallRounds; ++r) {
            const uint32_t i = wave * (kRsSmall / 16) + r * kWave + lane;
            if (i < n) {
                k[r] = k_s[i];
                v[r] = v_s[i];
            }
        }
        __syncthreads();
    }
    for (uint32_t r = 0; r < kRsSmallRounds; ++r) {
        const uint32_t i = wave * (kRsSmall / 16) + r * kWave + lane;
        if (i < n) {
            key[i] = k[r];
            val[i] = v[r];
        }
    }
}

uint32_t scan_blk_words(uint32_t n) { return (n + 1023) / 1024 + 1; }
uint32_t radix_hist_words(uint32_t n) { return 256u * ((n + kRsTile - 1) / kRsTile); }

// In-place exclusive scan (a 16-byte aligned); the total lands in
// blk[ceil(n / 1024)]. Tiles of 4 096 words; beyond 2^22 words of 16 384, so
// that a tile adds up a few thousand sums at most.
void exclusive_scan(uint32_t *a, uint32_t n, uint32_t *blk, hipStream_t s) {
    const uint32_t total_at = (n + 1023) / 1024;
    if (n <= 1024 * kScanOne) {
        hipLaunchKernelGGL(k_scan_tiles<kScanOne>, dim3(1), dim3(1024), 0, s, a, n, blk, total_at);
    } else if (n <= (1u << 22)) {
        const uint32_t nb = (n + 4095) / 4096;
        hipLaunchKernelGGL(k_scan_sums<4>, dim3(nb), dim3(1024), 0, s, a, n, blk);
        hipLaunchKernelGGL(k_scan_tiles<4>, dim3(nb), dim3(1024), 0, s, a, n, blk, total_at);
    } else {
        const uint32_t nb = (uint32_t)(((uint64_t)n + 16383) / 16384);
        hipLaunchKernelGGL(k_scan_sums<16>, dim3(nb), dim3(1024), 0, s, a, n, blk);
        hipLaunchKernelGGL(k_scan_tiles<16>, dim3(nb), dim3(1024), 0, s, a, n, blk, total_at);
    }
}

// Sorts (key, value) by key bits [bit_lo, bit_hi) with 8-bit passes; returns
// true if the sorted data ended in (k1, v1), false if in (k0, v0).
bool radix_sort_u64(uint64_t *k0, uint32_t *v0, uint64_t *k1, uint32_t *v1, uint32_t n, int bit_lo, int bit_hi,
                    uint32_t *hist, uint32_t *blk, hipStream_t s) {
    if (n <= kRsSmall) {
        hipLaunchKernelGGL(k_rs_small, dim3(1), dim3(1024), 0, s, k0, v0, n, bit_lo, bit_hi);
        return false;
    }
    const uint32_t tiles = (n + kRsTile - 1) / kRsTile;
    bool flip = false;
    for (int shift = bit_lo; shift < bit_hi; shift += 8) {
        uint64_t *ki = flip ? k1 : k0, *ko = flip ? k0 : k1;
        uint32_t *vi = flip ? v1 : v0, *vo = flip ? v0 : v1;
        hipLaunchKernelGGL(k_rs_hist, dim3(tiles), dim3(kRsBlock), 0, s, ki, n, shift, hist, tiles);
        exclusive_scan(hist, 256 * tiles, blk, s);
        hipLaunchKernelGGL(k_rs_scatter, dim3(tiles), dim3(kRsBlock), 0, s, ki, vi, ko, vo, n, shift, hist, tiles);
        flip = !flip;
    }
    return flip;
}

}  // namespace pcrt
