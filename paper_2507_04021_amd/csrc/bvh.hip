// Scene ingest and linear BVH build over disk bounding boxes.
//
// The paper hands point-set AABBs to a hardware ray-tracing API (Sec. II-A).
// gfx950 has no ray-tracing units, so the hierarchy is built here: Morton
// codes of disk centres, a hand-written LSD radix sort, the Karras (2012)
// binary radix tree over the sorted codes, and a bottom-up refit that also
// collapses small subtrees into leaves of up to `leaf_size` disks.
#include "common.h"
#include "internal.h"

#include <hip/hip_fp16.h>
#include <vector>

namespace pcrt {

// --------------------------------------------------------------- ingest
// Validates and normalises each point; writes the by-id tables and the
// per-block bounds of disk centres. status bits: 1 non-finite position,
// 2 zero or non-finite normal.
__device__ __forceinline__ void max_to(uint32_t v, uint32_t *to) {  // (looks first: most blocks add nothing)
    if (v > __hip_atomic_load(to, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(to, v);
}

// A block takes kIngest points: an atomic on one word costs 11 ns whoever issues it, and one per
// wavefront and statistic was nearly all of the 0.36 ms this took for 1M points (now 0.022; 68 MB read and written,
// 0.014 at the rate of a large copy).
constexpr uint32_t kIngest = 1024;
__global__ __launch_bounds__(256) void k_ingest(const float *__restrict__ pos, const float *__restrict__ nrm,
                                                const uint16_t *__restrict__ mat, const uint32_t *__restrict__ surf,
                                                uint32_t n, float4 *__restrict__ pos_id, float4 *__restrict__ nrm_id,
                                                float *__restrict__ blk_bounds, uint32_t *__restrict__ stat) {
    __shared__ float red[6][4];
    __shared__ uint32_t redi[3][4];
    float b[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
    uint32_t st[3] = {0, 0, 0};  // bad, largest surface, largest material
    for (uint32_t k = 0; k < kIngest / 256; ++k) {
        const uint32_t i = blockIdx.x * kIngest + k * 256 + threadIdx.x;
        if (i >= n) break;
        uint32_t bad = 0;
        float px = pos[3 * i], py = pos[3 * i + 1], pz = pos[3 * i + 2];
        float nx = nrm[3 * i], ny = nrm[3 * i + 1], nz = nrm[3 * i + 2];
        if (!(isfinite(px) && isfinite(py) && isfinite(pz))) bad |= 1;
        float l2 = nx * nx + ny * ny + nz * nz;
        if (!(l2 > 0.f) || !isfinite(l2)) bad |= 2;
        float il = bad & 2 ? 0.f : 1.0f / sqrtf(l2);
        uint32_t s = surf[i], m = mat[i];
        pos_id[i] = make_float4(px, py, pz, __uint_as_float(s));
        nrm_id[i] = make_float4(nx * il, ny * il, nz * il, __uint_as_float(m));
        st[0] |= bad;
        st[1] = max(st[1], s);
        st[2] = max(st[2], m);
        if (!bad) {
            const float p[3] = {px, py, pz};
            for (int a = 0; a < 3; ++a) {
                b[a] = fminf(b[a], p[a]);
                b[3 + a] = fmaxf(b[3 + a], p[a]);
            }
        }
    }
    for (int o = 32; o > 0; o >>= 1) {
        for (int a = 0; a < 3; ++a) {
            b[a] = fminf(b[a], __shfl_xor(b[a], o, kWave));
            b[3 + a] = fmaxf(b[3 + a], __shfl_xor(b[3 + a], o, kWave));
        }
        st[0] |= __shfl_xor(st[0], o, kWave);
        st[1] = max(st[1], (uint32_t)__shfl_xor(st[1], o, kWave));
        st[2] = max(st[2], (uint32_t)__shfl_xor(st[2], o, kWave));
    }
    if (threadIdx.x % kWave == 0) {
        for (int a = 0; a < 6; ++a) red[a][threadIdx.x / kWave] = b[a];
        for (int a = 0; a < 3; ++a) redi[a][threadIdx.x / kWave] = st[a];
    }
    __syncthreads();
    if (threadIdx.x < 6) {
        const float *r = red[threadIdx.x];
        blk_bounds[6 * blockIdx.x + threadIdx.x] =
            threadIdx.x < 3 ? fminf(fminf(r[0], r[1]), fminf(r[2], r[3])) : fmaxf(fmaxf(r[0], r[1]), fmaxf(r[2], r[3]));
    }
    if (threadIdx.x == 64) {
        const uint32_t bad = redi[0][0] | redi[0][1] | redi[0][2] | redi[0][3];
        if (bad) atomicOr(&stat[0], bad);
        max_to(max(max(redi[1][0], redi[1][1]), max(redi[1][2], redi[1][3])), &stat[1]);
        max_to(max(max(redi[2][0], redi[2][1]), max(redi[2][2], redi[2][3])), &stat[2]);
    }
}

// Final bounds over the per-block bounds (one block).
__global__ void k_bounds(const float *__restrict__ blk, uint32_t nblk, float *__restrict__ out) {
    __shared__ float red[6][256];
    float v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};
    for (uint32_t b = threadIdx.x; b < nblk; b += blockDim.x)
        for (int a = 0; a < 3; ++a) {
            v[a] = fminf(v[a], blk[6 * b + a]);
            v[3 + a] = fmaxf(v[3 + a], blk[6 * b + 3 + a]);
        }
    for (int a = 0; a < 6; ++a) red[a][threadIdx.x] = v[a];
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s)
            for (int a = 0; a < 3; ++a) {
                red[a][threadIdx.x] = fminf(red[a][threadIdx.x], red[a][threadIdx.x + s]);
                red[3 + a][threadIdx.x] = fmaxf(red[3 + a][threadIdx.x], red[3 + a][threadIdx.x + s]);
            }
        __syncthreads();
    }
    if (threadIdx.x == 0)
        for (int a = 0; a < 6; ++a) out[a] = red[a][0];
}

__device__ __forceinline__ uint64_t spread21(uint64_t x) {
    x &= 0x1fffffull;
    x = (x | x << 32) & 0x1f00000000ffffull;
    x = (x | x << 16) & 0x1f0000ff0000ffull;
    x = (x | x << 8) & 0x100f00f00f00f00full;
    x = (x | x << 4) & 0x10c30c30c30c30c3ull;
    x = (x | x << 2) & 0x1249249249249249ull;
    return x;
}

// 63-bit Morton code of each disk centre in the scene bounds.
__global__ void k_morton(const float4 *__restrict__ pos_id, uint32_t n, const float *__restrict__ bounds,
                         uint64_t *__restrict__ code, uint32_t *__restrict__ idx) {
    uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float4 p = pos_id[i];
    float c[3] = {p.x, p.y, p.z};
    uint64_t q[3];
    for (int a = 0; a < 3; ++a) {
        float ext = bounds[3 + a] - bounds[a];
        float u = ext > 0.f ? (c[a] - bounds[a]) / ext : 0.5f;
        u = fminf(fmaxf(u, 0.f), 1.f);
        q[a] = (uint64_t)(u * 2097151.0f);
    }
    code[i] = spread21(q[0]) << 2 | spread21(q[1]) << 1 | spread21(q[2]);
    idx[i] = i;
}

// -------------------------------------------------- Karras radix tree
__device__ __forceinline__ int delta(const uint64_t *k, int n, int i, int j) {
    if (j < 0 || j >= n) return -1;
    uint64_t a = k[i], b = k[j];
    if (a == b) return 64 + __clz((uint32_t)i ^ (uint32_t)j);
    return __clzll(a ^ b);
}

// Internal node i of n-1: children (int index or leaf encoded as ~pos) and
// covered range [first, last] of sorted positions.
__global__ void k_karras(const uint64_t *__restrict__ k, int n, int2 *__restrict__ child, int2 *__restrict__ range,
                         int *__restrict__ parent_int, int *__restrict__ parent_leaf) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n - 1) return;
    int d = (delta(k, n, i, i + 1) - delta(k, n, i, i - 1)) >= 0 ? 1 : -1;
    int dmin = delta(k, n, i, i - d);
    int lmax = 2;
    while (delta(k, n, i, i + lmax * d) > dmin) lmax <<= 1;
    int l = 0;
    for (int t = lmax >> 1; t >= 1; t >>= 1)
        if (delta(k, n, i, i + (l + t) * d) > dmin) l += t;
    int j = i + l * d;
    int dnode = delta(k, n, i, j);
    int s = 0;
    int div = 2;
    for (;;) {
        int t = (l + div - 1) / div;
        if (delta(k, n, i, i + (s + t) * d) > dnode) s += t;
        if (t == 1) break;
        div <<= 1;
    }
    int gamma = i + s * d + min(d, 0);
    int first = min(i, j), last = max(i, j);
    int left = (first == gamma) ? ~gamma : gamma;
    int right = (last == gamma + 1) ? ~(gamma + 1) : gamma + 1;
    child[i] = make_int2(left, right);
    range[i] = make_int2(first, last);
    if (left < 0) parent_leaf[~left] = i;
    else parent_int[left] = i;
    if (right < 0) parent_leaf[~right] = i;
    else parent_int[right] = i;
    if (i == 0) parent_int[0] = -1;
}

// Leaf-ordered disks (unless disk is null) and their padded bounding boxes.
__global__ void k_gather(const float4 *__restrict__ pos_id, const float4 *__restrict__ nrm_id,
                         const uint32_t *__restrict__ perm, uint32_t n, float r, float4 *__restrict__ disk,
                         float *__restrict__ dbox) {
    uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint32_t id = perm[i];
    float4 p = pos_id[id], nn = nrm_id[id];
    if (disk) {
        disk[2 * i] = make_float4(p.x, p.y, p.z, __int_as_float((int)id));
        disk[2 * i + 1] = make_float4(nn.x, nn.y, nn.z, 0.f);
    }
    float c[3] = {p.x, p.y, p.z}, nv[3] = {nn.x, nn.y, nn.z};
    for (int a = 0; a < 3; ++a) {
        // tight half-extent of a disk along axis a, padded so that FP32
        // slab tests stay conservative
        float h = r * sqrtf(fmaxf(0.f, 1.f - nv[a] * nv[a]));
        float pad = 1e-5f + 2e-6f * (fabsf(c[a]) + r);
        dbox[6 * i + a] = c[a] - h - pad;
        dbox[6 * i + 3 + a] = c[a] + h + pad;
    }
}

// Bottom-up refit: the second thread to reach a node computes its box and
// writes its traversal record; children covering <= L disks become leaves.
__global__ void k_refit(int n, int L, const int2 *__restrict__ child, const int2 *__restrict__ range,
                        const int *__restrict__ parent_int, const int *__restrict__ parent_leaf,
                        const float *__restrict__ dbox, float *ibox, uint32_t *flags, float4 *__restrict__ node) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int cur = parent_leaf[i];
    while (cur >= 0) {
        __threadfence();
        if (atomicAdd(&flags[cur], 1u) == 0) return;
        __threadfence();
        int2 ch = child[cur];
        float b[2][6];
        int ref[2];
        int cc[2] = {ch.x, ch.y};
        for (int s = 0; s < 2; ++s) {
            int c = cc[s];
            if (c < 0) {
                int p = ~c;
                for (int a = 0; a < 6; ++a) b[s][a] = dbox[6 * p + a];
                ref[s] = leaf_ref(p, 1);
            } else {
                const volatile float *vb = ibox + 6 * c;
                for (int a = 0; a < 6; ++a) b[s][a] = vb[a];
                int2 rg = range[c];
                int cnt = rg.y - rg.x + 1;
                ref[s] = cnt <= L ? leaf_ref(rg.x, cnt) : c;
            }
        }
        volatile float *ob = ibox + 6 * cur;
        for (int a = 0; a < 3; ++a) {
            ob[a] = fminf(b[0][a], b[1][a]);
            ob[3 + a] = fmaxf(b[0][3 + a], b[1][3 + a]);
        }
        float4 *nd = node + 4 * (size_t)cur;
        nd[0] = make_float4(b[0][0], b[0][1], b[0][2], b[0][3]);
        nd[1] = make_float4(b[0][4], b[0][5], b[1][0], b[1][1]);
        nd[2] = make_float4(b[1][2], b[1][3], b[1][4], b[1][5]);
        nd[3] = make_float4(__int_as_float(ref[0]), __int_as_float(ref[1]), 0.f, 0.f);
        cur = parent_int[cur];
    }
}

// Node records when every internal node's box is already known (the
// clustering builder records them at merge time): one thread per node, no
// bottom-up climb. Same records as k_refit.
__global__ void k_node_records(int n_int, int L, const int2 *__restrict__ child, const int2 *__restrict__ range,
                               const float *__restrict__ dbox, const float *__restrict__ ibox,
                               float4 *__restrict__ node) {
    const int cur = blockIdx.x * blockDim.x + threadIdx.x;
    if (cur >= n_int) return;
    const int2 ch = child[cur];
    float b[2][6];
    int ref[2];
    const int cc[2] = {ch.x, ch.y};
    for (int s = 0; s < 2; ++s) {
        const int c = cc[s];
        if (c < 0) {
            const int p = ~c;
            for (int a = 0; a < 6; ++a) b[s][a] = dbox[6 * (size_t)p + a];
            ref[s] = leaf_ref(p, 1);
        } else {
            for (int a = 0; a < 6; ++a) b[s][a] = ibox[6 * (size_t)c + a];
            const int2 rg = range[c];
            const int cnt = rg.y - rg.x + 1;
            ref[s] = cnt <= L ? leaf_ref(rg.x, cnt) : c;
        }
    }
    float4 *nd = node + 4 * (size_t)cur;
    nd[0] = make_float4(b[0][0], b[0][1], b[0][2], b[0][3]);
    nd[1] = make_float4(b[0][4], b[0][5], b[1][0], b[1][1]);
    nd[2] = make_float4(b[1][2], b[1][3], b[1][4], b[1][5]);
    nd[3] = make_float4(__int_as_float(ref[0]), __int_as_float(ref[1]), 0.f, 0.f);
}

// Depth (number of internal ancestors) of each sorted leaf; max into *depth.
__global__ void k_depth(int n, const int *__restrict__ parent_int, const int *__restrict__ parent_leaf,
                        uint32_t *__restrict__ depth) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    uint32_t dd = 0;
    for (int cur = parent_leaf[i]; cur >= 0; cur = parent_int[cur]) ++dd;
    atomicMax(depth, dd);
}

__global__ void k_fill_u32(uint32_t *p, uint32_t v, size_t n) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}

__global__ void k_fill_u64(uint64_t *p, uint64_t v, size_t n) {
    size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; i < n; i += (size_t)gridDim.x * blockDim.x) p[i] = v;
}

// ------------------------------------------------------------ host side
static inline uint32_t cdiv(uint64_t a, uint64_t b) { return (uint32_t)((a + b - 1) / b); }

void fill_u32(uint32_t *p, uint32_t v, size_t n, hipStream_t s) {
    if (!n) return;
    uint32_t g = (uint32_t)std::min<size_t>(cdiv(n, 256), 4096);
    hipLaunchKernelGGL(k_fill_u32, dim3(g), dim3(256), 0, s, p, v, n);
}
void fill_u64(uint64_t *p, uint64_t v, size_t n, hipStream_t s) {
    if (!n) return;
    uint32_t g = (uint32_t)std::min<size_t>(cdiv(n, 256), 4096);
    hipLaunchKernelGGL(k_fill_u64, dim3(g), dim3(256), 0, s, p, v, n);
}

// --------------------------------------------------- clustering builder
// Parallel locally-ordered clustering (Meister & Bittner, 2018) over the
// Morton-ordered disks. Each pass: every cluster finds, within +-kPlocRadius
// positions, the cluster whose merged box has the smallest surface area
// (ties: smaller index); mutual nearest pairs merge into a new internal node
// (lower index keeps the slot) and the list is compacted by an exclusive
// scan. The order on pairs (area, lower index, higher index) is total, so
// the globally cheapest pair is always mutual and every pass merges at least
// one pair. Internal nodes are numbered in creation order; the root is the
// last. The disks are then renumbered in depth-first order so that every
// subtree owns a contiguous disk range, which is what the refit and the leaf
// references expect.
// Search radius, measured on the 1M-point office (diffuse / refine / trace
// ms): 4 -> 34.4 / 4.8 / 3.1, 6 -> 33.9 / 4.5 / 3.1, 8 -> 34.6 / 4.4 / 3.1,
// 16 -> 35.1 / 4.8 / 3.3, 32 -> 35.8 / 4.6 / 3.4, 64 -> 36.3 / 4.5 / 3.4.
constexpr int kPlocRadius = 6;

__device__ __forceinline__ float merged_half_area(const float *a, const float *b) {
    const float dx = fmaxf(a[3], b[3]) - fminf(a[0], b[0]);
    const float dy = fmaxf(a[4], b[4]) - fminf(a[1], b[1]);
    const float dz = fmaxf(a[5], b[5]) - fminf(a[2], b[2]);
    return dx * dy + dy * dz + dz * dx;
}

// Exclusive prefixes of the tiles of one launch, passed on from tile to tile
// (decoupled look-back; Merrill, Garland: Single-pass Parallel Prefix Scan with Decoupled
// Look-back, 2016): a tile publishes its sum, adds up what the tiles
// before it have published, 64 at a time, back to the first that already has
// its inclusive prefix, and publishes its own. Tiles are numbered by an atomic
// ticket, so every tile waited for has been started by a running block. Flag
// and payload (two 31-bit counts) share one 64-bit word, so relaxed atomics do.
// Every wait ends: after kTilePolls looks (a second or so; a wait takes some
// microseconds) the tile gives up with a prefix of 0 and sets the build's fail
// word: later levels then find no frontier, and the host, which looks at the
// word before it follows any count or reference, refuses the scene.
constexpr uint64_t kTileSum = 1ull << 62, kTilePrefix = 2ull << 62, kTileMask = kTileSum - 1;
constexpr uint32_t kTilePolls = 1u << 20;

__device__ __forceinline__ uint64_t tile_prefix(uint64_t *status, uint32_t tile, uint64_t sum,
                                                uint32_t *fail) {  // one wavefront
    const int lane = threadIdx.x & (kWave - 1);
    auto put = [&](uint64_t v) {
        if (lane == 0) __hip_atomic_store(&status[tile], v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    if (tile == 0) {
        put(kTilePrefix | sum);
        return 0;
    }
    put(kTileSum | sum);
    uint64_t before = 0;
    uint32_t polls = 0;
    for (int64_t t = (int64_t)tile - 1;; t -= kWave) {
        uint64_t v, first;
        for (;;) {
            if (++polls > kTilePolls) {
                if (lane == 0) atomicOr(fail, 1u);
                put(kTilePrefix);
                return 0;
            }
            v = t - lane < 0 ? kTilePrefix
                             : __hip_atomic_load(&status[t - lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const uint64_t full = __ballot(v >= kTilePrefix), none = __ballot(v < kTileSum);
            first = full ? (uint64_t)__ffsll((unsigned long long)full) - 1 : (uint64_t)kWave - 1;
            if (!(none & (~0ull >> (63 - first)))) break;  // every tile up to the first prefix has published
        }
        uint64_t add = (uint64_t)lane <= first ? v & kTileMask : 0ull;
        for (int o = 32; o > 0; o >>= 1) add += __shfl_xor(add, o, kWave);
        before += add;
        if (__ballot(v >= kTilePrefix)) break;
    }
    put(kTilePrefix | (before + sum));
    return before;
}

// Exclusive prefix of v (two 31-bit counts) over the launch's tiles of 64 kWaves
// threads; total: the inclusive prefix of this tile.
template <uint32_t kWaves>
__device__ __forceinline__ uint64_t tiles_scan(uint64_t *status, uint32_t tile, uint64_t v, uint64_t &total,
                                               uint32_t *fail) {
    __shared__ uint64_t part[kWaves + 1];
    const uint32_t lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    uint64_t in = v;
    for (uint32_t o = 1; o < (uint32_t)kWave; o <<= 1) {
        const uint64_t t = __shfl_up(in, o, kWave);
        if (lane >= o) in += t;
    }
    if (lane == kWave - 1) part[w] = in;
    __syncthreads();
    uint64_t all = 0;
    for (uint32_t i = 0; i < kWaves; ++i) all += part[i];
    if (w == 0) {
        const uint64_t b = tile_prefix(status, tile, all, fail);
        if (lane == 0) part[kWaves] = b;
    }
    __syncthreads();
    uint64_t before = part[kWaves];
    for (uint32_t i = 0; i < w; ++i) before += part[i];
    total = part[kWaves] + all;
    __syncthreads();
    return before + in - v;
}

// State of the passes (clustering) or levels (wide collapse) of a build.
struct PassState {
    uint32_t m, base;  // clusters (frontier nodes) of the pass, first node it creates (first wide node it writes)
};
struct PassBufs {
    PassState *st;       // by pass
    uint64_t *status[2]; // tile prefixes of even and odd passes
    uint32_t n_status;
    uint32_t *ticket;    // [2], then the number of clustering passes, then the build's fail word
};

// A pass clears the other parity's tickets and prefixes for the next one.
__device__ __forceinline__ void pass_clear(const PassBufs &B, uint32_t pass) {
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < B.n_status; i += gridDim.x * blockDim.x)
        B.status[(pass + 1) & 1][i] = 0ull;
    if (blockIdx.x == 0 && threadIdx.x == 0) B.ticket[(pass + 1) & 1] = 0u;
}

struct Clusters {
    const float *box;  // [m][6]
    const int *id;     // node, or ~leaf; null: cluster i is leaf i
    const uint32_t *size;
};

// Nearest cluster of i among those with boxes in the tile's LDS (i itself is
// excluded, ties to the smaller index); -1 if no merged area is finite.
template <int N>
__device__ __forceinline__ int ploc_nearest(const float (&bx)[6][N], int l, int lo, int hi) {
    const float me[6] = {bx[0][l], bx[1][l], bx[2][l], bx[3][l], bx[4][l], bx[5][l]};
    float best = INFINITY;
    int bj = -1;
    for (int j = lo; j <= hi; ++j) {  // increasing j: a strict < keeps the smaller index on ties
        if (j == l) continue;
        const float o[6] = {bx[0][j], bx[1][j], bx[2][j], bx[3][j], bx[4][j], bx[5][j]};
        const float c = merged_half_area(me, o);
        if (c < best) {
            best = c;
            bj = j;
        }
    }
    return bj;
}

// One clustering pass in one launch: a block loads the boxes of its
// kPlocTile clusters and 2 kPlocRadius on either side, finds the nearest
// neighbours of its own and of those within kPlocRadius (one per thread; so it
// knows which pairs are mutual), and writes merged and kept clusters at their
// scanned places. A launch covers at least the pass's m clusters; blocks
// beyond them end at once, without a ticket (11 ns each). Ten launches and a
// host round trip per pass took 3.6 ms for the 51 passes of a 1M-point build;
// this 0.69 with tiles of 256 clusters, 0.46 with these, and the tail below 0.06.
constexpr int kPlocThreads = 1024, kPlocTile = kPlocThreads - 2 * kPlocRadius;
__global__ __launch_bounds__(kPlocThreads) void k_ploc_pass(Clusters in, float *__restrict__ obox,
                                                            int *__restrict__ oid, uint32_t *__restrict__ osize,
                                                            PassBufs B, uint32_t pass, int2 *__restrict__ child,
                                                            uint32_t *__restrict__ nsize, float *__restrict__ ibox) {
    constexpr int R = kPlocRadius, N = kPlocThreads + 2 * R;
    __shared__ float bx[6][N];
    __shared__ int nn[kPlocThreads];
    __shared__ uint32_t tile_s;
    pass_clear(B, pass);
    const uint32_t m = B.st[pass].m, node_base = B.st[pass].base;
    if ((uint64_t)blockIdx.x * kPlocTile >= m) return;
    if (threadIdx.x == 0) tile_s = atomicAdd(&B.ticket[pass & 1], 1u);
    __syncthreads();
    const uint32_t tile = tile_s;
    if ((uint64_t)tile * kPlocTile >= m) return;
    const int t0 = (int)(tile * kPlocTile);  // bx[.][l] is cluster t0 + l - 2R, nn[l] and thread l cluster t0 + l - R
    for (int i = (int)threadIdx.x; i < 6 * N; i += kPlocThreads) {
        const int l = i / 6, a = i % 6, g = t0 + l - 2 * R;
        if (g >= 0 && g < (int)m) bx[a][l] = in.box[6 * (size_t)g + a];
    }
    __syncthreads();
    const int i = t0 + (int)threadIdx.x - R;
    if (i >= 0 && i < (int)m) {
        const int lo = max(0, i - R) - t0 + 2 * R, hi = min((int)m - 1, i + R) - t0 + 2 * R;
        const int j = ploc_nearest<N>(bx, (int)threadIdx.x + R, lo, hi);
        nn[threadIdx.x] = j < 0 ? -1 : j + t0 - 2 * R;
    }
    __syncthreads();
    const bool ok = (int)threadIdx.x >= R && (int)threadIdx.x < kPlocThreads - R && i < (int)m;
    const int j = ok ? nn[threadIdx.x] : -1;
    const bool mutual = j >= 0 && nn[j - t0 + R] == i;
    const bool merge = mutual && i < j, keep = ok && !(mutual && i > j);
    uint64_t total;
    const uint64_t at = tiles_scan<kPlocThreads / kWave>(B.status[pass & 1], tile, (uint64_t)keep | (uint64_t)merge << 31, total, B.ticket + 3);
    const uint32_t p = (uint32_t)at & 0x7fffffffu;
    if (tile == (m - 1) / kPlocTile && threadIdx.x == 0)
        B.st[pass + 1] = {(uint32_t)total & 0x7fffffffu, node_base + (uint32_t)(total >> 31)};
    if (!keep) return;
    const int l = (int)threadIdx.x + R;
    if (!merge) {
        for (int a = 0; a < 6; ++a) obox[6 * (size_t)p + a] = bx[a][l];
        oid[p] = in.id ? in.id[i] : ~i;
        osize[p] = in.id ? in.size[i] : 1u;
        return;
    }
    const int node = (int)(node_base + (uint32_t)(at >> 31)), lj = j - t0 + 2 * R;
    const uint32_t sz = in.id ? in.size[i] + in.size[j] : 2u;
    child[node] = in.id ? make_int2(in.id[i], in.id[j]) : make_int2(~i, ~j);
    nsize[node] = sz;
    for (int k = 0; k < 3; ++k) {
        const float lo = fminf(bx[k][l], bx[k][lj]), hi = fmaxf(bx[3 + k][l], bx[3 + k][lj]);
        obox[6 * (size_t)p + k] = lo;
        obox[6 * (size_t)p + 3 + k] = hi;
        ibox[6 * (size_t)node + k] = lo;  // the node's box: min / max are exact, so the same
        ibox[6 * (size_t)node + 3 + k] = hi;  // values a refit over its disks would give
    }
    oid[p] = node;
    osize[p] = sz;
}

// The last passes, from at most kPlocTail clusters on, in one block with the
// clusters in LDS (half of the passes of a 1M-point build). Ends with one
// cluster, or when a pass merges nothing (then m > 1 is left in the state).
// st[pass ..] receives the passes' states; *n_pass their number.
constexpr int kPlocTail = 1024;

__global__ __launch_bounds__(kPlocTail) void k_ploc_tail(Clusters in, PassBufs B, uint32_t pass,
                                                         int2 *__restrict__ child, uint32_t *__restrict__ nsize,
                                                         float *__restrict__ ibox, uint32_t *__restrict__ n_pass) {
    __shared__ float bx[6][kPlocTail];
    __shared__ int nn[kPlocTail], id[kPlocTail];
    __shared__ uint32_t sz[kPlocTail], part[kPlocTail / kWave];
    const int t = threadIdx.x;
    const uint32_t lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    int m = (int)B.st[pass].m;
    uint32_t node_base = B.st[pass].base;
    if (m > kPlocTail) return;  // (the host checks m before it launches this)
    if (t < m) {
        for (int a = 0; a < 6; ++a) bx[a][t] = in.box[6 * (size_t)t + a];
        id[t] = in.id ? in.id[t] : ~t;
        sz[t] = in.id ? in.size[t] : 1u;
    }
    __syncthreads();
    while (m > 1) {
        nn[t] = t < m ? ploc_nearest<kPlocTail>(bx, t, max(0, t - kPlocRadius), min(m - 1, t + kPlocRadius)) : -1;
        __syncthreads();
        const int j = nn[t];
        const bool mutual = j >= 0 && nn[j] == t;
        const bool merge = mutual && t < j, keep = t < m && !(mutual && t > j);
        uint32_t in2 = (uint32_t)keep | (uint32_t)merge << 16;  // at most 1024 each
        const uint32_t own = in2;
        for (uint32_t o = 1; o < (uint32_t)kWave; o <<= 1) {
            const uint32_t v = __shfl_up(in2, o, kWave);
            if (lane >= o) in2 += v;
        }
        if (lane == kWave - 1) part[w] = in2;
        float b[6];
        int me = 0;
        uint32_t size = 0;
        int2 ch = make_int2(0, 0);
        if (keep) {
            for (int a = 0; a < 6; ++a) b[a] = bx[a][t];
            me = id[t];
            size = sz[t];
            if (merge) {
                for (int k = 0; k < 3; ++k) {
                    b[k] = fminf(b[k], bx[k][j]);
                    b[3 + k] = fmaxf(b[3 + k], bx[3 + k][j]);
                }
                ch = make_int2(me, id[j]);
                size += sz[j];
            }
        }
        __syncthreads();
        uint32_t before = 0, all = 0;
        for (uint32_t i = 0; i < kPlocTail / kWave; ++i) {
            before += i < w ? part[i] : 0u;
            all += part[i];
        }
        const uint32_t at = before + in2 - own, p = at & 0xffffu;
        if (keep) {
            if (merge) {
                me = (int)(node_base + (at >> 16));
                child[me] = ch;
                nsize[me] = size;
                for (int a = 0; a < 6; ++a) ibox[6 * (size_t)me + a] = b[a];
            }
            for (int a = 0; a < 6; ++a) bx[a][p] = b[a];
            id[p] = me;
            sz[p] = size;
        }
        const int left = (int)(all & 0xffffu);
        node_base += all >> 16;
        ++pass;
        if (t == 0) B.st[pass] = {(uint32_t)left, node_base};
        const bool stuck = left == m;
        m = left;
        __syncthreads();
        if (stuck) break;
    }
    if (t == 0) *n_pass = pass;
}

// Depth-first offsets and depths, one creation pass at a time from the root's
// down (a node's parent is always created in a later pass).
__device__ __forceinline__ void dfs_node(uint32_t node, const int2 *child, const uint32_t *nsize, uint32_t *noff,
                                         uint32_t *ndepth, uint32_t *leaf_pos) {
    const uint32_t o = noff[node], d = ndepth[node];
    const int2 c = child[node];
    const uint32_t sa = c.x < 0 ? 1u : nsize[c.x];
    if (c.x < 0) leaf_pos[~c.x] = o;
    else {
        noff[c.x] = o;
        ndepth[c.x] = d + 1;
    }
    if (c.y < 0) leaf_pos[~c.y] = o + sa;
    else {
        noff[c.y] = o + sa;
        ndepth[c.y] = d + 1;
    }
}

__global__ __launch_bounds__(256) void k_dfs_pass(const int2 *child, const uint32_t *nsize, uint32_t lo, uint32_t hi,
                                                  uint32_t *noff, uint32_t *ndepth, uint32_t *leaf_pos) {
    const uint32_t node = lo + blockIdx.x * 256 + threadIdx.x;
    if (node < hi) dfs_node(node, child, nsize, noff, ndepth, leaf_pos);
}

// The passes from p0 on (each of at most kTopNodes nodes) in one block,
// which starts at the root.
__global__ __launch_bounds__(1024) void k_dfs_top(const PassState *st, uint32_t p0, uint32_t p1, const int2 *child,
                                                  const uint32_t *nsize, uint32_t *noff, uint32_t *ndepth,
                                                  uint32_t *leaf_pos) {
    if (threadIdx.x == 0) {
        noff[st[p1].base - 1] = 0;
        ndepth[st[p1].base - 1] = 1;
    }
    __syncthreads();
    for (uint32_t p = p1; p-- > p0;) {
        for (uint32_t node = st[p].base + threadIdx.x; node < st[p + 1].base; node += 1024)
            dfs_node(node, child, nsize, noff, ndepth, leaf_pos);
        __syncthreads();
    }
}

__global__ void k_dfs_leaves(uint32_t n, const uint32_t *__restrict__ leaf_pos, const uint32_t *__restrict__ sorted_id,
                             uint32_t *__restrict__ perm) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    perm[leaf_pos[i]] = sorted_id[i];
}

// References to leaves and ranges, and the depth of the deepest leaf (a node's depth counts the node and its
// ancestors): a maximum per block of kDfsNodes, as an atomic per wavefront and pass made up most of the passes above.
constexpr uint32_t kDfsNodes = 1024;
__global__ __launch_bounds__(256) void k_dfs_nodes(uint32_t n_int, const uint32_t *__restrict__ leaf_pos,
                                                   const uint32_t *__restrict__ noff, const uint32_t *__restrict__ nsize,
                                                   const uint32_t *__restrict__ ndepth, int2 *__restrict__ child,
                                                   int2 *__restrict__ range, uint32_t *depth) {
    __shared__ uint32_t red[4];
    uint32_t d = 0;
    for (uint32_t k = 0; k < kDfsNodes / 256; ++k) {
        const uint32_t node = blockIdx.x * kDfsNodes + k * 256 + threadIdx.x;
        if (node >= n_int) break;
        int2 c = child[node];
        if (c.x < 0 || c.y < 0) d = max(d, ndepth[node]);
        if (c.x < 0) c.x = ~(int)leaf_pos[~c.x];
        if (c.y < 0) c.y = ~(int)leaf_pos[~c.y];
        child[node] = c;
        range[node] = make_int2((int)noff[node], (int)(noff[node] + nsize[node] - 1));
    }
    for (int o = 32; o > 0; o >>= 1) d = max(d, (uint32_t)__shfl_xor(d, o, kWave));
    if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave] = d;
    __syncthreads();
    if (threadIdx.x == 0) max_to(max(max(red[0], red[1]), max(red[2], red[3])), depth);
}

// --------------------------------------------------------- wide nodes
// Collapse of the binary hierarchy into nodes of up to W children, level by
// level from the root. Which binary nodes become wide nodes is chosen by the
// surface-area cost below (a pass over the binary tree before the collapse);
// the greedy rule it replaced (open the internal child with the largest box
// surface area until the node holds W children) is kept for comparison
// builds. On the 1M-point office: 285 369 -> 232 866 wide nodes, solve
// 37.2 -> 36.6 ms, results bitwise the same. Children get wide indices in
// level order through an
// exclusive scan of the per-node internal-child counts, so the layout is
// deterministic. Wide node: 7W floats -- lo x[W], lo y[W], lo z[W], hi x[W],
// hi y[W], hi z[W], child refs[W] -- padded to 8W floats (128 B for W = 4,
// 256 B for W = 8). An empty slot holds a point box at 1e30, which no slab
// test over a finite segment accepts, and a one-disk leaf reference.
struct WSlot {
    float b[6];
    int ref;
};

__device__ __forceinline__ float half_area(const float *b) {
    const float dx = b[3] - b[0], dy = b[4] - b[1], dz = b[5] - b[2];
    return dx * dy + dy * dz + dz * dx;
}

__device__ __forceinline__ void binary_children(const float4 *__restrict__ bnode, int b, WSlot &c0, WSlot &c1) {
    const float4 *nd = bnode + 4 * (size_t)b;
    const float4 x0 = nd[0], x1 = nd[1], x2 = nd[2], x3 = nd[3];
    c0 = {{x0.x, x0.y, x0.z, x0.w, x1.x, x1.y}, __float_as_int(x3.x)};
    c1 = {{x1.z, x1.w, x2.x, x2.y, x2.z, x2.w}, __float_as_int(x3.y)};
}

// Surface-area cost of the collapse into W-wide nodes, chosen per node
// (the cost-based collapse of Ylitie, Karras and Laine 2017). For a binary
// node n and i = 1..W, C(n, i) is the least expected traversal cost of n's
// subtree when it may take up to i child slots of its wide parent, with A
// the half surface area (a ray's chance of entering a box is proportional to
// it), c_node the cost of one wide node visit (W box tests) and c_disk that of
// one disk test:
//   C1(n) = A(n) c_node + D(n, W)                      n becomes a wide node
//   D(n, j) = min over j_l + j_r = j of C(l, j_l) + C(r, j_r)   n dissolved
//   C(n, 1) = C1(n),  C(n, i) = min(C1(n), D(n, i))     (i >= 2)
//   C(leaf, i) = A(leaf) c_disk |leaf|
// choice[n * W + i - 1] keeps, for i >= 2, the split j_l of D(n, i) in its low
// four bits and whether C(n, i) takes n as one slot in bit 4. Where nodes have no
// creation passes the rows are filled bottom-up by one thread per node whose
// children are both leaves; a thread climbs while it is the last child to
// arrive at the parent (atomic countdown), and stops where the parent does
// not reference the node (the node lies inside a leaf the build collapsed).
constexpr float kSahNode = 1.0f, kSahDisk = 0.4f;  // a node step costs about 2.5 disk tests (4-wide any-hit walk)

__global__ void k_sah_pending(const float4 *__restrict__ bnode, uint32_t ni, uint32_t *pending) {
    const uint32_t n = blockIdx.x * blockDim.x + threadIdx.x;
    if (n >= ni) return;
    const float4 r = bnode[4 * (size_t)n + 3];
    pending[n] = (__float_as_int(r.x) >= 0) + (__float_as_int(r.y) >= 0);
}

// C(n, .) and choice of one node whose children have theirs.
template <int W, typename Cost, typename Choice>
__device__ __forceinline__ void sah_node(const float4 *__restrict__ bnode, int n, Cost *cost, Choice *choice) {
    WSlot c[2];
    binary_children(bnode, n, c[0], c[1]);
    float row[2][W];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int v = -1 - c[s].ref;
        const float leaf = half_area(c[s].b) * kSahDisk * (float)((v & 7) + 1);
#pragma unroll
        for (int i = 0; i < W; ++i) row[s][i] = c[s].ref < 0 ? leaf : cost[(size_t)max(c[s].ref, 0) * W + i];
    }
    float d[W + 1];
    uint32_t split[W + 1];
#pragma unroll
    for (int j = 2; j <= W; ++j) {
        d[j] = INFINITY;
        split[j] = 1;
#pragma unroll
        for (int jl = 1; jl < j; ++jl) {
            const float v = row[0][jl - 1] + row[1][j - jl - 1];
            if (v < d[j]) {
                d[j] = v;
                split[j] = (uint32_t)jl;
            }
        }
    }
    float lo[3], hi[3];
    for (int a = 0; a < 3; ++a) {
        lo[a] = fminf(c[0].b[a], c[1].b[a]);
        hi[a] = fmaxf(c[0].b[3 + a], c[1].b[3 + a]);
    }
    const float box[6] = {lo[0], lo[1], lo[2], hi[0], hi[1], hi[2]};
    const float c1 = half_area(box) * kSahNode + d[W];
    Cost *out = cost + (size_t)n * W;
    Choice *ch = choice + (size_t)n * W;
    out[0] = c1;
    ch[0] = 0;
#pragma unroll
    for (int i = 2; i <= W; ++i) {
        const bool single = c1 <= d[i];
        out[i - 1] = single ? c1 : d[i];
        ch[i - 1] = (uint8_t)(split[i] | (single ? 16 : 0));
    }
}

// Trees whose nodes are numbered by creation pass (the clustering builder): a
// node's children were created in earlier passes, so the rows are filled pass
// by pass, without the climb's atomics and device-scope fences (1M points:
// 2.76 -> 0.14 ms). Nodes inside a collapsed leaf get rows that nobody reads.
template <int W>
__global__ __launch_bounds__(256) void k_sah_pass(const float4 *__restrict__ bnode, uint32_t lo, uint32_t hi,
                                                  float *cost, uint8_t *choice) {
    const uint32_t n = lo + blockIdx.x * 256 + threadIdx.x;
    if (n < hi) sah_node<W>(bnode, (int)n, cost, choice);
}

// The passes from p0 on, each of a few thousand nodes at most, in one block.
template <int W>
__global__ __launch_bounds__(1024) void k_sah_top(const float4 *__restrict__ bnode, const PassState *st, uint32_t p0,
                                                  uint32_t p1, float *cost, uint8_t *choice) {
    for (uint32_t p = p0; p < p1; ++p) {
        for (uint32_t n = st[p].base + threadIdx.x; n < st[p + 1].base; n += 1024)
            sah_node<W>(bnode, (int)n, cost, choice);
        __syncthreads();
    }
}

// Other trees: bottom-up by one thread per node whose children are both leaves.
template <int W>
__global__ void k_sah_rows(const float4 *__restrict__ bnode, const int *__restrict__ parent, uint32_t ni,
                           uint32_t *pending, float *cost, uint8_t *choice) {
    const uint32_t i0 = blockIdx.x * blockDim.x + threadIdx.x;
    if (i0 >= ni) return;
    int n = (int)i0;
    {
        const float4 r = bnode[4 * (size_t)n + 3];
        if (__float_as_int(r.x) >= 0 || __float_as_int(r.y) >= 0) return;
    }
    for (;;) {
        sah_node<W>(bnode, n, (volatile float *)cost, (volatile uint8_t *)choice);
        __threadfence();
        const int p = parent[n];
        if (p < 0) return;
        const float4 pr = bnode[4 * (size_t)p + 3];
        if (__float_as_int(pr.x) != n && __float_as_int(pr.y) != n) return;  // inside a collapsed leaf
        if (atomicSub(&pending[p], 1u) != 1u) return;  // the other child is not done yet
        __threadfence();
        n = p;
    }
}

// The children of the wide node standing for binary node b, by the choices
// above: b is dissolved into W slots; a child given j slots takes one if it
// is a leaf, if j = 1 or if its row says so, else it is dissolved in turn.
template <int W>
__device__ int wide_children_sah(const float4 *__restrict__ bnode, const uint8_t *__restrict__ choice, int b,
                                 WSlot *sl) {
    int st_n[W], st_j[W];
    int sp = 0, cnt = 0;
    st_n[sp] = b;
    st_j[sp++] = W;
    while (sp > 0) {
        --sp;
        const int n = st_n[sp], j = st_j[sp];
        WSlot c[2];
        binary_children(bnode, n, c[0], c[1]);
        const int jl = choice[(size_t)n * W + j - 1] & 15;
        const int js[2] = {jl, j - jl};
        for (int s = 0; s < 2; ++s) {
            if (c[s].ref < 0 || js[s] == 1 || (choice[(size_t)c[s].ref * W + js[s] - 1] & 16)) {
                sl[cnt++] = c[s];
            } else {
                st_n[sp] = c[s].ref;
                st_j[sp++] = js[s];
            }
        }
    }
    return cnt;
}

template <int W>
__device__ int wide_children(const float4 *__restrict__ bnode, int b, WSlot *sl) {
    binary_children(bnode, b, sl[0], sl[1]);
    int cnt = 2;
    while (cnt < W) {
        int best = -1;
        float ba = -1.f;
        for (int j = 0; j < cnt; ++j)
            if (sl[j].ref >= 0) {
                const float ar = half_area(sl[j].b);
                if (ar > ba) {
                    ba = ar;
                    best = j;
                }
            }
        if (best < 0) break;
        WSlot c0, c1;
        binary_children(bnode, sl[best].ref, c0, c1);
        sl[best] = c0;
        sl[cnt++] = c1;
    }
    return cnt;
}

// One level of the collapse in one launch: every block takes tiles of 256
// frontier nodes by ticket, finds their wide children once, and writes the
// nodes and the next frontier at its scanned places. A launch after the last
// level finds an empty frontier and ends, and so does one after a failed level:
// one thread looks at the fail word, which another block may be setting, so
// that a block takes one decision. Five launches and a host round trip
// per level before: 14 levels of a 1M-point build 1.0 -> 0.3 ms.
template <int W>
__global__ __launch_bounds__(256) void k_wide_level(const float4 *__restrict__ bnode, const uint8_t *__restrict__ choice,
                                                    const int *__restrict__ frontier, PassBufs B, uint32_t level,
                                                    int *__restrict__ next, float *__restrict__ wnode) {
    __shared__ uint32_t tile_s;
    __shared__ PassState now;
    pass_clear(B, level);
    if (threadIdx.x == 0) {
        now = B.st[level];
        if (__hip_atomic_load(&B.ticket[3], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) now.m = 0u;
    }
    __syncthreads();
    const uint32_t nf = now.m, base_cur = now.base, base_next = base_cur + nf;
    if (nf == 0) {
        if (blockIdx.x == 0 && threadIdx.x == 0) B.st[level + 1] = {0u, base_cur};
        return;
    }
    for (;;) {
        if (threadIdx.x == 0) tile_s = atomicAdd(&B.ticket[level & 1], 1u);
        __syncthreads();
        const uint32_t tile = tile_s;
        __syncthreads();
        if ((uint64_t)tile * 256 >= nf) return;
        const uint32_t i = tile * 256 + threadIdx.x;
        WSlot sl[W];
        int c = 0;
        uint32_t k = 0;
        if (i < nf) {
            c = choice ? wide_children_sah<W>(bnode, choice, frontier[i], sl) : wide_children<W>(bnode, frontier[i], sl);
            for (int j = 0; j < c; ++j) k += sl[j].ref >= 0;
        }
        uint64_t total;
        k = (uint32_t)tiles_scan<4>(B.status[level & 1], tile, k, total, B.ticket + 3);
        if (tile == (nf - 1) / 256 && threadIdx.x == 0) B.st[level + 1] = {(uint32_t)total, base_next};
        float *o = wnode + (size_t)(base_cur + i) * 8 * W;
        for (int j = 0; j < (i < nf ? W : 0); ++j) {
            int ref = leaf_ref(0, 1);
            float bx[6] = {1e30f, 1e30f, 1e30f, 1e30f, 1e30f, 1e30f};
            if (j < c) {
                for (int a = 0; a < 6; ++a) bx[a] = sl[j].b[a];
                ref = sl[j].ref;
                if (ref >= 0) {
                    next[k] = ref;
                    ref = (int)(base_next + k);
                    ++k;
                }
            }
            for (int a = 0; a < 6; ++a) o[a * W + j] = bx[a];
            o[6 * W + j] = __int_as_float(ref);
            o[7 * W + j] = 0.f;
        }
    }
}

// Compact copy of the wide nodes for the any-hit walks (layout and error
// bound at wide_hits): per axis, the grid step is the power of two 2^e with
// 2^e >= the node's extent / 2040 and >= 2^-19 times its largest coordinate
// (so the origin's rounding stays below 1/16 step); the origin is the largest
// float at or below lo - 2^e; lower planes round down, upper planes up (in
// FP64, where these differences and quotients are exact). Coordinates then
// lie in 1..2042. Empty slots get lo = 2047, hi = 0 on every axis, a box no
// segment enters. The node is written in eight copies, one per direction
// octant (copy o: bit a set for a negative direction component on axis a),
// the near plane rows first: lo rows on positive axes, hi rows on negative
// ones.
template <int W>
__global__ void k_wide_quant(const float *__restrict__ wnode, uint32_t n_nodes, float4 *__restrict__ qnode,
                             int *__restrict__ qref) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_nodes) return;
    const float *o = wnode + (size_t)i * 8 * W;
    float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
    for (int j = 0; j < W; ++j) {
        if (!(o[j] < 1e30f)) continue;  // empty slot
        for (int a = 0; a < 3; ++a) {
            lo[a] = fminf(lo[a], o[a * W + j]);
            hi[a] = fmaxf(hi[a], o[(3 + a) * W + j]);
        }
    }
    float org[3];
    double inv_step[3];  // reciprocals of powers of two: quotients by them are exact products
    uint32_t eb = 0;
    for (int a = 0; a < 3; ++a) {
        if (!(lo[a] <= hi[a])) lo[a] = hi[a] = 0.f;  // no child (never for a built node)
        const double ext = (double)hi[a] - (double)lo[a];
        const double m = fmax(fmax(fabs((double)lo[a]), fabs((double)hi[a])), 1.0);
        const double need = fmax(ext / 2040.0, m * 0x1p-19);
        int e;
        frexp(need, &e);  // need < 2^e
        e = max(e, -100);
        inv_step[a] = ldexp(1.0, -e);
        const double od = (double)lo[a] - ldexp(1.0, e);
        float of = (float)od;
        if ((double)of > od) of = nextafterf(of, -INFINITY);
        org[a] = of;
        eb |= ((uint32_t)e & 0xffu) << (8 * a);
    }
    // the six rows, two FP16 coordinates per word; the copies differ in their order only
    uint32_t row[6][W / 2];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int j = 0; j < W; ++j) {
            double gl = 2047.0, gh = 0.0;
            if (o[j] < 1e30f) {
                gl = floor(((double)o[a * W + j] - (double)org[a]) * inv_step[a]);
                gh = ceil(((double)o[(3 + a) * W + j] - (double)org[a]) * inv_step[a]);
                gl = fmin(fmax(gl, 0.0), 2047.0);
                gh = fmin(fmax(gh, 0.0), 2047.0);
            }
            const uint32_t l = __half_as_ushort((__half)(_Float16)gl), h = __half_as_ushort((__half)(_Float16)gh);
            if (j % 2 == 0) {
                row[a][j / 2] = l;
                row[3 + a][j / 2] = h;
            } else {
                row[a][j / 2] |= l << 16;
                row[3 + a][j / 2] |= h << 16;
            }
        }
#pragma unroll
    for (int k = 0; k < W / 4; ++k)
        *(float4 *)(qref + (size_t)i * W + 4 * k) = *(const float4 *)(o + 6 * W + 4 * k);
#pragma unroll
    for (uint32_t oc = 0; oc < 8u; ++oc) {
        uint32_t w[4 + 3 * W];
        w[0] = __float_as_uint(org[0]);
        w[1] = __float_as_uint(org[1]);
        w[2] = __float_as_uint(org[2]);
        w[3] = eb;
#pragma unroll
        for (int a = 0; a < 3; ++a)
#pragma unroll
            for (int k = 0; k < W / 2; ++k) {  // copy for a negative direction component: hi planes are near
                const bool neg = (oc >> a) & 1u;
                w[4 + a * (W / 2) + k] = row[neg ? 3 + a : a][k];
                w[4 + (3 + a) * (W / 2) + k] = row[neg ? a : 3 + a][k];
            }
        uint4 *q = (uint4 *)((char *)qnode + ((size_t)oc * n_nodes + i) * (16 + 12 * W));
#pragma unroll
        for (int k = 0; k < 1 + 3 * W / 4; ++k) q[k] = make_uint4(w[4 * k], w[4 * k + 1], w[4 * k + 2], w[4 * k + 3]);
    }
}

constexpr uint32_t kMaxLevels = 128;  // of the wide collapse

SceneLayout scene_layout(uint32_t n, uint32_t width, uint32_t builder, bool dps) {
    Bump b;
    SceneLayout L;
    uint32_t ni = n > 1 ? n - 1 : 1;
    uint32_t blk = cdiv(n, 256);
    L.pos_id = b.take(sizeof(float4) * n);
    L.nrm_id = b.take(sizeof(float4) * n);
    L.disk = b.take(sizeof(float4) * 2 * n);
    L.node = b.take(sizeof(float4) * 4 * (size_t)ni);
    L.stat = b.take(sizeof(uint32_t) * 8);
    L.bounds = b.take(sizeof(float) * 8);
    L.dps_stat = b.take(sizeof(uint32_t) * 2);
    L.ticket = b.take(sizeof(uint32_t) * 4);  // stat, bounds, dps_stat, ticket: cleared together
    if (width > 2) L.level_st = b.take(sizeof(PassState) * (kMaxLevels + 8));  // read back with the ticket's fail word
    L.blk_bounds = b.take(sizeof(float) * 6 * blk);
    L.code0 = b.take(sizeof(uint64_t) * n);
    L.code1 = b.take(sizeof(uint64_t) * n);
    L.idx0 = b.take(sizeof(uint32_t) * n);
    L.idx1 = b.take(sizeof(uint32_t) * n);
    L.hist = b.take(sizeof(uint32_t) * radix_hist_words(n));
    L.scan_blk = b.take(sizeof(uint32_t) * scan_blk_words(radix_hist_words(n)));
    L.child = b.take(sizeof(int2) * ni);
    L.range = b.take(sizeof(int2) * ni);
    L.dbox = b.take(sizeof(float) * 6 * n);
    L.ibox = b.take(sizeof(float) * 6 * ni);
    L.flags = b.take(sizeof(uint32_t) * ni);
    for (int k = 0; k < 2; ++k) L.tile_status[k] = b.take(sizeof(uint64_t) * cdiv(n, 256));
    L.width = width;
    L.n_internal = ni;
    L.builder = builder;
    if (builder == kBuildPloc) {
        for (int k = 0; k < 2; ++k) {
            L.cbox[k] = b.take(sizeof(float) * 6 * (size_t)n);
            L.cid[k] = b.take(sizeof(int) * n);
            L.csz[k] = b.take(sizeof(uint32_t) * n);
        }
        L.nsize = b.take(sizeof(uint32_t) * ni);
        L.noff = b.take(sizeof(uint32_t) * ni);
        L.leaf_pos = b.take(sizeof(uint32_t) * n);
        L.perm2 = b.take(sizeof(uint32_t) * n);
        L.pass_st = b.take(sizeof(PassState) * ((size_t)n + 8));  // every pass merges a pair
    } else {  // the radix tree is climbed from its leaves
        L.parent_int = b.take(sizeof(int) * ni);
        L.parent_leaf = b.take(sizeof(int) * n);
        if (width > 2) L.sah_pending = b.take(sizeof(uint32_t) * ni);
    }
    if (width > 2) {  // every wide node stands for a distinct binary internal node
        L.wnode = b.take(sizeof(float) * 8 * width * (size_t)ni);
        L.qnode = b.take((16 + 12 * (size_t)width) * ni * 8);  // one copy per octant
        L.qref = b.take(sizeof(int) * width * (size_t)ni);
        L.front0 = b.take(sizeof(int) * ni);
        L.front1 = b.take(sizeof(int) * ni);
        L.sah_cost = b.take(sizeof(float) * width * (size_t)ni);
        L.sah_choice = b.take((size_t)width * ni);
    }
    if (dps) {  // point sets; their sort reuses the build's code / idx / hist buffers
        L.dps_pt = b.take(sizeof(float4) * 2 * (size_t)n);
        L.dps_off = b.take(sizeof(uint32_t) * ((size_t)n + 1));
        L.dps_of = b.take(sizeof(uint32_t) * n);
        L.dps_flag = b.take(sizeof(uint32_t) * n);
        L.dps_blk = b.take(sizeof(uint32_t) * scan_blk_words(n));
        L.dps_recv = b.take(sizeof(float4) * n);
    }
    L.total = b.off;
    return L;
}

static PassBufs pass_bufs(const SceneLayout &L, char *ws, uint32_t n, size_t st) {
    return {(PassState *)(ws + st),
            {(uint64_t *)(ws + L.tile_status[0]), (uint64_t *)(ws + L.tile_status[1])},
            cdiv(n, 256),
            (uint32_t *)(ws + L.ticket)};
}

// n_st: states to clear, the first included (a failed level may leave the next one's unwritten)
__global__ __launch_bounds__(256) void k_pass_init(PassBufs B, PassState first, uint32_t n_st, int *front, int root,
                                                   uint32_t *depth) {
    const uint32_t t = blockIdx.x * 256 + threadIdx.x;
    for (uint32_t i = t; i < B.n_status; i += gridDim.x * 256) B.status[0][i] = B.status[1][i] = 0ull;
    for (uint32_t i = t + 1; i < n_st; i += gridDim.x * 256) B.st[i] = {0u, 0u};
    if (t != 0) return;
    B.ticket[0] = B.ticket[1] = 0u;
    B.st[0] = first;
    if (front) front[0] = root;
    if (depth) *depth = 0u;
}

static hipError_t read_back(void *to, const void *from, size_t bytes, hipStream_t s) {
    const hipError_t e = hipMemcpyAsync(to, from, bytes, hipMemcpyDeviceToHost, s);
    return e == hipSuccess ? hipStreamSynchronize(s) : e;
}

// Clustering build over the Morton-ordered disk boxes in dbox (n >= 2):
// fills the child arrays, renumbers the disks depth-first (perm2, range) and
// returns the root and the passes' states on the device and the host. The host
// reads the cluster count every few passes (a launch sized for an older
// count only starts blocks that end at once), then hands the tail over.
constexpr uint32_t kPlocBatch = 4;      // passes between two looks at the count
constexpr uint32_t kTopNodes = 1024;    // passes of at most so many nodes share one block's launch

// First of the last passes that one block goes through (later passes are smaller
// or of the same order; at least the root's is among them).
static uint32_t top_pass(const std::vector<PassState> &st) {
    uint32_t p = (uint32_t)st.size() - 1;
    while (p > 0 && st[p].base - st[p - 1].base <= kTopNodes) --p;
    return std::min(p, (uint32_t)st.size() - 2);
}

hipError_t build_ploc(const SceneLayout &L, char *ws, uint32_t n, const uint32_t *sorted_id, hipStream_t s,
                      int *root, std::vector<PassState> &st) {
    auto P = [&](size_t off) { return ws + off; };
    float *cbox[2] = {(float *)P(L.cbox[0]), (float *)P(L.cbox[1])};
    int *cid[2] = {(int *)P(L.cid[0]), (int *)P(L.cid[1])};
    uint32_t *csz[2] = {(uint32_t *)P(L.csz[0]), (uint32_t *)P(L.csz[1])};
    uint32_t *nsize = (uint32_t *)P(L.nsize), *noff = (uint32_t *)P(L.noff), *leaf_pos = (uint32_t *)P(L.leaf_pos);
    uint32_t *ndepth = (uint32_t *)P(L.flags), *depth = (uint32_t *)P(L.stat) + 3;
    int2 *child = (int2 *)P(L.child), *range = (int2 *)P(L.range);
    float *ibox = (float *)P(L.ibox);
    const PassBufs B = pass_bufs(L, ws, n, L.pass_st);
    hipLaunchKernelGGL(k_pass_init, dim3(std::min<uint32_t>(cdiv(B.n_status, 256), 256)), dim3(256), 0, s, B,
                       PassState{n, 0u}, 1u, (int *)nullptr, 0, depth);
    auto clusters = [&](uint32_t pass) {
        if (pass == 0) return Clusters{(const float *)P(L.dbox), nullptr, nullptr};
        return Clusters{cbox[pass & 1], cid[pass & 1], csz[pass & 1]};
    };
    st.assign(1, PassState{n, 0u});
    uint32_t pass = 0;
    while (st.back().m > (uint32_t)kPlocTail) {
        const uint32_t m = st.back().m;
        for (uint32_t k = 0; k < kPlocBatch; ++k, ++pass)
            hipLaunchKernelGGL(k_ploc_pass, dim3(cdiv(m, kPlocTile)), dim3(kPlocThreads), 0, s, clusters(pass), cbox[(pass + 1) & 1],
                               cid[(pass + 1) & 1], csz[(pass + 1) & 1], B, pass, child, nsize, ibox);
        st.resize(pass + 1);
        const hipError_t e = read_back(&st[pass + 1 - kPlocBatch], B.st + pass + 1 - kPlocBatch,
                                       sizeof(PassState) * kPlocBatch, s);
        if (e != hipSuccess) return e;
        if (st[pass].m >= m || st[pass].m == 0 || st[pass].base + st[pass].m != n) return hipErrorUnknown;
    }
    hipLaunchKernelGGL(k_ploc_tail, dim3(1), dim3(kPlocTail), 0, s, clusters(pass), B, pass, child, nsize, ibox,
                       B.ticket + 2);
    uint32_t end[2] = {0, 0};  // number of passes, fail word
    hipError_t e = read_back(end, B.ticket + 2, sizeof end, s);
    if (e != hipSuccess) return e;
    const uint32_t last = end[0];
    if (end[1] || last < pass || last > n) return hipErrorUnknown;
    st.resize((size_t)last + 1);
    if (last > pass) e = read_back(&st[pass + 1], B.st + pass + 1, sizeof(PassState) * (last - pass), s);
    if (e != hipSuccess) return e;
    if (st[last].m != 1 || st[last].base != n - 1) return hipErrorUnknown;  // a pass merged nothing
    *root = (int)(n - 2);
    const uint32_t p0 = top_pass(st);
    hipLaunchKernelGGL(k_dfs_top, dim3(1), dim3(1024), 0, s, B.st, p0, last, child, nsize, noff, ndepth, leaf_pos);
    for (uint32_t p = p0; p-- > 0;)
        hipLaunchKernelGGL(k_dfs_pass, dim3(cdiv(st[p + 1].base - st[p].base, 256)), dim3(256), 0, s, child, nsize,
                           st[p].base, st[p + 1].base, noff, ndepth, leaf_pos);
    hipLaunchKernelGGL(k_dfs_leaves, dim3(cdiv(n, 256)), dim3(256), 0, s, n, leaf_pos, sorted_id,
                       (uint32_t *)P(L.perm2));
    hipLaunchKernelGGL(k_dfs_nodes, dim3(cdiv(n - 1, kDfsNodes)), dim3(256), 0, s, n - 1, leaf_pos, noff, nsize, ndepth,
                       child, range, depth);
    return hipGetLastError();
}

// Level-by-level collapse, one launch per level; the host looks at the frontier
// every few levels. Host outputs: the number of wide levels and of wide nodes.
constexpr uint32_t kLevelBatch = 8;

template <int W>
hipError_t build_wide_w(const SceneLayout &L, char *ws, hipStream_t s, int broot, const std::vector<PassState> &passes,
                        uint32_t *levels, uint32_t *nodes) {
    const float4 *bnode = (const float4 *)(ws + L.node);
    int *fr[2] = {(int *)(ws + L.front0), (int *)(ws + L.front1)};
    float *wnode = (float *)(ws + L.wnode);
    const uint32_t ni = L.n_internal;
    const uint8_t *choice = nullptr;
    if (kSahCollapse) {
        uint32_t *pending = (uint32_t *)(ws + L.sah_pending);
        float *cost = (float *)(ws + L.sah_cost);
        uint8_t *ch = (uint8_t *)(ws + L.sah_choice);
        if (!passes.empty()) {
            const uint32_t p0 = top_pass(passes), p1 = (uint32_t)passes.size() - 1;
            for (uint32_t p = 0; p < p0; ++p)
                hipLaunchKernelGGL(k_sah_pass<W>, dim3(cdiv(passes[p + 1].base - passes[p].base, 256)), dim3(256), 0, s,
                                   bnode, passes[p].base, passes[p + 1].base, cost, ch);
            hipLaunchKernelGGL(k_sah_top<W>, dim3(1), dim3(1024), 0, s, bnode, (const PassState *)(ws + L.pass_st), p0,
                               p1, cost, ch);
        } else {
            hipLaunchKernelGGL(k_sah_pending, dim3(cdiv(ni, 256)), dim3(256), 0, s, bnode, ni, pending);
            hipLaunchKernelGGL(k_sah_rows<W>, dim3(cdiv(ni, 256)), dim3(256), 0, s, bnode,
                               (const int *)(ws + L.parent_int), ni, pending, cost, ch);
        }
        choice = ch;
    }
    const PassBufs B = pass_bufs(L, ws, ni, L.level_st);
    hipLaunchKernelGGL(k_pass_init, dim3(std::min<uint32_t>(cdiv(B.n_status, 256), 256)), dim3(256), 0, s, B,
                       PassState{1u, 0u}, kMaxLevels + 8, fr[0], broot, (uint32_t *)nullptr);
    uint32_t lv = 0;
    uint64_t bound = 1;  // of the frontier
    struct {
        uint32_t ticket[64];  // (256 bytes: the layout's alignment)
        PassState st[kMaxLevels + 8];
    } back;
    const PassState *st = back.st;
    PassState last{1u, 0u};
    while (last.m > 0) {
        // every wide node stands for a distinct binary internal node
        if ((uint64_t)last.base + last.m > ni || lv >= kMaxLevels) return hipErrorUnknown;
        for (uint32_t k = 0; k < kLevelBatch; ++k, ++lv) {
            const uint32_t g = (uint32_t)std::min<uint64_t>(cdiv(bound, 256), 1024);
            hipLaunchKernelGGL(k_wide_level<W>, dim3(g), dim3(256), 0, s, bnode, choice, fr[lv & 1], B, lv,
                               fr[(lv + 1) & 1], wnode);
            bound = std::min<uint64_t>(bound * W, ni);
        }
        const hipError_t e = read_back(&back, ws + L.ticket, sizeof back, s);
        if (e != hipSuccess) return e;
        if (back.ticket[3]) return hipErrorUnknown;  // a look-back gave up
        last = st[lv];
    }
    uint32_t n_lv = 0;
    while (st[n_lv].m > 0) ++n_lv;
    *levels = n_lv;
    *nodes = st[n_lv].base;
    hipLaunchKernelGGL(k_wide_quant<W>, dim3(cdiv(*nodes, 256)), dim3(256), 0, s, wnode, *nodes,
                       (float4 *)(ws + L.qnode), (int *)(ws + L.qref));
    return hipGetLastError();
}

static hipError_t build_wide(const SceneLayout &L, char *ws, hipStream_t s, int broot,
                             const std::vector<PassState> &passes, uint32_t *levels, uint32_t *nodes) {
    return L.width == 4 ? build_wide_w<4>(L, ws, s, broot, passes, levels, nodes)
                        : build_wide_w<8>(L, ws, s, broot, passes, levels, nodes);
}

hipError_t build_scene(const float *pos, const float *nrm, const uint16_t *mat, const uint32_t *surf, uint32_t n,
                       float r, uint32_t leaf, char *ws, const SceneLayout &L, hipStream_t s, uint32_t *wide_levels,
                       uint32_t *wide_nodes, int *root) {
    auto P = [&](size_t off) { return ws + off; };
    float4 *pos_id = (float4 *)P(L.pos_id), *nrm_id = (float4 *)P(L.nrm_id);
    uint32_t *stat = (uint32_t *)P(L.stat);
    float *bounds = (float *)P(L.bounds), *blkb = (float *)P(L.blk_bounds);
    uint64_t *c0 = (uint64_t *)P(L.code0), *c1 = (uint64_t *)P(L.code1);
    uint32_t *i0 = (uint32_t *)P(L.idx0), *i1 = (uint32_t *)P(L.idx1);
    uint32_t *hist = (uint32_t *)P(L.hist);
    uint32_t blk = cdiv(n, 256);
    fill_u32(stat, 0, (L.ticket - L.stat) / 4 + 4, s);
    const uint32_t iblk = cdiv(n, kIngest);
    hipLaunchKernelGGL(k_ingest, dim3(iblk), dim3(256), 0, s, pos, nrm, mat, surf, n, pos_id, nrm_id, blkb, stat);
    hipLaunchKernelGGL(k_bounds, dim3(1), dim3(256), 0, s, blkb, iblk, bounds);
    hipLaunchKernelGGL(k_morton, dim3(blk), dim3(256), 0, s, pos_id, n, bounds, c0, i0);
    const bool in_tmp = radix_sort_u64(c0, i0, c1, i1, n, 0, 64, hist, (uint32_t *)P(L.scan_blk), s);
    if (in_tmp) {
        std::swap(c0, c1);
        std::swap(i0, i1);
    }
    float *dbox = (float *)P(L.dbox);
    // (the clustering builder orders the disks again; their boxes are all it needs here)
    const bool again = n > 1 && L.builder == kBuildPloc;
    hipLaunchKernelGGL(k_gather, dim3(blk), dim3(256), 0, s, pos_id, nrm_id, i0, n, r,
                       again ? (float4 *)nullptr : (float4 *)P(L.disk), dbox);
    int broot = 0;
    std::vector<PassState> passes;  // of the clustering builder
    if (n > 1) {
        int2 *child = (int2 *)P(L.child), *range = (int2 *)P(L.range);
        int *pint = (int *)P(L.parent_int), *pleaf = (int *)P(L.parent_leaf);
        if (L.builder == kBuildPloc) {
            hipError_t e = build_ploc(L, ws, n, i0, s, &broot, passes);
            if (e != hipSuccess) return e;
            // disks and their boxes again, now in depth-first order
            hipLaunchKernelGGL(k_gather, dim3(blk), dim3(256), 0, s, pos_id, nrm_id, (const uint32_t *)P(L.perm2), n, r,
                               (float4 *)P(L.disk), dbox);
        } else {
            hipLaunchKernelGGL(k_karras, dim3(cdiv(n - 1, 256)), dim3(256), 0, s, c0, (int)n, child, range, pint,
                               pleaf);
        }
        if (L.builder == kBuildPloc) {
            hipLaunchKernelGGL(k_node_records, dim3(cdiv(n - 1, 256)), dim3(256), 0, s, (int)(n - 1), (int)leaf,
                               child, range, dbox, (const float *)P(L.ibox), (float4 *)P(L.node));
        } else {
            fill_u32((uint32_t *)P(L.flags), 0, n - 1, s);
            hipLaunchKernelGGL(k_refit, dim3(blk), dim3(256), 0, s, (int)n, (int)leaf, child, range, pint, pleaf,
                               dbox, (float *)P(L.ibox), (uint32_t *)P(L.flags), (float4 *)P(L.node));
        }
        if (L.builder != kBuildPloc)
            hipLaunchKernelGGL(k_depth, dim3(blk), dim3(256), 0, s, (int)n, pint, pleaf, stat + 3);
    }
    *root = broot;
    *wide_levels = *wide_nodes = 0;
    if (L.width > 2 && n > leaf) {
        hipError_t e = build_wide(L, ws, s, broot, passes, wide_levels, wide_nodes);
        if (e != hipSuccess) return e;
    }
    return hipGetLastError();
}

}  // namespace pcrt
