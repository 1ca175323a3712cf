// The part of HIP that the hierarchy build's kernels use, on the CPU: blocks run one after another, a block's threads
// as fibers that switch at barriers and wavefront operations. For tests of control flow, not of speed.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <vector>
using std::isfinite;
using std::max;
using std::min;

#define __global__
#define __device__
#define __host__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __restrict__
// variables of LDS lie in one section, so that every block can find zeros there (a real one finds anything)
#define __shared__ static __attribute__((section("lds")))

struct float4 { float x, y, z, w; } __attribute__((aligned(16)));
struct uint4 { uint32_t x, y, z, w; } __attribute__((aligned(16)));
struct int4 { int x, y, z, w; } __attribute__((aligned(16)));
struct int2 { int x, y; };
inline float4 make_float4(float a, float b, float c, float d) { return {a, b, c, d}; }
inline uint4 make_uint4(uint32_t a, uint32_t b, uint32_t c, uint32_t d) { return {a, b, c, d}; }
inline int2 make_int2(int a, int b) { return {a, b}; }
struct dim3 {
    uint32_t x, y, z;
    dim3(uint32_t a = 1, uint32_t b = 1, uint32_t c = 1) : x(a), y(b), z(c) {}
};

typedef int hipError_t;
typedef void *hipStream_t;
enum { hipSuccess = 0, hipErrorUnknown = 999 };
enum { hipMemcpyDeviceToHost = 2 };
inline hipError_t hipMemcpyAsync(void *a, const void *b, size_t n, int, hipStream_t) {
    memcpy(a, b, n);
    return 0;
}
inline hipError_t hipStreamSynchronize(hipStream_t) { return 0; }
inline hipError_t hipGetLastError() { return 0; }

namespace emu {
struct Idx { uint32_t x, y, z; };
extern Idx tid, bid, bdim, gdim;
extern uint64_t wave_buf[16][64];
extern bool backwards;                                               // threads of a block in falling order
extern std::function<void(const char *, uint32_t, uint32_t)> start;  // before a thread first runs: kernel, block, thread
void block_sync();
void wave_sync();
void launch(dim3 g, dim3 b, const std::function<void()> &f, const char *name);
}  // namespace emu
#define threadIdx emu::tid
#define blockIdx emu::bid
#define blockDim emu::bdim
#define gridDim emu::gdim
#define hipLaunchKernelGGL(f, g, b, s, st, ...) emu::launch(g, b, [&] { f(__VA_ARGS__); }, #f)

inline void __syncthreads() { emu::block_sync(); }
inline void __threadfence() {}
template <class T>
T emu_shfl(T v, uint32_t from) {
    const uint32_t w = emu::tid.x / 64, l = emu::tid.x % 64;
    uint64_t u = 0;
    memcpy(&u, &v, sizeof v);
    emu::wave_buf[w][l] = u;
    emu::wave_sync();
    u = emu::wave_buf[w][from];
    emu::wave_sync();
    T r;
    memcpy(&r, &u, sizeof r);
    return r;
}
template <class T>
T __shfl_up(T v, int o, int) {
    const uint32_t l = emu::tid.x % 64;
    return emu_shfl(v, (int)l - o < 0 ? l : l - o);
}
template <class T>
T __shfl_xor(T v, int o, int) { return emu_shfl(v, emu::tid.x % 64 ^ o); }
inline uint64_t __ballot(int p) {
    const uint32_t w = emu::tid.x / 64, l = emu::tid.x % 64, n = std::min(64u, emu::bdim.x - w * 64);
    emu::wave_buf[w][l] = p != 0;
    emu::wave_sync();
    uint64_t m = 0;
    for (uint32_t i = 0; i < n; ++i) m |= emu::wave_buf[w][i] << i;
    emu::wave_sync();
    return m;
}
inline int __popcll(uint64_t v) { return __builtin_popcountll(v); }
inline int __ffsll(unsigned long long v) { return __builtin_ffsll(v); }
inline int __clz(uint32_t v) { return v ? __builtin_clz(v) : 32; }
inline int __clzll(uint64_t v) { return v ? __builtin_clzll(v) : 64; }
template <class T, class U> T atomicAdd(T *p, U v) { T o = *p; *p += v; return o; }
template <class T, class U> T atomicSub(T *p, U v) { T o = *p; *p -= v; return o; }
template <class T, class U> T atomicMax(T *p, U v) { T o = *p; if (v > o) *p = v; return o; }
template <class T, class U> T atomicMin(T *p, U v) { T o = *p; if (v < o) *p = v; return o; }
template <class T, class U> T atomicOr(T *p, U v) { T o = *p; *p |= v; return o; }
#define __HIP_MEMORY_SCOPE_AGENT 3
#define __hip_atomic_load(p, o, s) (*(p))
#define __hip_atomic_store(p, v, o, s) (void)(*(p) = (v))
#define __hip_atomic_fetch_add(p, v, o, s) atomicAdd(p, v)
inline uint32_t __float_as_uint(float f) { uint32_t u; memcpy(&u, &f, 4); return u; }
inline int __float_as_int(float f) { int u; memcpy(&u, &f, 4); return u; }
inline float __uint_as_float(uint32_t u) { float f; memcpy(&f, &u, 4); return f; }
inline float __int_as_float(int u) { float f; memcpy(&f, &u, 4); return f; }
inline void sincospif(float, float *, float *) {}
inline uint32_t emu_bits_below(uint32_t m, int l, uint32_t b) {
    return b + (l <= 0 ? 0 : __builtin_popcount(l >= 32 ? m : m & ((1u << l) - 1)));
}
#define __builtin_amdgcn_mbcnt_lo(m, b) emu_bits_below(m, (int)(emu::tid.x % 64), b)
#define __builtin_amdgcn_mbcnt_hi(m, b) emu_bits_below(m, (int)(emu::tid.x % 64) - 32, b)
#define __builtin_amdgcn_fence(...) ((void)0)
#define __builtin_amdgcn_wave_barrier() emu::wave_sync()
#define __builtin_amdgcn_readfirstlane(x) (x)
