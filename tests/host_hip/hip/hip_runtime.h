// Host stand-in for the HIP headers: one workgroup at a time, a std::thread per work-item, enough to run kernels that use
// LDS, workgroup barriers, lane shuffles and agent-scope atomics (no matrix cores, no direct loads into LDS).
#pragma once
#include <math.h>
#include <pthread.h>
#include <stdint.h>
#include <string.h>
#include <algorithm>
#include <functional>
#include <thread>
#include <vector>

#define __global__ static
#define __device__
#define __host__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __shared__ HOST_SHARED
#define HOST_SHARED static          // kernels with an `extern __shared__` array can be parsed (HOST_SHARED empty), not run

struct dim3h { unsigned x = 0, y = 0, z = 0; };
inline thread_local dim3h threadIdx, blockIdx, blockDim, gridDim;

struct int2 { int x, y; };
struct float2 { float x, y; };
struct float4 { float x, y, z, w; };
struct uint2 { uint32_t x, y; };
struct uint4 { uint32_t x, y, z, w; };
inline float2 make_float2(float x, float y) { return {x, y}; }
inline float4 make_float4(float x, float y, float z, float w) { return {x, y, z, w}; }
inline uint2 make_uint2(uint32_t x, uint32_t y) { return {x, y}; }
using std::max;
using std::min;

inline float __uint_as_float(uint32_t u) { float f; memcpy(&f, &u, 4); return f; }
inline uint32_t __float_as_uint(float f) { uint32_t u; memcpy(&u, &f, 4); return u; }
inline uint32_t __umulhi(uint32_t a, uint32_t b) { return (uint32_t)(((uint64_t)a * b) >> 32); }
inline int __popcll(unsigned long long v) { return __builtin_popcountll(v); }
inline int __clz(int v) { return __builtin_clz((unsigned)v); }
#define __expf expf

// the workgroup that is running: a barrier for all, one per wave, and a word per work-item to shuffle through
struct HostGroup {
    pthread_barrier_t all, wave[16];
    uint32_t word[1024];
};
inline HostGroup host_group;
inline void __syncthreads() { pthread_barrier_wait(&host_group.all); }
template <typename T> inline T host_from_lane(T v, int lane) {
    static_assert(sizeof(T) == 4, "one word per lane");
    const unsigned w = threadIdx.x >> 6;
    memcpy(&host_group.word[threadIdx.x], &v, 4);
    pthread_barrier_wait(&host_group.wave[w]);
    T r; memcpy(&r, &host_group.word[w * 64 + (unsigned)(lane & 63)], 4);
    pthread_barrier_wait(&host_group.wave[w]);
    return r;
}
template <typename T> inline T __shfl_xor(T v, int o, int) { return host_from_lane(v, (int)(threadIdx.x & 63) ^ o); }
template <typename T> inline T __shfl(T v, int l, int) { return host_from_lane(v, l); }
template <typename T> inline T __shfl_up(T v, int o, int) { const int l = (int)(threadIdx.x & 63); return host_from_lane(v, l >= o ? l - o : l); }

#define __HIP_MEMORY_SCOPE_AGENT 0
template <typename P> inline P host_atomic_load(const P *p) { P v; __atomic_load(p, &v, __ATOMIC_SEQ_CST); return v; }
#define __hip_atomic_load(p, order, scope) host_atomic_load(p)
#define __hip_atomic_fetch_add(p, v, order, scope) __atomic_fetch_add(p, v, __ATOMIC_SEQ_CST)
template <typename P, typename V> inline void host_atomic_store(P *p, V v) { P w = v; __atomic_store(p, &w, __ATOMIC_SEQ_CST); }
#define __hip_atomic_store(p, v, order, scope) host_atomic_store(p, v)
template <typename P> inline P host_atomic_max(P *p, P v) { P o = __atomic_load_n(p, __ATOMIC_SEQ_CST); while (o < v && !__atomic_compare_exchange_n(p, &o, v, false, __ATOMIC_SEQ_CST, __ATOMIC_SEQ_CST)) {} return o; }
#define __hip_atomic_fetch_max(p, v, order, scope) host_atomic_max(p, v)
inline void atomicOr(int *p, int v) { __atomic_fetch_or(p, v, __ATOMIC_SEQ_CST); }

#define __builtin_amdgcn_readfirstlane(x) (x)
#define __builtin_amdgcn_sched_barrier(x) ((void)0)
#define __builtin_amdgcn_exp2f(x) exp2f(x)
#define __builtin_amdgcn_s_barrier() ((void)0)
#define __builtin_amdgcn_s_waitcnt(x) ((void)0)
#define __builtin_amdgcn_global_load_lds(...) ((void)0)
#define __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, ...) (c)

// run `body` as every workgroup of a grid, one after the other
template <typename F> inline void host_launch(unsigned grid, unsigned threads, F body) {
    for (unsigned b = 0; b < grid; ++b) {
        pthread_barrier_init(&host_group.all, nullptr, threads);
        for (unsigned w = 0; w < (threads + 63) / 64; ++w) pthread_barrier_init(&host_group.wave[w], nullptr, std::min(64u, threads - 64 * w));
        std::vector<std::thread> pool;
        for (unsigned t = 0; t < threads; ++t)
            pool.emplace_back([=] { threadIdx = {t, 0, 0}; blockIdx = {b, 0, 0}; blockDim = {threads, 1, 1}; gridDim = {grid, 1, 1}; body(); });
        for (auto &t : pool) t.join();
    }
}
