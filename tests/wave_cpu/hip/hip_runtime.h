// Stand-in for the HIP runtime that lets a CPU test run the kernels' own source, lane by lane.
//
// Every thread of a workgroup is a fiber.  A fiber runs until it meets an operation in which the lanes of
// its wave (or, for a barrier, all waves) take part, and goes on when all of them are there; lanes that
// have returned do not take part.  Workgroups run one after another.  Only what the tested sources use is
// here.  Built with g++ (the AMDGCN builtins are ordinary functions then), without -pie, so that the
// 32-bit addresses some kernels keep of their LDS arrays are whole pointers.
#pragma once

#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <ucontext.h>

#include <functional>
#include <vector>

#define __device__
#define __host__
#define __global__
#define __shared__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __align__(n) alignas(n)

struct dim3 {
    unsigned x, y, z;
    dim3(unsigned x_ = 1, unsigned y_ = 1, unsigned z_ = 1) : x(x_), y(y_), z(z_) {}
};
struct int2 { int x, y; };
struct uint2 { unsigned x, y; };
inline uint2 make_uint2(unsigned x, unsigned y) { return {x, y}; }
struct int4 { int x, y, z, w; };
inline int2 make_int2(int x, int y) { return {x, y}; }
inline int4 make_int4(int x, int y, int z, int w) { return {x, y, z, w}; }
struct float2 { float x, y; };
inline float2 make_float2(float x, float y) { return {x, y}; }
typedef void *hipStream_t;
typedef int hipError_t;
enum { hipSuccess = 0, hipErrorInvalidConfiguration = 9 };

inline dim3 threadIdx, blockIdx, blockDim, gridDim;

namespace wave {
enum op { NONE, BALLOT, SHFL_XOR, SHFL_UP, DPP, READLANE, WAVE_BARRIER, BLOCK_BARRIER };
struct lane {
    ucontext_t at;
    std::vector<char> stack;
    bool done = false;
    op waits = NONE;
    long long v = 0, old = 0, out = 0;  // what the lane brings to the operation and gets from it
    int arg = 0;
};
inline std::vector<lane> lanes;
inline ucontext_t scheduler;
inline int me;
inline const std::function<void()> *body;
inline unsigned long long votes = 1;  // changes with every vote's outcome

inline long long meet(op o, long long v, int arg = 0, long long old = 0) {
    lane &l = lanes[me];
    l.waits = o;
    l.v = v;
    l.arg = arg;
    l.old = old;
    swapcontext(&l.at, &scheduler);
    return lanes[me].out;
}

inline void start() {
    (*body)();
    lanes[me].done = true;
    swapcontext(&lanes[me].at, &scheduler);
}

// What the DPP controls used by the kernels read: the source lane, or -1 (the lane keeps `old`).
inline int dpp_source(int ctrl, int i) {
    const int row = i & ~15;
    if (ctrl == 0x130) return i + 1 < 64 ? i + 1 : -1;
    if (ctrl == 0x138) return i - 1;
    if (ctrl > 0x100 && ctrl < 0x110) return (i & 15) + (ctrl & 15) < 16 ? i + (ctrl & 15) : -1;
    if (ctrl > 0x110 && ctrl < 0x120) return (i & 15) >= (ctrl & 15) ? i - (ctrl & 15) : -1;
    if (ctrl < 0x100) return (i & ~3) | (ctrl >> 2 * (i & 3) & 3);
    if (ctrl == 0x140) return row + 15 - (i & 15);
    if (ctrl == 0x141) return (i & ~7) + 7 - (i & 7);
    fprintf(stderr, "dpp control %x\n", ctrl);
    abort();
}

// Lets the lanes [a, b) that wait for a wave operation have its result.
inline void serve(int a, int b) {
    op o = NONE;
    unsigned long long vote = 0;
    for (int i = a; i < b; ++i)
        if (!lanes[i].done) {
            if (o == NONE) o = lanes[i].waits;
            if (lanes[i].waits != o) { fprintf(stderr, "the lanes of a wave meet different operations\n"); abort(); }
            if (lanes[i].v) vote |= 1ull << (i - a);
        }
    if (o == BALLOT) {
        votes = (votes ^ vote) * 0x9e3779b97f4a7c15ull;
        votes ^= votes >> 32;
    }
    for (int i = a; i < b; ++i) {
        lane &l = lanes[i];
        if (l.done) continue;
        auto of = [&](int j) { return j >= 0 && a + j < b && !lanes[a + j].done; };
        if (o == BALLOT) l.out = (long long)vote;
        else if (o == SHFL_XOR) l.out = of((i - a) ^ l.arg) ? lanes[a + ((i - a) ^ l.arg)].v : l.v;
        else if (o == SHFL_UP) l.out = i - a >= l.arg ? lanes[i - l.arg].v : l.v;
        else if (o == READLANE) l.out = lanes[a + l.arg].v;
        else if (o == DPP) {
            const int j = dpp_source(l.arg, i - a);
            l.out = of(j) ? lanes[a + j].v : l.old;
        }
        l.waits = NONE;
    }
}

// One workgroup of `threads` threads.
inline void run_group(int threads, const std::function<void()> &kernel) {
    body = &kernel;
    lanes.clear();
    lanes.resize(threads);
    for (int i = 0; i < threads; ++i) {
        lanes[i].stack.resize(128 * 1024);
        getcontext(&lanes[i].at);
        lanes[i].at.uc_stack.ss_sp = lanes[i].stack.data();
        lanes[i].at.uc_stack.ss_size = lanes[i].stack.size();
        lanes[i].at.uc_link = &scheduler;
        makecontext(&lanes[i].at, start, 0);
    }
    for (;;) {
        bool any = false, at_barrier = true;
        for (int i = 0; i < threads; ++i) {
            if (lanes[i].done || lanes[i].waits != NONE) continue;
            me = i;
            threadIdx = dim3(i);
            swapcontext(&scheduler, &lanes[i].at);
        }
        for (int a = 0; a < threads; a += 64) {
            const int b = a + 64 < threads ? a + 64 : threads;
            bool block = true;
            for (int i = a; i < b; ++i)
                if (!lanes[i].done) { any = true; block &= lanes[i].waits == BLOCK_BARRIER; }
            if (block) continue;
            at_barrier = false;
            serve(a, b);
        }
        if (!any) return;
        if (at_barrier) {
            long long all = 1;
            for (lane &l : lanes) if (!l.done) all &= l.v != 0;
            for (lane &l : lanes) { l.out = all; l.waits = NONE; }
        }
    }
}

// Launches: threads of a dimension are limited as HIP limits them.  With `dry` set nothing runs.
inline bool dry = false;
inline hipError_t last = hipSuccess;
struct launched { dim3 grid, block; size_t lds; };
inline std::vector<launched> launches;

template <typename K, typename A>
void launch(K kernel, dim3 grid, dim3 block, size_t lds, const A &args) {
    launches.push_back({grid, block, lds});
    if ((unsigned long long)grid.x * block.x >= 1ull << 32 || !grid.x || block.x > 1024) {
        last = hipErrorInvalidConfiguration;
        return;
    }
    if (dry) return;
    gridDim = grid;
    blockDim = block;
    for (unsigned y = 0; y < grid.y; ++y)
        for (unsigned x = 0; x < grid.x; ++x) {
            blockIdx = dim3(x, y);
            run_group((int)block.x, [&] { kernel(args); });
        }
}
}  // namespace wave

#define hipLaunchKernelGGL(kernel, grid, block, lds, stream, ...) wave::launch(kernel, grid, block, lds, __VA_ARGS__)
inline hipError_t hipGetLastError() { const hipError_t e = wave::last; wave::last = hipSuccess; return e; }

inline unsigned long long __ballot(bool v) { return (unsigned long long)wave::meet(wave::BALLOT, v); }
inline unsigned long long __builtin_amdgcn_ballot_w64(bool v) { return __ballot(v); }
inline int __shfl_xor(int v, int m) { return (int)wave::meet(wave::SHFL_XOR, v, m); }
inline long long __shfl_xor(long long v, int m) { return wave::meet(wave::SHFL_XOR, v, m); }
inline unsigned long long __shfl_xor(unsigned long long v, int m) { return (unsigned long long)wave::meet(wave::SHFL_XOR, (long long)v, m); }
inline long long __shfl_up(long long v, int d) { return wave::meet(wave::SHFL_UP, v, d); }
inline int __shfl(int v, int i) { return (int)wave::meet(wave::READLANE, v, i); }
inline float __shfl(float v, int i) { return __builtin_bit_cast(float, __shfl(__builtin_bit_cast(int, v), i)); }
inline int __shfl_up(int v, int d) { return (int)wave::meet(wave::SHFL_UP, v, d); }
inline int __builtin_amdgcn_update_dpp(int old, int v, int ctrl, int, int, bool) { return (int)wave::meet(wave::DPP, v, ctrl, old); }
inline int __builtin_amdgcn_readfirstlane(int v) { return (int)wave::meet(wave::READLANE, v, 0); }
inline int __builtin_amdgcn_readlane(int v, int i) { return (int)wave::meet(wave::READLANE, v, i); }
inline void __builtin_amdgcn_wave_barrier() { wave::meet(wave::WAVE_BARRIER, 0); }
#define __builtin_amdgcn_fence(...) ((void)0)
#define __builtin_amdgcn_s_setprio(...) ((void)0)
// (the hardware's reciprocal is off by an ulp or so: a little more here, now too large and now too small)
inline double __builtin_amdgcn_rcp(double x) { return 1.0 / x * (1.0 + ((long long)x & 1 ? 1 : -1) * 0x1p-24); }
inline int __popc(unsigned v) { return __builtin_popcount(v); }
inline int __float_as_int(float v) { return __builtin_bit_cast(int, v); }
inline float __int_as_float(int v) { return __builtin_bit_cast(float, v); }
inline int __mul24(int a, int b) { return a * b; }
inline void __syncthreads() { wave::meet(wave::BLOCK_BARRIER, 1); }
inline int __syncthreads_and(int v) { return (int)wave::meet(wave::BLOCK_BARRIER, v); }
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __hip_atomic_load(p, order, scope) (*(p))
template <typename T, typename V> T atomicOr(T *p, V v) { T o = *p; *p |= (T)v; return o; }
template <typename T, typename V> T atomicAdd(T *p, V v) { T o = *p; *p += (T)v; return o; }
template <typename T, typename V> T atomicMax(T *p, V v) { T o = *p; if ((T)v > o) *p = (T)v; return o; }
template <typename T, typename V> T atomicMin(T *p, V v) { T o = *p; if ((T)v < o) *p = (T)v; return o; }
