// One workgroup of a HIP kernel on the CPU: every thread is a fiber, threads run
// one after another in a chosen order, and each runs on until it waits at a
// workgroup barrier or a wave's exchange.  Threads that no barrier orders are so
// run in orders that a GPU may take but seldom does, which shows a missing
// barrier every time.  Included before the kernel's source, which is compiled as
// plain C++.
#pragma once

#include <hip/hip_runtime.h>
#include <ucontext.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <vector>

#define __launch_bounds__(...)
#ifndef __align__
#define __align__(n) __attribute__((aligned(n)))
#endif
#ifndef hipLaunchKernelGGL
#define hipLaunchKernelGGL(...) ((void)0)
#endif
using std::isfinite;
using std::max;
using std::min;

namespace cpu_group {

struct Index {
    unsigned x = 0, y = 0, z = 0;
};
enum Wait { kRun, kBarrier, kWave, kDone };
struct Thread {
    ucontext_t context;
    std::vector<char> stack;
    Wait wait = kRun;
    uint64_t slot = 0;   // this thread's value in a wave's exchange
};

inline std::vector<Thread> threads;
inline ucontext_t scheduler;
inline int current = 0;
inline std::function<void()> body;
inline unsigned char lds[160 * 1024];

inline void wait(Wait w) {
    const int t = current;
    threads[t].wait = w;
    swapcontext(&threads[t].context, &scheduler);
}
inline void entry() {
    body();
    wait(kDone);
}

}  // namespace cpu_group

inline cpu_group::Index threadIdx, blockIdx, blockDim, gridDim;

namespace cpu_group {

// Runs `kernel` as workgroup `block` of the threads in `order`.
inline void run(unsigned block, const std::vector<int> &order, std::function<void()> kernel) {
    body = std::move(kernel);
    threads = std::vector<Thread>(order.size());
    std::memset(lds, 0xA5, sizeof lds);
    blockIdx.x = block;
    blockDim.x = (unsigned)order.size();
    for (Thread &t : threads) {
        t.stack.resize(128 * 1024);
        getcontext(&t.context);
        t.context.uc_stack.ss_sp = t.stack.data();
        t.context.uc_stack.ss_size = t.stack.size();
        t.context.uc_link = &scheduler;
        makecontext(&t.context, entry, 0);
    }
    auto all = [&](size_t from, size_t to, Wait w) {
        for (size_t i = from; i < to; ++i)
            if (threads[i].wait != w && threads[i].wait != kDone) return false;
        return true;
    };
    while (!all(0, threads.size(), kDone)) {
        bool moved = false;
        for (int t : order) {
            if (threads[t].wait != kRun) continue;
            current = t;
            threadIdx.x = (unsigned)t;
            swapcontext(&scheduler, &threads[t].context);
            moved = true;
        }
        for (size_t w = 0; w < threads.size(); w += 64)
            if (all(w, w + 64, kWave)) {
                for (size_t i = w; i < w + 64; ++i)
                    if (threads[i].wait == kWave) threads[i].wait = kRun, moved = true;
            }
        if (all(0, threads.size(), kBarrier))
            for (Thread &t : threads)
                if (t.wait == kBarrier) t.wait = kRun, moved = true;
        if (!moved) {
            std::puts("threads wait for each other");
            std::exit(2);
        }
    }
}

// A wave's exchange: this lane's value, then that of lane `from`.
inline uint64_t exchange(uint64_t v, int from) {
    const int t = current;
    threads[t].slot = v;
    wait(kWave);
    const uint64_t got = threads[(t & ~63) + (from & 63)].slot;
    wait(kWave);
    return got;
}
template <class T>
T shuffle(T v, int from, bool valid) {
    uint64_t bits = 0;
    std::memcpy(&bits, &v, sizeof v);
    const uint64_t got = exchange(bits, valid ? from : current & 63);
    T r;
    std::memcpy(&r, &got, sizeof r);
    return r;
}

}  // namespace cpu_group

inline void __syncthreads() { cpu_group::wait(cpu_group::kBarrier); }
template <class T>
T __shfl_up(T v, int d, int = 64) {
    const int lane = cpu_group::current & 63;
    return cpu_group::shuffle(v, lane - d, lane >= d);
}
template <class T>
T __shfl_down(T v, int d, int = 64) {
    const int lane = cpu_group::current & 63;
    return cpu_group::shuffle(v, lane + d, lane + d < 64);
}
template <class T>
T __shfl_xor(T v, int d, int = 64) {
    return cpu_group::shuffle(v, (cpu_group::current & 63) ^ d, true);
}
// Votes that only choose between two ways to the same result: each lane decides.
inline int __all(int p) { return p; }
inline int __any(int p) { return p; }

template <class T>
T atomicAdd(T *p, T v) {
    const T old = *p;
    *p += v;
    return old;
}
template <class T>
T atomicMax(T *p, T v) {
    const T old = *p;
    *p = std::max(old, v);
    return old;
}
template <class To, class From>
To bits_as(From v) {
    To r;
    std::memcpy(&r, &v, sizeof r);
    return r;
}
inline uint32_t __float_as_uint(float v) { return bits_as<uint32_t>(v); }
inline float __uint_as_float(uint32_t v) { return bits_as<float>(v); }
inline long long __double_as_longlong(double v) { return bits_as<long long>(v); }
inline float __builtin_amdgcn_rsqf(float v) { return 1.0f / std::sqrt(v); }
inline float __builtin_amdgcn_rcpf(float v) { return 1.0f / v; }
inline double __builtin_amdgcn_rcp(double v) { return 1.0 / v; }
inline double __builtin_amdgcn_div_scale(double n, double d, bool num, bool *flag) {
    *flag = false;
    return num ? n : d;
}
inline double __builtin_amdgcn_div_fmas(double a, double b, double c, bool) {
    return std::fma(a, b, c);
}
inline double __builtin_amdgcn_div_fixup(double, double d, double n) { return n / d; }
// The conversion instruction of the kernels, which saturates.
inline int32_t saturating_int32(double v) {
    return v <= -2147483648.0 ? INT32_MIN : v >= 2147483647.0 ? INT32_MAX : (int32_t)v;
}

// Named by code that is compiled but not run here.
uint64_t __ballot(int);
int __syncthreads_or(int);
int __builtin_amdgcn_readfirstlane(int);
int __builtin_amdgcn_readlane(int, int);
unsigned __builtin_amdgcn_mbcnt_lo(unsigned, unsigned);
unsigned __builtin_amdgcn_mbcnt_hi(unsigned, unsigned);
inline void __builtin_amdgcn_sched_barrier(int) {}
inline void __builtin_amdgcn_wave_barrier() {}
inline void __builtin_amdgcn_s_sleep(int) {}
#define __builtin_amdgcn_fence(...) ((void)0)
#define __hip_atomic_load(p, ...) (*(p))
#define __hip_atomic_fetch_add(p, v, ...) (*(p) += (v))
