// The sweep kernel's code on the CPU: sv_sweep.hip compiled as plain C++, one
// host thread per lane of a workgroup, with the GPU's builtins as far as the
// checks that include this file need them (matrix instructions leave their
// accumulator as it is, lane exchanges are not available).
#pragma once

#include <hip/hip_runtime.h>
#include <pthread.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <random>
#include <string>
#include <thread>
#include <vector>

#include "sv.h"

struct Dim {
    unsigned x = 0, y = 0, z = 0;
};
static thread_local Dim threadIdx, blockIdx;

// One workgroup.  Its first wave runs ahead: the others start once it has met
// a barrier or ended, the order that a missing barrier cannot survive.
struct Workgroup {
    pthread_barrier_t bar;
    std::atomic<int> ahead{0};
    bool first_wave() const { return threadIdx.x < 64; }
};
static Workgroup* g_wg = nullptr;
static thread_local bool t_counted = false;

static void wave0_done()
{
    if (g_wg->first_wave() && !t_counted) {
        t_counted = true;
        ++g_wg->ahead;
    }
}

static void __syncthreads()
{
    wave0_done();
    pthread_barrier_wait(&g_wg->bar);
}

static void run_workgroup(int nt, const std::function<void()>& body)
{
    Workgroup wg;
    g_wg = &wg;
    pthread_barrier_init(&wg.bar, nullptr, unsigned(nt));
    std::vector<std::thread> threads;
    for (int t = 0; t < nt; ++t)
        threads.emplace_back([&, t] {
            threadIdx.x = unsigned(t);
            t_counted = false;
            while (!wg.first_wave() && wg.ahead.load() < 64) std::this_thread::yield();
            body();
            wave0_done();
        });
    for (auto& t : threads) t.join();
    pthread_barrier_destroy(&wg.bar);
}

template <typename T>
static T no_lanes(T)
{
    std::printf("a lane exchange was reached\n");
    std::exit(2);
}

static void sincospif(float x, float* s, float* c)
{
    *s = std::sin(float(M_PI) * x);
    *c = std::cos(float(M_PI) * x);
}

#define __launch_bounds__(...)
#undef __align__
#define __align__(x) __attribute__((aligned(x)))
#define __popcll(x) __builtin_popcountll(x)
#define __dadd_rn(x, y) ((x) + (y))
#define __dsub_rn(x, y) ((x) - (y))
#define __dmul_rn(x, y) ((x) * (y))
#define __shfl_xor(x, mask, width) no_lanes(x)
#define __ballot(x) uint64_t(no_lanes(x))
#define __builtin_amdgcn_readlane(x, l) no_lanes(x)
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __builtin_amdgcn_sched_barrier(x) ((void)0)
#define __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, x, y, z) ((void)(a), (void)(b), (c))
#define __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, x, y, z) ((void)(a), (void)(b), (c))
#define __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, x, y, z) ((void)(a), (void)(b), (c))
#define __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, x, y, z) ((void)(a), (void)(b), (c))
#define hipLaunchKernelGGL(...) ((void)0)
#define hipGetLastError() hipSuccess
#define hipGetErrorString(e) "error"
// inline assembly only pins registers there
#define asm
#define volatile(...)
