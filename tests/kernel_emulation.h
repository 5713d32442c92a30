// A gfx950 workgroup on the CPU, enough of it to run the library's single-pass
// kernels from their own source (kernel_emulation.cpp includes
// lamb_kernels.hip after this header): every workgroup is an OS thread, every
// lane a fiber of it, __shared__ a thread_local static, a buffer descriptor a
// bounds-checked pointer.
//
// Nothing runs in lockstep. Between two points where the hardware makes lanes
// meet (a barrier for a workgroup, a DPP move or a readlane for a wave) a wave
// runs as far ahead of the others as it can, in the order of waves that the
// caller picks. A result that depends on that order is a race.
#pragma once

#ifndef __HIP_PLATFORM_AMD__
#define __HIP_PLATFORM_AMD__
#endif
#include <hip/hip_runtime_api.h>

#include <sched.h>
#include <stdint.h>
#include <string.h>
#include <ucontext.h>

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <memory>
#include <thread>
#include <vector>

using std::isfinite;
using std::isinf;
using std::isnan;

#define __device__
#define __global__
#define __host__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define amdgpu_waves_per_eu(n)
#define __shared__ static thread_local

namespace emulation {

constexpr int kWave = 64;
constexpr size_t kStack = 256 * 1024;

struct Dim {
    uint32_t x = 1, y = 1, z = 1;
};

enum class At { kRunnable, kWave, kBarrier, kDone };

struct Lane {
    ucontext_t context;
    std::unique_ptr<char[]> stack;
    At at = At::kRunnable;
    uint32_t exchanges = 0;
    int value[2] = {0, 0};  // what the lane shows the others, by exchange parity
};

struct Workgroup {
    Dim block_idx, block_dim, grid_dim;
    std::vector<Lane> lanes;
    ucontext_t scheduler;
    int current = 0;
    void (*body)(void *) = nullptr;
    void *argument = nullptr;
    int any = 0;  // of __syncthreads_or
};

inline thread_local Workgroup *group = nullptr;
inline thread_local Dim thread_index;
inline thread_local uint64_t sleeps = 0;  // s_sleep calls of the workgroup's lanes

inline void lane_main() {
    Workgroup *g = group;
    g->body(g->argument);
    Lane &lane = g->lanes[size_t(g->current)];
    lane.at = At::kDone;
    swapcontext(&lane.context, &g->scheduler);
}

inline void stop_at(At at) {
    Workgroup *g = group;
    Lane &lane = g->lanes[size_t(g->current)];
    lane.at = at;
    swapcontext(&lane.context, &g->scheduler);
}

inline void run_lane(Workgroup &g, int k) {
    g.current = k;
    thread_index.x = uint32_t(k);
    swapcontext(&g.scheduler, &g.lanes[size_t(k)].context);
}

// Runs body(argument) on every lane of workgroup `index` of `grid`; waves
// first to last, or last to first.
inline void run_workgroup(uint32_t index, uint32_t grid, uint32_t threads, bool last_first,
                          void (*body)(void *), void *argument) {
    Workgroup g;
    g.block_idx.x = index;
    g.grid_dim.x = grid;
    g.block_dim.x = threads;
    g.body = body;
    g.argument = argument;
    g.lanes.resize(threads);
    group = &g;
    for (Lane &lane : g.lanes) {
        lane.stack.reset(new char[kStack]);
        getcontext(&lane.context);
        lane.context.uc_stack.ss_sp = lane.stack.get();
        lane.context.uc_stack.ss_size = kStack;
        lane.context.uc_link = nullptr;
        makecontext(&lane.context, lane_main, 0);
    }
    const int waves = int(threads) / kWave;
    for (;;) {
        for (int w = 0; w < waves; ++w) {
            const int first = (last_first ? waves - 1 - w : w) * kWave;
            for (;;) {  // this wave, until it waits for the workgroup
                bool ran = false;
                int meeting = 0;
                for (int k = first; k < first + kWave; ++k)
                    if (g.lanes[size_t(k)].at == At::kRunnable) {
                        run_lane(g, k);
                        ran = true;
                    }
                for (int k = first; k < first + kWave; ++k)
                    meeting += g.lanes[size_t(k)].at == At::kWave;
                if (meeting == kWave) {
                    for (int k = first; k < first + kWave; ++k)
                        g.lanes[size_t(k)].at = At::kRunnable;
                    continue;
                }
                if (meeting != 0) {
                    fprintf(stderr, "a wave operation without all 64 lanes\n");
                    abort();
                }
                if (!ran)
                    break;
            }
        }
        size_t done = 0, waiting = 0;
        for (const Lane &lane : g.lanes) {
            done += lane.at == At::kDone;
            waiting += lane.at == At::kBarrier;
        }
        if (done == g.lanes.size())
            break;
        if (waiting != g.lanes.size()) {
            fprintf(stderr, "a barrier that %zu of %zu lanes reach\n", waiting, g.lanes.size());
            abort();
        }
        for (Lane &lane : g.lanes)
            lane.at = At::kRunnable;
    }
    group = nullptr;
}

// The value that lane `source` of the calling lane's wave shows, each lane
// showing `v`.
inline int exchange(int v, int source) {
    Workgroup *g = group;
    Lane &lane = g->lanes[size_t(g->current)];
    const uint32_t parity = lane.exchanges++ & 1u;
    lane.value[parity] = v;
    stop_at(At::kWave);
    return g->lanes[size_t(g->current / kWave * kWave + source)].value[parity];
}

}  // namespace emulation

#define threadIdx (emulation::thread_index)
#define blockIdx (emulation::group->block_idx)
#define blockDim (emulation::group->block_dim)
#define gridDim (emulation::group->grid_dim)

inline void __syncthreads() { emulation::stop_at(emulation::At::kBarrier); }

inline int __syncthreads_or(int v) {
    int *any = &emulation::group->any;
    __syncthreads();  // (every lane has read the value of the call before)
    *any |= v;
    __syncthreads();
    const int r = *any;
    __syncthreads();
    *any = 0;
    return r;
}

template <typename To, typename From>
inline To emulated_bits(From v) {
    static_assert(sizeof(To) == sizeof(From), "sizes");
    To r;
    memcpy(&r, &v, sizeof r);
    return r;
}
inline float __uint_as_float(uint32_t v) { return emulated_bits<float>(v); }
inline uint32_t __float_as_uint(float v) { return emulated_bits<uint32_t>(v); }
inline double __longlong_as_double(long long v) { return emulated_bits<double>(v); }
inline long long __double_as_longlong(double v) { return emulated_bits<long long>(v); }
inline float __fdiv_rn(float a, float b) { return a / b; }
inline float __fadd_rn(float a, float b) { return a + b; }
inline float __fsqrt_rn(float a) { return std::sqrt(a); }
inline uint32_t atomicOr(uint32_t *p, uint32_t v) { return __atomic_fetch_or(p, v, __ATOMIC_SEQ_CST); }

#ifndef __HIP_MEMORY_SCOPE_AGENT
#define __HIP_MEMORY_SCOPE_AGENT 0
#endif
#define __hip_atomic_load(p, order, scope) __atomic_load_n(p, __ATOMIC_SEQ_CST)
#define __hip_atomic_store(p, v, order, scope) __atomic_store_n(p, v, __ATOMIC_SEQ_CST)
#define __hip_atomic_fetch_add(p, v, order, scope) __atomic_fetch_add(p, v, __ATOMIC_SEQ_CST)
#define __hip_atomic_fetch_or(p, v, order, scope) __atomic_fetch_or(p, v, __ATOMIC_SEQ_CST)

#define __builtin_amdgcn_s_setprio(p) ((void)0)
#define __builtin_amdgcn_sched_barrier(m) ((void)0)
#define __builtin_amdgcn_s_memrealtime() uint64_t(0)
#define __builtin_amdgcn_s_sleep(n) ((void)++emulation::sleeps, (void)sched_yield())

// quad_perm (controls below 0x100), row_mirror, row_half_mirror
inline int __builtin_amdgcn_mov_dpp(int v, int control, int, int, bool) {
    const int lane = int(threadIdx.x) % emulation::kWave;
    int source = lane;
    if (control < 0x100)
        source = (lane & ~3) | (control >> 2 * (lane & 3) & 3);
    else if (control == 0x140)
        source = (lane & ~15) | (15 - (lane & 15));
    else if (control == 0x141)
        source = (lane & ~7) | (7 - (lane & 7));
    else
        abort();
    return emulation::exchange(v, source);
}
inline int __builtin_amdgcn_readlane(int v, int lane) { return emulation::exchange(v, lane); }

struct EmulatedBuffer {
    char *base;
    uint32_t bytes;
};
#define __amdgpu_buffer_rsrc_t EmulatedBuffer
typedef uint32_t emulated_u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t emulated_u32x2 __attribute__((ext_vector_type(2)));

inline EmulatedBuffer __builtin_amdgcn_make_buffer_rsrc(void *p, int, int bytes, int) {
    return EmulatedBuffer{static_cast<char *>(p), uint32_t(bytes)};
}
template <typename T>
inline T emulated_load(const EmulatedBuffer &b, uint32_t at) {
    T r = {};
    if (uint64_t(at) + sizeof(T) <= b.bytes)
        memcpy(&r, b.base + at, sizeof r);
    return r;
}
template <typename T>
inline void emulated_store(const EmulatedBuffer &b, uint32_t at, T v) {
    if (uint64_t(at) + sizeof(T) <= b.bytes)
        memcpy(b.base + at, &v, sizeof v);
}
#define __builtin_amdgcn_raw_buffer_load_b128(r, at, base, aux) emulated_load<emulated_u32x4>(r, at)
#define __builtin_amdgcn_raw_buffer_load_b64(r, at, base, aux) emulated_load<emulated_u32x2>(r, at)
#define __builtin_amdgcn_raw_buffer_store_b128(v, r, at, base, aux) emulated_store<emulated_u32x4>(r, at, v)
#define __builtin_amdgcn_raw_buffer_store_b64(v, r, at, base, aux) emulated_store<emulated_u32x2>(r, at, v)
