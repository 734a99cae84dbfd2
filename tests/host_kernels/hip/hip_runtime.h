// A stand-in for <hip/hip_runtime.h> that runs kernels on the CPU, so that their indexing can
// be checked under AddressSanitizer: every thread of a workgroup is a fiber of one host thread,
// which changes fibers at __syncthreads and at the wave operations (ballot, shuffles).
// Workgroups run one after another; LDS is static memory.  Kernels of inline assembly or
// MFMAs compile but must not be run (their instructions are left out).
#pragma once

#include <limits.h>
#include <math.h>
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <functional>
#include <memory>
#include <mutex>
#include <random>
#include <type_traits>
#include <vector>

#define __device__
#define __host__
#define __global__
#define __shared__ static
#define __forceinline__ inline __attribute__((always_inline))
#define __launch_bounds__(...)

struct dim3 {
    unsigned x, y, z;
    dim3(unsigned x_ = 1, unsigned y_ = 1, unsigned z_ = 1) : x(x_), y(y_), z(z_) {}
};
struct int4 {
    int x, y, z, w;
};
inline int4 make_int4(int x, int y, int z, int w) { return {x, y, z, w}; }
inline dim3 threadIdx, blockIdx, blockDim, gridDim;

enum hipError_t { hipSuccess = 0 };
enum hipDeviceAttribute_t { hipDeviceAttributeMultiprocessorCount };
typedef void* hipStream_t;
typedef void* hipEvent_t;
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
inline int emu_cus = 256;  // the device's CUs
inline hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { return *v = emu_cus, hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }

using std::max;
using std::min;

namespace emu {

constexpr int kLanes = 64;
constexpr size_t kStack = 128 * 1024;
enum State { kRun, kAtWave, kAtBlock, kDone };
struct Fiber {
    void* sp;
    State state;
    int ops;  // wave operations so far
};
struct Machine {
    void* sched;
    std::vector<Fiber> fibers;
    std::vector<uint64_t> slot;  // [thread][parity]: a lane's value in a wave operation
    std::unique_ptr<char[]> stacks;
    std::function<void()> body;
    int current = 0, threads = 0;
};
inline Machine m;

// Saves the callee-saved registers and the stack pointer (x86-64) and continues on stack `to`.
__attribute__((naked, noinline)) inline void switch_stack(void** /*save*/, void* /*to*/) {
    __asm__("push %rbp; push %rbx; push %r12; push %r13; push %r14; push %r15; mov %rsp, (%rdi); mov %rsi, %rsp;"
            "pop %r15; pop %r14; pop %r13; pop %r12; pop %rbx; pop %rbp; ret");
}
inline void yield(State s) {
    m.fibers[m.current].state = s;
    const int me = m.current;
    switch_stack(&m.fibers[me].sp, m.sched);
    threadIdx.x = (unsigned)me;
}
inline void entry() {
    m.body();
    m.fibers[m.current].state = kDone;
    switch_stack(&m.fibers[m.current].sp, m.sched);
}
// One wave operation: v of every lane of this wave after all live ones have arrived.
inline const uint64_t* exchange(uint64_t v) {
    Fiber& f = m.fibers[m.current];
    const int wave = m.current / kLanes, lane = m.current % kLanes, parity = f.ops++ & 1;
    uint64_t* row = m.slot.data() + (size_t)(2 * wave + parity) * kLanes;
    row[lane] = v;
    yield(kAtWave);
    return row;
}
inline void run_workgroup() {
    for (int i = 0; i < m.threads; ++i) {
        Fiber& f = m.fibers[i];
        void** top = reinterpret_cast<void**>(m.stacks.get() + (size_t)(i + 1) * kStack - 16);
        top[-2] = reinterpret_cast<void*>(entry);  // below it six registers; aligned at entry as after a call
        f.sp = top - 8;
        f.state = kRun;
        f.ops = 0;
    }
    std::fill(m.slot.begin(), m.slot.end(), 0);
    for (;;) {
        bool ran = false, alive = false, all_block = true;
        for (int i = 0; i < m.threads; ++i) {
            if (m.fibers[i].state != kRun) continue;
            ran = true;
            m.current = i;
            threadIdx.x = (unsigned)i;
            switch_stack(&m.sched, m.fibers[i].sp);
        }
        for (int w = 0; w < m.threads; w += kLanes) {
            bool wave = false, all = true;
            for (int i = w; i < min(m.threads, w + kLanes); ++i) {
                const State s = m.fibers[i].state;
                if (s == kDone) continue;
                alive = true;
                wave |= s == kAtWave;
                all &= s == kAtWave;
                all_block &= s == kAtBlock;
            }
            if (wave && all) {
                ran = true;
                all_block = false;
                for (int i = w; i < min(m.threads, w + kLanes); ++i)
                    if (m.fibers[i].state == kAtWave) m.fibers[i].state = kRun;
            }
        }
        if (!alive) return;
        if (all_block) {
            for (int i = 0; i < m.threads; ++i)
                if (m.fibers[i].state == kAtBlock) m.fibers[i].state = kRun;
        } else if (!ran) {
            fprintf(stderr, "divergent barrier or wave operation\n");
            abort();
        }
    }
}
template <typename F>
void launch(dim3 grid, dim3 block, F&& body) {
    m.threads = (int)block.x;
    m.fibers.resize(m.threads);
    m.slot.assign((size_t)(m.threads + kLanes - 1) / kLanes * 2 * kLanes, 0);
    m.stacks.reset(new char[(size_t)m.threads * kStack]);
    m.body = body;
    gridDim = grid;
    blockDim = block;
    for (unsigned y = 0; y < grid.y; ++y)
        for (unsigned x = 0; x < grid.x; ++x) {
            blockIdx = dim3(x, y);
            run_workgroup();
        }
}
template <typename T>
uint64_t bits(T v) {
    uint64_t b = 0;
    memcpy(&b, &v, sizeof(T));
    return b;
}
template <typename T>
T value(uint64_t b) {
    T v;
    memcpy(&v, &b, sizeof(T));
    return v;
}

}  // namespace emu

#define hipLaunchKernelGGL(kernel, grid, block, lds, stream, ...) \
    emu::launch(grid, block, [=] { (kernel)(__VA_ARGS__); })

inline void __syncthreads() { emu::yield(emu::kAtBlock); }
inline unsigned long long __ballot(bool p) {
    const uint64_t* v = emu::exchange(p);
    unsigned long long b = 0;
    for (int i = 0; i < emu::kLanes; ++i) b |= (unsigned long long)(v[i] & 1) << i;
    return b;
}
template <typename T>
T __shfl(T v, int src, int) {
    return emu::value<T>(emu::exchange(emu::bits(v))[src]);
}
template <typename T>
T __shfl_up(T v, int off, int) {
    const int lane = emu::m.current % emu::kLanes;
    return emu::value<T>(emu::exchange(emu::bits(v))[lane >= off ? lane - off : lane]);
}
template <typename T>
T __shfl_xor(T v, int mask, int) {
    const int lane = emu::m.current % emu::kLanes;
    return emu::value<T>(emu::exchange(emu::bits(v))[lane ^ mask]);
}
inline int __popcll(unsigned long long v) { return __builtin_popcountll(v); }
inline int __ffsll(long long v) { return __builtin_ffsll(v); }
inline int atomicAdd(int* p, int v) {
    const int old = *p;
    *p += v;
    return old;
}
inline int atomicMin(int* p, int v) {
    const int old = *p;
    *p = min(*p, v);
    return old;
}
inline uint32_t __float_as_uint(float f) { return emu::value<uint32_t>(emu::bits(f)); }
inline int __float_as_int(float f) { return emu::value<int>(emu::bits(f)); }
inline float __uint_as_float(uint32_t u) { return emu::value<float>(u); }
inline float __int_as_float(int i) { return emu::value<float>(emu::bits(i)); }

// device builtins of kernels that are compiled here but not run
#define __hip_atomic_load(p, order, scope) (*(p))
#define __hip_atomic_fetch_add(p, v, order, scope) (*(p) += (v))
#define __builtin_amdgcn_readfirstlane(v) (v)
#define __builtin_amdgcn_readlane(v, l) (v)
#define __builtin_amdgcn_mov_dpp(v, ...) (v)
#define __builtin_amdgcn_s_waitcnt(n) ((void)0)
#define __builtin_amdgcn_sched_barrier(n) ((void)0)
#define __builtin_amdgcn_rcpf(v) (1.0f / (v))
#define __expf(v) expf(v)
#define __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, ...) (c)
#define __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, ...) (c)
// inline assembly: `asm volatile(...)` is left out
#define asm
#define volatile(...) ((void)0)
