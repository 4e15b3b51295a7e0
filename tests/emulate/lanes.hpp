// One workgroup of 64-lane waves on the CPU.  A lane is a fiber; it runs until
// it waits: for the other lanes of its wave (ballots, lane exchanges) or for
// the workgroup (a barrier).  Which wave runs next is a test's choice, so a
// wave can be held back at a barrier it has already been let through, or run
// ahead of all others: what one wave does must not depend on it.  Waves that
// meet at different barriers, or a wave that ends while others wait, end the
// program with an error.
#pragma once
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include <ucontext.h>

#include <functional>
#include <memory>
#include <vector>

#define __global__
#define __device__
#define __host__
#define __constant__ static
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __shared__ static

namespace lanes {

enum class State { ready, wave, barrier, done };

struct Wave {
    uint64_t value[2][64];
    int arrived = 0, turn = 0, priority = 0;
};

struct Lane {
    ucontext_t ctx;
    State state = State::ready;
    int line = 0;                                  // of the barrier it waits at; 0: of none yet
    std::unique_ptr<char[]> stack;
};

inline std::vector<Lane> lane;
inline std::vector<Wave> wave;
inline int current, waiting, present;              // present: lanes but those that ended before any barrier
inline unsigned block;
inline ucontext_t scheduler;
inline std::function<void()> body;

[[noreturn]] inline void fail(const char *what, int a = 0, int b = 0)
{
    printf("FAILED: %s (%d, %d)\n", what, a, b);
    fflush(stdout);
    _exit(1);
}

inline void wait_as(State s)
{
    Lane &l = lane[current];
    l.state = s;
    swapcontext(&l.ctx, &scheduler);
}

// Every lane's value, once all 64 lanes of the wave have come here.
inline const uint64_t *exchange(uint64_t v)
{
    Wave &w = wave[current / 64];
    const int turn = w.turn & 1;
    w.value[turn][current % 64] = v;
    if (++w.arrived < 64) wait_as(State::wave);
    else {
        w.arrived = 0;
        ++w.turn;
        const int first = current / 64 * 64;
        for (int i = first; i < first + 64; ++i)
            if (lane[i].state == State::wave) lane[i].state = State::ready;
        wait_as(State::ready);
    }
    return w.value[turn];
}

// All present wait: at one and the same barrier, or waves have parted.
inline void release()
{
    int line = 0;
    waiting = 0;
    for (auto &l : lane) {
        if (l.state == State::done) continue;
        if (line == 0) line = l.line;
        if (l.line != line) fail("waves meet at different barriers, at lines", line, l.line);
        l.state = State::ready;
    }
}

inline void barrier(int line)
{
    lane[current].line = line;
    ++waiting;
    if (waiting < present) {
        wait_as(State::barrier);
        return;
    }
    lane[current].state = State::barrier;
    release();
    wait_as(State::ready);
}

inline void entry()
{
    body();
    lane[current].state = State::done;
    if (lane[current].line == 0 && --present > 0 && waiting == present) release();
    swapcontext(&lane[current].ctx, &scheduler);
}

// Runs `kernel` as workgroup `b` of `threads` threads.  The wave of the
// highest priority that can go on goes on; of its lanes the highest first, so
// that what lane 0 alone stores comes after the whole wave's reads before it,
// as in a wave that runs in step.
inline void run(int threads, unsigned b, const std::vector<int> &priority, std::function<void()> kernel)
{
    constexpr size_t kStack = 64 << 10;
    body = std::move(kernel);
    block = b;
    waiting = 0;
    present = threads;
    lane.resize(threads);
    wave.assign(threads / 64, Wave{});
    for (int w = 0; w < threads / 64; ++w) wave[w].priority = priority[w];
    for (int i = 0; i < threads; ++i) {
        Lane &l = lane[i];
        if (!l.stack) l.stack.reset(new char[kStack]);
        l.state = State::ready;
        l.line = 0;
        getcontext(&l.ctx);
        l.ctx.uc_stack.ss_sp = l.stack.get();
        l.ctx.uc_stack.ss_size = kStack;
        l.ctx.uc_link = nullptr;
        makecontext(&l.ctx, entry, 0);
    }
    for (;;) {
        int best = -1, left = 0;
        for (int w = 0; w < threads / 64; ++w) {
            if (best >= 0 && wave[w].priority <= wave[best / 64].priority) continue;
            for (int i = 64 * w + 63; i >= 64 * w; --i)
                if (lane[i].state == State::ready) {
                    best = i;
                    break;
                }
        }
        if (best < 0) {
            for (auto &l : lane) left += l.state != State::done;
            if (left) fail("a wave ended while others wait at a barrier; lanes left, line", left, lane[0].line);
            return;
        }
        current = best;
        swapcontext(&scheduler, &lane[best].ctx);
    }
}

struct ThreadIdx {
    struct {
        operator unsigned() const { return (unsigned)current; }
    } x;
};
struct BlockIdx {
    struct {
        operator unsigned() const { return block; }
    } x;
};

}  // namespace lanes

static const lanes::ThreadIdx threadIdx{};
static const lanes::BlockIdx blockIdx{};

// ---- the device functions the kernels under test use ----
#define __syncthreads() lanes::barrier(__LINE__)
#define __builtin_amdgcn_s_barrier() lanes::barrier(-1)
#define __builtin_amdgcn_fence(...) ((void)0)

inline uint32_t __float_as_uint(float f) { return __builtin_bit_cast(uint32_t, f); }
inline float __uint_as_float(uint32_t u) { return __builtin_bit_cast(float, u); }
inline int __float_as_int(float f) { return __builtin_bit_cast(int, f); }
inline float __int_as_float(int u) { return __builtin_bit_cast(float, u); }
inline int __popcll(uint64_t v) { return __builtin_popcountll(v); }
inline uint64_t __ballot(uint64_t v)
{
    const uint64_t *all = lanes::exchange(v);
    uint64_t b = 0;
    for (int i = 0; i < 64; ++i) b |= (uint64_t)(all[i] != 0) << i;
    return b;
}
inline int __builtin_amdgcn_readlane(int v, int from) { return (int)lanes::exchange((uint32_t)v)[from]; }
inline int __builtin_amdgcn_readfirstlane(int v) { return (int)lanes::exchange((uint32_t)v)[0]; }
inline float __shfl(float v, int from) { return __uint_as_float((uint32_t)lanes::exchange(__float_as_uint(v))[from]); }
inline uint32_t __builtin_amdgcn_mbcnt_lo(uint32_t mask, uint32_t add)
{
    const int l = lanes::current % 64;
    return add + (uint32_t)__builtin_popcount(l >= 32 ? mask : mask & ((1u << l) - 1));
}
inline uint32_t __builtin_amdgcn_mbcnt_hi(uint32_t mask, uint32_t add)
{
    const int l = lanes::current % 64;
    return add + (uint32_t)__builtin_popcount(l < 32 ? 0 : mask & ((1u << (l - 32)) - 1));
}
// row_shr:1..15 and the row broadcasts, all banks.
inline int __builtin_amdgcn_update_dpp(int old, int src, int ctrl, int row_mask, int, bool zero_fill)
{
    const uint64_t *all = lanes::exchange((uint32_t)src);
    const int l = lanes::current % 64, row = l / 16;
    if (!(row_mask >> row & 1)) return old;
    int from = -1;
    if (ctrl > 0x110 && ctrl < 0x120) from = l % 16 >= (ctrl & 15) ? l - (ctrl & 15) : -1;
    else if (ctrl == 0x142) from = row > 0 ? 16 * row - 1 : -1;
    else if (ctrl == 0x143) from = row > 1 ? 31 : -1;
    else lanes::fail("lane exchange not known here", ctrl);
    return from < 0 ? (zero_fill ? 0 : old) : (int)all[from];
}
inline int atomicAdd(int *p, int v)
{
    const int o = *p;
    *p += v;
    return o;
}

// ---- the host side of the header: launches are the test's own ----
typedef int hipError_t;
typedef void *hipStream_t;
struct dim3 {
    unsigned x, y, z;
    dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
enum { hipSuccess = 0, hipDeviceAttributeMultiprocessorCount = 0 };
inline hipError_t hipGetLastError() { return 0; }
inline hipError_t hipGetDevice(int *) { return 1; }
inline hipError_t hipDeviceGetAttribute(int *, int, int) { return 1; }
#define hipLaunchKernelGGL(...) ((void)0)
