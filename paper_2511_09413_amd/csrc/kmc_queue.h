// Multi-step launches whose workgroups wait for one another need all of them
// resident at once.  Where other work holds the GPU that may not come true, so
// such a launch begins at a gate: either every workgroup passes or every one
// leaves with nothing changed.  The launch behind it then takes the same steps
// from a queue, which needs no two workgroups resident together: tickets are
// handed out in the order (step, tile), and a workgroup holding one waits only
// for tiles of earlier steps, whose tickets were all taken by workgroups that
// are running.  Whatever part of the GPU is free does the work, and workgroups
// that become resident later join in.
#pragma once
#include <stdint.h>

#include <hip/hip_runtime.h>

namespace kmc {

// Words of one launch and its queue, all zero when the launch begins.  A call
// uses two sets in turn; a launch clears the other one for its successor.
struct QueueWords {
    uint32_t gate[32];    // (a 128-byte line each) arrivals, and kQueueAbort when the launch left undone
    uint32_t ticket[32];  // tickets handed out
    uint32_t done[32];    // tiles completed
    uint32_t ready[32];   // steps whose end has been written
};
constexpr uint32_t kQueueAbort = 0x80000000u;
constexpr int64_t kGateTicks = 1000;  // 10 us per step of the launch: what the wait at its gate may cost
constexpr int kQueueWords = (int)(sizeof(QueueWords) / sizeof(uint32_t));

#if defined(__HIPCC__)
// One thread of each of the launch's `members` workgroups: whether all are
// resident.  After `ticks` (10 ns each) one of them gives up, unless the last
// one arrives first: one atomic word decides, so all pass or none.  No ticks:
// none passes (unless there is one alone).
__device__ inline bool queue_gate(uint32_t *gate, uint32_t members, int32_t ticks) {
    if (ticks <= 0 && members > 1u) {
        __hip_atomic_fetch_or(gate, kQueueAbort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return false;
    }
    uint32_t seen = __hip_atomic_fetch_add(gate, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u;
    const uint64_t t0 = __builtin_amdgcn_s_memrealtime();
    while (!(seen & kQueueAbort) && seen < members) {
        if ((int64_t)(__builtin_amdgcn_s_memrealtime() - t0) >= (int64_t)ticks) {
            uint32_t expect = seen;
            if (__hip_atomic_compare_exchange_strong(gate, &expect, seen | kQueueAbort, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                     __HIP_MEMORY_SCOPE_AGENT))
                expect = seen | kQueueAbort;
            seen = expect;
            continue;
        }
        __builtin_amdgcn_s_sleep(1);
        seen = __hip_atomic_load(gate, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    return !(seen & kQueueAbort);
}

// One thread: waits until *word is at least `want`.  False (and the flag is
// raised) after `limit` polls, or once another workgroup has raised it.
__device__ inline bool queue_wait(const uint32_t *word, uint32_t want, int32_t *flag, int32_t limit) {
    for (int32_t polls = 0; __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < want;) {
        if (++polls > limit) {
            __hip_atomic_store(flag, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return false;
        }
        if (__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return false;
        __builtin_amdgcn_s_sleep(2);
    }
    return true;
}

// Device-scope accesses of what other workgroups of the launch write: with them
// alone between workgroups, a tile counted as done needs no write-back of a
// whole L2 (only that its stores have been performed), and a wait no
// invalidation.
template <typename T>
__device__ __forceinline__ T queue_load(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ void queue_store(T *p, T v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// By every thread, before one counts the workgroup's tile.
__device__ __forceinline__ void queue_stores_done() {
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
}
#endif

}  // namespace kmc
