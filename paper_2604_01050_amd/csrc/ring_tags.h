// Step tags of the words that workgroups of one launch exchange (narrow sparse
// loop, many-step dense loop): the workgroups that exchange with each other (a
// ring) share a base in device memory, read at the launch's start; step s of
// the launch uses tag base + s + 1, and the last workgroup of the ring to
// finish moves the base past them. So no word left by an earlier launch, nor
// by an earlier replay of the same captured launch, carries a tag that is
// waited for.
#pragma once

#include "sbqa_internal.h"

namespace sbqa {

// state: { base, workgroups finished } of the ring
__device__ __forceinline__ uint32_t ring_base(const uint32_t *state) {
    return __hip_atomic_load(const_cast<uint32_t *>(state), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// By one thread of each workgroup of the ring, once its last word is read.
__device__ __forceinline__ void ring_done(uint32_t *state, int members, uint32_t base, int steps) {
    const uint32_t n = __hip_atomic_fetch_add(state + 1, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (n + 1u == (uint32_t)members) {
        __hip_atomic_store(state + 1, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(state, base + (uint32_t)steps + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// One value and its tag in a word, stored and loaded coherently for the whole
// device (across the XCDs' L2 caches): a reader that sees the tag has the value.
__device__ __forceinline__ uint64_t tagged(uint32_t v, uint32_t tag) { return ((uint64_t)tag << 32) | v; }
__device__ __forceinline__ void put_word(uint64_t *p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t get_word(const uint64_t *p) {
    return __hip_atomic_load(const_cast<uint64_t *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// After a poll that found a word missing: whether the wave stops waiting.
// Bounded: on timeout the error word is set, and once it is set every later
// wait ends within 16 polls, so the grid always drains. A poll is 0.7 us or more,
// the bound 6 s: launches that could hold each other up are kept in order
// (launch_order.h) and none lasts a tenth of a second (MAX_EXCHANGE_STEPS), so only
// the kernels of others can keep a workgroup off the device for long.
constexpr int RING_POLL_LIMIT = 1 << 23;
__device__ __forceinline__ bool stop_waiting(int polls, int *err) {
    if ((polls & 15) == 15 && __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0) return true;
    if (polls > RING_POLL_LIMIT) {
        __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return true;
    }
    return false;
}

}  // namespace sbqa
