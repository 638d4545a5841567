// A result handed from some workgroups of a launch to others of the same launch.
//
// A launch that waits for the one before costs 2.8 us on this chip before it does anything, 4 to 5 with its requests.  Where what is
// handed over is there long before it is needed, the launch that needs it can form it on the side.
//
//   data     written and read past the caches of one XCD (sc1: agent scope), since the eight XCDs' L2s are not kept equal within a
//            launch.  A writer waits until memory has acknowledged its stores (stores_done) before it says so.  Fences of that scope
//            would write back or drop a whole L2 instead.
//   pairs    one word for two that need each other's part: the one that comes first leaves the call's tag there and is done, the one that
//            finds the tag does what is left.  Nobody has to wait, so nothing depends on which workgroups run at the same time.  The tag
//            is the call's own 64 bits, so whatever the word holds before does no harm (a counter would want cleared memory, i.e. a
//            launch in front).  Whoever finds the tag clears the word: a captured launch, whose tag is the same on every
//            replay, starts from clear words.
//   knockout of many: in pairs, the one that finds the tag goes on to the next round.
// At the end of a launch sums of a split contraction handed over so were no faster than a launch that adds them up: under load a store's
// acknowledgement, an exchange and a load are 1 us each, one after the other (16 x 4096 x 14336 in two slices 23.2 to 24.5 us a call so, 23.9
// with the launch; 16 x 14336 x 4096 up to 33 so, 24.4 with it).
// Beside something longer they cost nothing (the backward pass's gradients).
#pragma once

#include "salr_device.hpp"
#include "salr_row_stream.hpp"

namespace salr {

constexpr int kAgentScope = 16;   // cache policy of the raw buffer accesses: sc1

__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

__device__ __forceinline__ u32x4 shared_load4(Buffer b, uint32_t offset) {
    return __builtin_amdgcn_raw_buffer_load_b128(b, (int)offset, 0, kAgentScope);
}
__device__ __forceinline__ u32x4 shared_load4(const void* p) {   // (where 32-bit offsets do not reach)
    u32x4 v;
    const uint64_t* q = static_cast<const uint64_t*>(p);
    const uint64_t lo = __hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), hi = __hip_atomic_load(q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    v[0] = (uint32_t)lo; v[1] = (uint32_t)(lo >> 32); v[2] = (uint32_t)hi; v[3] = (uint32_t)(hi >> 32);
    return v;
}
__device__ __forceinline__ void shared_store4(Buffer b, uint32_t offset, u32x4 v) {
    __builtin_amdgcn_raw_buffer_store_b128(v, b, (int)offset, 0, kAgentScope);
}
__device__ __forceinline__ void shared_store2(Buffer b, uint32_t offset, u32x2 v) {
    __builtin_amdgcn_raw_buffer_store_b64(v, b, (int)offset, 0, kAgentScope);
}

__device__ __forceinline__ uint64_t look_at(const uint64_t* word) {
    return __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void leave_clear(uint64_t* word) {
    __hip_atomic_store(word, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// One of a pair arrives: true for the second.
__device__ __forceinline__ bool meet(uint64_t* word, uint64_t tag) {
    if (__hip_atomic_exchange(word, tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != tag) return false;
    leave_clear(word);
    return true;
}
// Number `i` of `n` arrives (one lane): true for the last.  words[1 .. n - 1] are the pairs'.
__device__ __forceinline__ bool knockout(uint64_t* words, int i, int n, uint64_t tag) {
    for (int round = 0; (1 << round) < n; ++round) {
        if ((((i >> round) ^ 1) << round) >= n) continue;   // nobody on the other side
        if (!meet(words + (((i >> round) | 1) << round), tag)) return false;
    }
    return true;
}

}  // namespace salr
