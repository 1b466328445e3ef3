// Decoupled look-back: the exclusive prefix of the workgroups' counts within
// one launch.  A workgroup publishes its count and finds its place by looking
// over the workgroups before it: one wave reads 64 predecessors' states at a
// time, each {empty, count, or count of everything up to it}, and adds counts
// until it meets a sum.
//
// The states have to be empty when a launch begins: launches alternate
// between two arrays (the parity of a launch count kept on the device, so
// that a replayed graph alternates too), and each clears what the one before
// it filled.  A workgroup waits only for workgroups of smaller number, and
// takes its number from a counter when it starts running, so the smallest
// number still at work never waits and every wait ends.  That counter serves
// one workgroup per 12 ns, so a launch wants few, large workgroups.
#pragma once

#include "hough_internal.h"

namespace hough {

// entries of the counters, the first in a cache line of its own
constexpr uint32_t kNumber = 0, kLaunches = 32, kLastGrid = 33;
static_assert(kPeakCounterBase + kLastGrid < kCounterDwords, "peak counters fit the counter array");

constexpr uint64_t kStateCount = uint64_t(1) << 62, kStateSum = uint64_t(2) << 62, kStateValue = kStateCount - 1;

__device__ __forceinline__ uint64_t state_load(const uint64_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint32_t load_counter(const uint32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void state_store(uint64_t *p, uint64_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Sum of the counts of workgroups 0 .. w - 1, by one wave (uniform result).
__device__ __forceinline__ uint64_t look_back(const uint64_t *state, uint32_t w, uint32_t lane)
{
    uint64_t sum = 0;
    for (int64_t top = int64_t(w) - 1; top >= 0; top -= 64) {
        const int64_t i = top - int64_t(lane);
        uint64_t v, sums;
        for (;;) {
            v = i >= 0 ? state_load(state + i) : kStateSum;      // before the first: the sum 0
            sums = __ballot((v & kStateSum) != 0);
            // the lanes up to the nearest sum have to be filled
            const uint64_t need = sums ? (sums & (~sums + 1)) - 1 : ~uint64_t(0);
            if ((__ballot(v == 0) & need) == 0) break;
            __builtin_amdgcn_s_sleep(1);
        }
        const uint32_t last = sums ? uint32_t(__builtin_ctzll(sums)) : 63u;
        uint64_t x = lane <= last ? v & kStateValue : 0u;
        for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
        sum += x;
        if (sums) break;
    }
    return sum;
}

// This workgroup's number (by all threads, with a barrier); `state` receives
// the launch's state array.  join: two dwords of LDS.
__device__ __forceinline__ uint32_t look_back_join(uint64_t *states, uint64_t n_states, uint32_t *counters,
                                                   uint32_t *join, uint64_t *&state)
{
    if (threadIdx.x == 0) {
        const uint32_t number = atomicAdd(counters + kNumber, 1u);
        const uint32_t parity = load_counter(counters + kLaunches) & 1u, filled = load_counter(counters + kLastGrid);
        uint64_t *other = states + (parity ? 0 : n_states);
        for (uint64_t i = number; i < filled; i += gridDim.x) state_store(other + i, 0);
        join[0] = number;
        join[1] = parity;
    }
    __syncthreads();
    state = states + (__builtin_amdgcn_readfirstlane(join[1]) ? n_states : 0);
    return __builtin_amdgcn_readfirstlane(join[0]);
}

// Publishes the workgroup's count and returns the sum of those before it
// (one wave, uniform).
__device__ __forceinline__ uint64_t look_back_place(uint64_t *state, uint32_t *counters, uint32_t number,
                                                    uint64_t count, uint32_t lane)
{
    if (lane == 0 && number > 0) state_store(state + number, kStateCount | count);
    const uint64_t sum = look_back(state, number, lane);
    if (lane == 0) {
        state_store(state + number, kStateSum | (sum + count));
        // the last number's sum means that every workgroup has filled its
        // state, and so has read the counters
        if (number == gridDim.x - 1) {
            counters[kNumber] = 0;
            counters[kLaunches] += 1;
            counters[kLastGrid] = gridDim.x;
        }
    }
    return sum;
}

}  // namespace hough
