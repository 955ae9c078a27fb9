// Block order and wave-level helpers shared by the kernels (FFT passes, deposit sort, friends-of-friends).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace cola {

// Block b runs on XCD b % 8 (round-robin dispatch); hand each XCD a contiguous run of the grid's blocks
// (along x), so that neighbouring blocks, which share cache lines -- the 128-byte lines of narrow FFT tiles, the
// cells and mesh lines around neighbouring particles -- meet in the same L2.
__device__ __forceinline__ int xcd_block() {
    const int nb = gridDim.x, b = blockIdx.x;
    const int q = nb >> 3, r = nb & 7, x = b & 7, i = b >> 3;
    return (x < r) ? x * (q + 1) + i : r * (q + 1) + (x - r) * q + i;
}

// Increment for items in no order, whose keys lanes of a wave may share without being neighbours: the keys of up to
// sixteen lanes, each held by another one at least, take one atomic each, every other lane its own, and all
// are in flight together; three lanes whose key none shares end the search.
__device__ __forceinline__ uint32_t wave_increment_shared(uint32_t* counter_base, uint32_t key, unsigned long long left) {
    constexpr int kKeys = 16;
    const int lane = __lane_id();
    const unsigned long long below = (1ull << lane) - 1ull;
    unsigned long long cold = 0ull;
    uint32_t add = left >> lane & 1ull ? 1u : 0u;  // of this lane's atomic
    int from = lane;                               // the lane whose atomic counts this one
    uint32_t rank = 0;
#pragma unroll
    for (int t = 0; t < kKeys; ++t) {
        const unsigned long long c = left & ~cold;
        if (!c || __popcll(cold) > 2) continue;
        const int lead = __ffsll((long long)c) - 1;
        const unsigned long long m = __ballot(key == (uint32_t)__builtin_amdgcn_readlane((int)key, lead)) & left;
        if (__popcll(m) < 2) {
            cold |= 1ull << lead;
            continue;
        }
        left &= ~m;
        if (m >> lane & 1ull) {
            add = lane == lead ? (uint32_t)__popcll(m) : 0u;
            from = lead;
            rank = (uint32_t)__popcll(m & below);
        }
    }
    uint32_t base = 0;
    if (add) base = atomicAdd(&counter_base[key], add);
    return (uint32_t)__shfl((int)base, from) + rank;
}

// Wave-aggregated atomic increment by runs: consecutive lanes with equal keys share one atomic,
// and every run of the wave issues its atomic at once (one memory round trip per wave; particles
// in Lagrangian order give a few runs per wave).  Returns the old counter value plus the lane's
// rank in its run; equal keys in separate runs take separate slot ranges.
//
// ANY_ORDER: a wave of more than 32 runs looks for shared keys.  Atomics on one line of counters pass at about one
// in 3 ns: 1e6 points within 3 cells of one point, 250^3 cells, 2994 -> 497 us; no difference where keys are spread.
template <bool ANY_ORDER = false>
__device__ __forceinline__ uint32_t wave_increment(uint32_t* counter_base, uint32_t key, bool valid) {
    const int lane = __lane_id();
    const uint32_t prev_key = __shfl_up(key, 1);
    const int prev_valid = __shfl_up(valid ? 1 : 0, 1);
    const bool head = valid && (lane == 0 || prev_valid == 0 || prev_key != key);
    const unsigned long long hm = __ballot(head), vm = __ballot(valid);
    if (ANY_ORDER && __popcll(hm) > 32) return wave_increment_shared(counter_base, key, vm);
    const unsigned long long upto = lane == 63 ? ~0ull : ((2ull << lane) - 1ull);  // lanes 0..lane
    uint32_t base = 0;
    if (head) {
        const unsigned long long brk = (hm | ~vm) & ~upto;  // where the runs after this lane start
        const int next = brk ? __ffsll((long long)brk) - 1 : 64;
        base = atomicAdd(&counter_base[key], (uint32_t)(next - lane));
    }
    const unsigned long long mine = hm & upto;
    const int my_head = mine ? 63 - __clzll((long long)mine) : lane;
    return __shfl(base, my_head) + (uint32_t)(lane - my_head);
}

}  // namespace cola
