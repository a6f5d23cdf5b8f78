// premise.h -- counting of the pairs that break the premise r >= 2a of Eq. 4
// (sd_premise_counts), for the kernels that evaluate near pairs themselves.
#pragma once

#include "pair_terms.h"

namespace sd {

// The current device's counters (defined beside the product kernels in
// mobility.hip): PREMISE_SLOTS slots of 64 bytes, each [0] pairs with 0 < r < 2a and
// [1] with r = 0, to be added up.  Work-groups take the slots in turn, since atomics
// on one address serialise: microseconds with one slot -> this: products of N =
// 3000 with 0.6 near partners per particle 18.6 -> 14.9 (5000 30.5 -> 27.8), the
// fold of N = 65536 with 0.4 85 -> 73.
constexpr int PREMISE_SLOTS = 256, PREMISE_STRIDE = 8;
hipError_t premise_counters(unsigned long long** counters);

__device__ __forceinline__ void add_premise(unsigned long long* counters, uint32_t sub,
                                            uint32_t co)
{
    unsigned long long* const c = counters + (blockIdx.x % PREMISE_SLOTS) * PREMISE_STRIDE;
    if (sub) atomicAdd(&c[0], (unsigned long long)sub);
    if (co) atomicAdd(&c[1], (unsigned long long)co);
}

// Called by the lanes active at that point, each with the class of its pair
// (PREMISE_OK for none): one atomic add per class and call, by one lane, for
// the whole wave.
__device__ __forceinline__ void count_premise(unsigned long long* counters, int cls)
{
    const uint64_t sub = __builtin_amdgcn_ballot_w64(cls == PREMISE_SUB2A);
    const uint64_t co = __builtin_amdgcn_ballot_w64(cls == PREMISE_COINCIDENT);
    if ((sub | co) == 0) return;
    const uint64_t act = __builtin_amdgcn_ballot_w64(true);
    if ((int)(threadIdx.x & 63) != __builtin_ctzll(act)) return;
    add_premise(counters, __builtin_popcountll(sub), __builtin_popcountll(co));
}

}  // namespace sd
