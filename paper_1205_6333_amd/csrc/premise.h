// premise.h -- counting of the pairs that break the premise r >= 2a of Eq. 4
// (sd_premise_counts), for the kernels that evaluate near pairs themselves.
#pragma once

#include "pair_terms.h"

namespace sd {

// The current device's counters, [0] pairs with 0 < r < 2a, [1] with r = 0
// (defined beside the product kernels in mobility.hip).
hipError_t premise_counters(unsigned long long** counters);

// Called by the lanes active at that point, each with the class of its pair
// (PREMISE_OK for none): one atomic add per class and call, by one lane, for
// the whole wave (a dense suspension meets thousands of such pairs per
// product, and atomics on one address serialise).
__device__ __forceinline__ void count_premise(unsigned long long* counters, int cls)
{
    const uint64_t sub = __builtin_amdgcn_ballot_w64(cls == PREMISE_SUB2A);
    const uint64_t co = __builtin_amdgcn_ballot_w64(cls == PREMISE_COINCIDENT);
    if ((sub | co) == 0) return;
    const uint64_t act = __builtin_amdgcn_ballot_w64(true);
    if ((int)(threadIdx.x & 63) != __builtin_ctzll(act)) return;
    if (sub) atomicAdd(&counters[0], (unsigned long long)__builtin_popcountll(sub));
    if (co) atomicAdd(&counters[1], (unsigned long long)__builtin_popcountll(co));
}

}  // namespace sd
