// Pieces of the permutation shared by its own kernels (moe_permute.hip) and by the router that places its rows itself
// (moe_route.hip).
#pragma once

#include "moe_internal.h"

namespace moe {

__device__ __forceinline__ int lanes_below(uint64_t mask, int lane) {
    return __popcll(mask & ((1ull << lane) - 1ull));
}

// lanes of the wavefront with the same id as this one (0: this lane's id is not an expert); only as many ballots as the
// number of experts has bits (300000 ids of a single expert: 31.7 us with six, 30.4 with none)
__device__ __forceinline__ uint64_t same_expert(int id, int E) {
    const bool valid = id >= 0 && id < E;
    uint64_t m = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 6; ++b) {
        if ((E - 1) >> b == 0) break;
        const bool bit = (id >> b) & 1;
        const uint64_t set = __ballot(bit);
        m &= bit ? set : ~set;
    }
    return valid ? m : 0;
}
static_assert(MOE_MAX_EXPERTS == 64, "an expert id has six bits");

}  // namespace moe
