// One pass of a radix selection in LDS, shared by the selections of the reducer, the cube engine's
// bounds and the device greedy.
#pragma once

#include "thoi_internal.hpp"

namespace thoi {

// First wavefront of the workgroup (lane = threadIdx.x < 64), all lanes: rh[256] counts the entries that
// match the prefix so far by their next 8 bits; the bin in which the running count reaches `rank` is
// appended to the prefix, and rank becomes the rank inside that bin.  The counts reach the rank.
__device__ __forceinline__ void radix_pick(const uint32_t* rh, int lane, int pass, uint32_t& prefix, int& rank)
{
    // lane t sums bins 4t .. 4t+3; the lane whose running sum first reaches the rank picks
    uint32_t v[4], own = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) { v[u] = rh[4 * lane + u]; own += v[u]; }
    uint32_t incl = own;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) { const uint32_t y = __shfl_up(incl, o, 64); incl += lane >= o ? y : 0u; }
    const uint32_t r = (uint32_t)rank;
    const uint64_t m = __ballot(incl >= r);
    if (lane == __builtin_ctzll(m)) {
        uint32_t before = incl - own;
        int u = 0;
        while (u < 3 && before + v[u] < r) before += v[u++];
        prefix |= (uint32_t)(4 * lane + u) << (8 * pass);
        rank = (int)(r - before);
    }
}

// Whether the upper key word h matches the prefix in the bits above `pass`.
__device__ __forceinline__ bool radix_match(uint32_t h, uint32_t prefix, int pass)
{
    return pass == 3 || (h >> (8 * (pass + 1))) == (prefix >> (8 * (pass + 1)));
}

}  // namespace thoi
