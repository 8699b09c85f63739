// N-plets of the device searches as two-word bit masks (N <= 128): variable i is bit i % 64 of word
// i / 64.
#pragma once

#include "thoi_internal.hpp"

namespace thoi {

struct Mask {
    uint64_t w[2];
};

__device__ __forceinline__ int popc(const Mask& m) { return __popcll(m.w[0]) + __popcll(m.w[1]); }

// Index of the (n+1)-th set bit of m counted from bit 0, or 0 when m has fewer set bits: six
// halvings of the word that holds it.
__device__ __forceinline__ int nth_set(const Mask& m, int n)
{
    const int c0 = __popcll(m.w[0]);
    const bool hi = n >= c0;
    uint64_t x = hi ? m.w[1] : m.w[0];
    n -= hi ? c0 : 0;
    if (n >= __popcll(x)) return 0;
    int pos = hi ? 64 : 0;
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) {
        const int c = __popcll(x & ((1ull << s) - 1ull));
        const bool up = n >= c;
        n -= up ? c : 0;
        x = up ? x >> s : x;
        pos += up ? s : 0;
    }
    return pos;
}

}  // namespace thoi
