// The subset-table engine's margin: where its filter (nplets_cube.hip) takes the table's word for an n-plet, and
// what the estimate of its open share (nplets_cube_gate.hip) goes by.
#pragma once

#include "nplets_fwd_common.hpp"

namespace thoi {
namespace {

constexpr double kFixMax = 63.5;        // |log det| of the fixed-point table's entries

// How far Omega and the VIFs of a factorisation per n-plet (FP32 or FP64) may be from the table's.  With
// E the perturbation of R_S by rounding it and factoring it (entries of a few units u = 2^-24 or 2^-53),
// log det moves by tr(R_S^-1 E) and log a_j by (R_S^-1 E R_S^-1)_jj / a_j, to first order; |R_S^-1|_ij
// <= sqrt(a_i a_j), so both are at most |E| (sum sqrt a)^2 <= |E| k sum a.  Taken: 4 u k sum_j a_j in FP32
// (about 200 times what the engines differ by on the test systems) and 64 u k sum_j a_j in FP64, where a
// wide margin costs nothing, plus the rounding of the measures and of the table's sum (k terms of up to
// |ld| = 2 |TC|, each addition to within u of a sum of up to k |ld|; fixed point: half a unit in each of up
// to 25 entries).
struct Margin {
    double rel;              // of log det, log a_j, and relative of a_j
    double round;
    int vif;                 // FP32: 0 below the refinement threshold, 1 may be on either side, 2 above
    __device__ __forceinline__ double value(double TC, double DTC) const
    {
        return rel + round * (fabs(TC) + fabs(DTC) + 1.0);
    }
};
template <bool F32>
__device__ __forceinline__ Margin margin_of(int k, double ld, float mx, float ex, float tau)
{
    Margin m;
    if constexpr (F32) {
        const float rel = 4.0f * 5.9604645e-8f * (float)k * ex;
        const float v = __builtin_amdgcn_exp2f(mx * 1.442695041f), d = rel + 1e-5f + 2e-6f * fabsf((float)ld);
        m.rel = (double)rel + 4e-7;
        m.round = 2.4e-7;
        m.vif = !(v * (1.0f + d) < tau) ? (v > tau * (1.0f + d) ? 2 : 1) : 0;
        if (!(rel < 0.25f)) m.vif = m.vif == 0 ? 1 : m.vif;
    } else {
        m.rel = 64.0 * 1.1102230246251565e-16 * k * (double)ex;
        m.round = 4e-15 + 4.5e-16 * (double)(k * k);
        m.vif = 0;
    }
    return m;
}

}  // namespace
}  // namespace thoi
