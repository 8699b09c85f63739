// The subset-table engine's margin: where its filter (nplets_cube.hip) takes the table's word for an n-plet, and
// what the estimate of its open share (nplets_cube_gate.hip) goes by.
#pragma once

#include "nplets_fwd_common.hpp"

namespace thoi {
namespace {

constexpr double kFixMax = 63.5;        // |log det| of the fixed-point table's entries

// How far Omega and the VIFs of a factorisation per n-plet (FP32 or FP64) may be from the table's.  With E the
// perturbation of R_S that its rounding and its factorisation amount to, entries of at most eps,
// |R_S^-1|_ij <= sqrt(a_i a_j) gives |y' E y| <= rel y' R_S y for every y, with rel = eps (sum sqrt a)^2 <=
// eps k sum a.  So a_j moves by a factor between 1 / (1 + rel) and 1 / (1 - rel), whatever rel < 1 is, and to first
// order log det by rel and the sum of the log a_j by k rel.  From rel = 1/4 on nothing is certain but a VIF above a
// threshold: near 1 a factorisation may find a pivot that is not positive.
//  - FP64: a Cholesky factorisation and an inversion of order k have eps <= 2 (k + 1) u, u = 2^-53 (Higham, "Accuracy
//    and Stability of Numerical Algorithms", chapters 8 and 10), so Omega moves by at most (k + 1) (k + 2) u k sum a;
//    twice that is taken (the table's own values move as much) and costs nothing.
//  - FP32: the same bound would leave most n-plets open.  4 u k sum a is taken, u = 2^-24, which is an assumption:
//    the largest difference from FP64 that 25 systems of 26 variables showed (factor models, AR(1) of 0.5 to
//    0.999, near-duplicate channels, equal correlations, 28 to 60 samples; 20,000 n-plets of each order 3..24 with VIFs
//    up to 1000) is 0.15 u k sum a.
// To both comes the rounding of the measures and of the table's sum (k terms of up to |ld| = 2 |TC|, each addition
// to within u of a sum of up to k |ld|; fixed point: half a unit in each of up to 25 entries).
struct Margin {
    double rel;              // of log det, log a_j, and relative of a_j
    double round;
    int vif;                 // 0 below the refinement threshold (FP32), 1 nothing is certain, 2 above
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
        m.vif = v < tau * (1.0f - d) && rel < 0.25f ? 0 : (v > tau * (1.0f + d) ? 2 : 1);
    } else {
        m.rel = 2.0 * 1.1102230246251565e-16 * ((k + 1) * (k + 2) * k) * (double)ex;
        m.round = 4e-15 + 4.5e-16 * (double)(k * k);
        m.vif = m.rel < 0.25 ? 0 : 1;
    }
    return m;
}

}  // namespace
}  // namespace thoi
