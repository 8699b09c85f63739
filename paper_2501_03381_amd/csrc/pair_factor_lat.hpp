// The pair factorisation (two n-plets per wavefront, rows in registers) for kernels with about one wave
// per SIMD, the searches: the same operations on each entry in the same order as pair_factor, so the
// same results bit for bit, arranged for latency instead of registers.
//
// pair_factor runs two loops of k dependent steps (Cholesky, then inversion), waits for each group of
// four columns by itself, and reads every entry under its own lane condition.  Here one loop does
// both, a step's reads go out together, the pivot is read from its lane (not through LDS), and the
// gather is unconditional.  1024 annealing chains at order 20 (N = 100): 22,500 cycles per iteration,
// 200 iterations in 2.4 ms; one launch per iteration with pair_factor took 6.2 ms.
#pragma once

#include "pair_factor.hpp"

namespace thoi {

// Pointers that keep their address space across a call.
typedef __attribute__((address_space(3))) double* LdsDouble;
typedef __attribute__((address_space(3))) int* LdsInt;
typedef const __attribute__((address_space(1))) double* GlobalDouble;

// Where a factorisation reads its entries (i, j), j <= i, scaled by 1/sqrt(Sigma_ii Sigma_jj): the
// covariance in global memory (each half may have its own dataset), or the covariance's lower
// triangle packed by rows in LDS with 1/sqrt(Sigma_jj) beside it.
enum class PairSource { Global, Lower };

__device__ __forceinline__ double inv_sd(double d) { return d > 0.0 ? 1.0 / sqrt(d) : __builtin_nan(""); }

// Lane j (< 32) of each half-wave's x.
__device__ __forceinline__ double half_lane(double x, int j)
{
    const long long u = __double_as_longlong(x);
    const int lo = (int)u, hi = (int)(u >> 32);
    const bool up = (threadIdx.x & 32) != 0;
    const int l0 = __builtin_amdgcn_readlane(lo, j), l1 = __builtin_amdgcn_readlane(lo, 32 + j);
    const int h0 = __builtin_amdgcn_readlane(hi, j), h1 = __builtin_amdgcn_readlane(hi, 32 + j);
    const int l = up ? l1 : l0, h = up ? h1 : h0;
    return __longlong_as_double(((long long)h << 32) | (uint32_t)l);
}

// The value is computed by here (no instruction; the host pass has no vector registers).
template <typename V>
__device__ __forceinline__ void pin_reg(V& x)
{
#ifdef __HIP_DEVICE_COMPILE__
    asm volatile("" : "+v"(x));
#endif
}

// One pass over the pivots of the half-waves' blocks (rows in r, see pair_factor), k <= KM: the pivot
// of this lane's row in piv and the squared norm of its column of W = L^-1 in aj.
//
// Right-looking Cholesky and inversion together.  Step j publishes column j of the Schur complement
// (lane i: a_ij) and lane j's running row sums s_m = sum_t L_jt W_tm (m < j), so that after one
// exchange every lane has L_ij = a_ij / sqrt(p) and row j of W (W_jm = -s_m / sqrt(p), W_jj =
// 1 / sqrt(p)): it updates its Schur entries m > j and adds L_ij W_jm to its own row sums m <= j, which
// take the registers of the consumed columns.  Lane i's entries r[m] with m > i, every entry of a
// lane whose row is published, and every entry of a lane beyond the order are never read for the
// result; the updates run on them too, so that the inner loops need no per-lane condition (LDS
// entries beyond the order are stale but in bounds).
template <int KM>
__device__ __forceinline__ void pair_pivots_lat(double (&r)[kW2Max], int k, int kh, int i, LdsDouble __restrict__ col,
                                                LdsDouble __restrict__ wrow, double& piv, double& aj)
{
    sfor<0, KM>([&](auto J) {
        constexpr int j = J;
        if (j < k) {
            const LdsDouble cl = col + (j & 1) * kW2Max;
            const LdsDouble wr = wrow + (j & 1) * kW2Max;
            cl[i] = r[j];                                 // a_ij of the current Schur complement
            if (i == j) {
                sfor<0, j>([&](auto M) {
                    constexpr int m = M;
                    wr[m] = r[m];
                });
            }
            wave_sync();
            const double p = half_lane(r[j], j);          // not through LDS: rsqrt overlaps the exchange
            double c[KM], wi = 0.0;
            sfor<j + 1, KM>([&](auto M) { c[M] = cl[M]; });
            sfor<0, j>([&](auto M) { c[M] = wr[M]; });
            if constexpr (j > 0) {
                wi = wr[i < j ? i : 0];
                pin_reg(wi);                              // a load of every lane, not under i < j
            }
            const double rs = rsqrt(p);
            const double aij = r[j];
            const double t = aij * rs * rs;               // a_ij / a_jj
            const double lit = aij * rs;                  // L_ij
            piv = i == j ? p : piv;
            sfor<j + 1, KM>([&](auto M) { r[M] -= t * c[M]; });
            const double w = i < j ? -wi * rs : rs;       // W_ji: column norms accumulate in aj
            aj += (i <= j && j < kh) ? w * w : 0.0;      // rows of this half's own n-plet only
            sfor<0, j>([&](auto M) {
                constexpr int m = M;
                const double wm = -c[m] * rs;
                r[m] += lit * wm;
            });
            r[j] = lit * rs;
            // keep each step's updates in the step: sunk to their uses, they hold the step's LDS
            // values in registers for many steps
            sfor<0, KM>([&](auto M) { pin_reg(r[M]); });
        }
    });
}

// Row `ci` of the block, entries m < i (and the unit diagonal) into r: all loads of a group of KG
// columns are issued before any is used, none of them under a condition (5,700 cycles at order 20
// when each waits for the one before it, 2,900 so); r[] is indexed by constants only.
template <PairSource SRC, int KM, int KG, typename SP>
__device__ __forceinline__ void pair_gather_lat(double (&r)[kW2Max], SP __restrict__ sR, int N,
                                                LdsInt __restrict__ cidx, int k, int kh, int i, int ci, double si,
                                                LdsDouble __restrict__ wrow)
{
    const bool mine = i < kh;
    sfor<0, kW2Max>([&](auto M) {
        constexpr int m = M;
        r[m] = (m == i && mine) ? 1.0 : 0.0;
    });
    sfor<0, KM / KG>([&](auto G) {
        constexpr int g = G;
        if (KG * g < k) {
            int cm[KG];
            double e[KG], sc[KG];
            sfor<0, KG>([&](auto U) { cm[U] = cidx[KG * g + U]; });
            sfor<0, KG>([&](auto U) {
                if constexpr (SRC == PairSource::Global) e[U] = sR[(int64_t)ci * N + cm[U]];
                else e[U] = sR[ci * (ci + 1) / 2 + (cm[U] < ci ? cm[U] : ci)];
            });
            sfor<0, KG>([&](auto U) { sc[U] = wrow[KG * g + U]; });
            sfor<0, KG>([&](auto U) {
                constexpr int u = U, m = KG * g + u;
                e[u] *= si * sc[u];
                pin_reg(e[u]);                            // the loads stay together, outside the condition
                if (m < i && mine) r[m] = e[u];
            });
        }
    });
}

// One class of pair_factor_lat (k <= KM).  A call, not inlined: four classes in one function, inside
// a loop over iterations, made the compiler hold 256 registers and spill.
template <PairSource SRC, bool SEQ, int KM, typename SP>
__device__ __attribute__((noinline)) FactorOut<double> pair_factor_class(SP sR, int N, LdsInt cidx, int k_in, int kh,
                                                                         LdsDouble col, LdsDouble wrow, LdsDouble isd)
{
    const int k = __builtin_amdgcn_readfirstlane(k_in);   // uniform: scalar loop guards
    const int i = threadIdx.x & 31;
    const bool mine = i < kh;
    if (!mine) cidx[i] = 0;
    wave_sync();
    const int ci = cidx[i];
    double r[kW2Max];
    // lane i scales its row by 1/sqrt(Sigma_ii) and publishes the factor for the columns
    double si;
    if constexpr (SRC == PairSource::Global) si = inv_sd(sR[(int64_t)ci * N + ci]);
    else si = isd[ci];
    wrow[i] = si;
    wave_sync();
    pair_gather_lat<SRC, KM, SRC == PairSource::Lower ? 8 : 4>(r, sR, N, cidx, k, kh, i, ci, si, wrow);
    wave_sync();                                          // wrow is reused below
    double piv = 1.0;
    double aj = 0.0;
    pair_pivots_lat<KM>(r, k, kh, i, col, wrow, piv, aj);
    FactorOut<double> o;
    if constexpr (SEQ) {
        wave_sync();                                      // every lane has read its last W row
        wrow[i] = mine ? log(piv) : 0.0;
        wrow[kW2Max + i] = mine ? log(aj) : 0.0;
        wave_sync();
        double s1 = 0.0, s2 = 0.0;
        if (i == 0) {
            for (int m = 0; m < kh; ++m) { s1 += wrow[m]; s2 += wrow[kW2Max + m]; }
        }
        o.ld = __shfl(s1, 0, 32);
        o.sa = __shfl(s2, 0, 32);
    } else {
        o.ld = half_sum(mine ? log(piv) : 0.0);
        o.sa = half_sum(mine ? log(aj) : 0.0);
    }
    o.vmax = half_max(mine ? aj : 0.0);
    o.ok = half_sum((mine && !(piv > 0.0)) ? 1.0 : 0.0) == 0.0;
    wave_sync();
    return o;
}

// pair_factor for the half-wave's n-plet cidx[0..kh-1], by the class of the wavefront's order k (up to
// 8, 16, 24 or 32).  cidx holds 32 entries per half; those beyond the order are cleared.  sR: Sigma in
// global memory, or its packed lower triangle in LDS with isd[j] = 1/sqrt(Sigma_jj).
template <PairSource SRC, bool SEQ = false>
__device__ __forceinline__ FactorOut<double> pair_factor_lat(const double* sR, int N, int* cidx, int k, int kh,
                                                             double* col, double* wrow, double* isd = nullptr)
{
    const LdsDouble c = (LdsDouble)col, w = (LdsDouble)wrow, q = (LdsDouble)isd;
    const LdsInt x = (LdsInt)cidx;
    const int ku = __builtin_amdgcn_readfirstlane(k);
    if constexpr (SRC == PairSource::Global) {
        const GlobalDouble sr = (GlobalDouble)sR;
        if (ku <= 8) return pair_factor_class<SRC, SEQ, 8>(sr, N, x, ku, kh, c, w, q);
        if (ku <= 16) return pair_factor_class<SRC, SEQ, 16>(sr, N, x, ku, kh, c, w, q);
        if (ku <= 24) return pair_factor_class<SRC, SEQ, 24>(sr, N, x, ku, kh, c, w, q);
        return pair_factor_class<SRC, SEQ, kW2Max>(sr, N, x, ku, kh, c, w, q);
    } else {
        const LdsDouble sr = (LdsDouble)sR;
        if (ku <= 8) return pair_factor_class<SRC, SEQ, 8>(sr, N, x, ku, kh, c, w, q);
        if (ku <= 16) return pair_factor_class<SRC, SEQ, 16>(sr, N, x, ku, kh, c, w, q);
        if (ku <= 24) return pair_factor_class<SRC, SEQ, 24>(sr, N, x, ku, kh, c, w, q);
        return pair_factor_class<SRC, SEQ, kW2Max>(sr, N, x, ku, kh, c, w, q);
    }
}

}  // namespace thoi
