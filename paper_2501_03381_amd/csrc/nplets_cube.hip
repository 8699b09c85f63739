// Subset-table ("cube") engine: streaming reductions over whole orders of many variables (FP64: 21..30,
// FP32 with refinement: 26..30).
//
// An exhaustive enumeration meets every subset of S as an n-plet of its own, so the leave-one-out
// determinants need no inverse: with ld(S) = log det R_S in a table over all 2^N subsets,
//   log a_j = log (R_S^-1)_jj = ld(S \ j) - ld(S)
// (the cofactor identity), and an n-plet costs one pivot and k table reads instead of a factorisation
// and an inversion of order k ("The combinatorial explosion": the number of subsets stays, the k^3
// per subset goes).  A reduction needs the value itself of few n-plets, so the table only filters: an
// n-plet whose bin is certain and which cannot enter a list is counted, the rest ("open") is evaluated
// as the lane and pair engines do (nplets_cube_verify.hip).  The results are theirs bit for bit: in
// FP64 by an error bound, in FP32 as far as an evaluation errs by no more than its margin assumes
// (nplets_cube_margin.hpp).  Covariances that would leave most n-plets open are given back to the
// factorisation by a look at a sample of them (FP32; nplets_cube_gate.hip).
//
// A subset is a prefix P (of the first h = N - 10 variables) and one of the 1024 subsets of the last
// ten; row P of the table holds the latter ordered by size and, within a size, lexicographically.
//  - k_cube_build, one wavefront per row: the prefix is eliminated from the matrix of P and the ten
//    variables (right-looking, one matrix row per lane), then every lane eliminates its subset of the
//    first six variables from its own copy of the 10 x 10 Schur complement and walks the 16 subsets
//    of the last four.  ld of a subset is ld of the subset without its last variable plus the log of
//    the pivot.
//  - k_cube_filter, one wavefront per (row, size): the n-plets P + (subsets of one size) have
//    consecutive global indices and read consecutive entries of the rows of P without one member;
//    removing one of the ten variables stays inside the row (a table of neighbours in LDS).
// Bound by VALU issue (the build: logarithms and eliminations in FP64; the filter, 57% busy) and the
// latency of the table reads (k + 1 per n-plet).  A factorisation per n-plet against the table, top-100 and
// 256 bins, orders 3..N, one dataset, ms:
//   FP32 + refinement  N = 26  3.80 / 1.97   27  7.34 / 3.60   28  14.6 / 6.80   29  30.3 / 13.4
//                      N = 30  65.4 / 27.6 (build 6.1, filter 22, open n-plets beside it)
//   FP64               N = 22  1.11 / 0.43   27  23.4 / 3.88   30  444 / 33.6
//                      N = 25  4.37 / 1.17 (build 0.20, bounds 0.09, filter 0.61, open n-plets 0.2, merge 0.06)
// Without bounds of the small orders (their lists open on every n-plet) N = 25 took 1.60 ms, and with an
// exponential per table read no more and no less.
// Taking the table's values themselves (no second evaluation) measured 1.05 ms at N = 25, with errors
// against 64-bit references of 1e-14 instead of 2e-15.
#include "nplets_cube.hpp"
#include "nplets_cube_margin.hpp"
#include "radix_pick.hpp"

#include <cmath>

namespace thoi {
namespace {

constexpr int kBuildThreads = 256;                    // four rows
constexpr int kBuildWaves = kBuildThreads / 64;
constexpr int kBuildRows = 4;                         // rows per wavefront (one staging of the matrix)
constexpr int kCubePrefix = kCubeMaxN - kCubeSuffix;  // largest prefix (20)
constexpr int kTri10 = kCubeSuffix * (kCubeSuffix + 1) / 2;

// Subsets of {0..9} as masks, by size and lexicographically inside a size; their positions; the first
// position of each size; and for entry i of size b, at nbr[noff[b] + t * C(10, b) + i - off[b]], the
// position of the subset without its t-th element (ascending).
struct SuffixTable {
    uint16_t mask[kCubeRow];
    uint16_t pos[kCubeRow];
    uint16_t off[kCubeSuffix + 2];
    uint16_t noff[kCubeSuffix + 2];
    uint16_t nbr[kCubeSuffix * kCubeRow / 2];
};
constexpr SuffixTable make_suffix()
{
    SuffixTable t{};
    int n = 0;
    for (int b = 0; b <= kCubeSuffix; ++b) {
        t.off[b] = (uint16_t)n;
        // lexicographic order of ascending tuples = descending order of the bit-reversed masks
        for (int v = kCubeRow - 1; v >= 0; --v) {
            int m = 0, c = 0;
            for (int i = 0; i < kCubeSuffix; ++i)
                if ((v >> (kCubeSuffix - 1 - i)) & 1) { m |= 1 << i; ++c; }
            if (c == b) {
                t.mask[n] = (uint16_t)m;
                t.pos[m] = (uint16_t)n;
                ++n;
            }
        }
    }
    t.off[kCubeSuffix + 1] = (uint16_t)n;
    int o = 0;
    for (int b = 0; b <= kCubeSuffix; ++b) {
        t.noff[b] = (uint16_t)o;
        const int len = t.off[b + 1] - t.off[b];
        for (int e = 0; e < b; ++e)
            for (int i = 0; i < len; ++i) {
                int m = t.mask[t.off[b] + i], seen = 0, bit = 0;
                for (int v = 0; v < kCubeSuffix; ++v)
                    if ((m >> v) & 1) {
                        if (seen == e) bit = 1 << v;
                        ++seen;
                    }
                t.nbr[o++] = t.pos[m & ~bit];
            }
    }
    t.noff[kCubeSuffix + 1] = (uint16_t)o;
    return t;
}
constexpr SuffixTable kSuffixHost = make_suffix();
__device__ constexpr SuffixTable kSuffix = make_suffix();

__device__ __forceinline__ void cube_wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Entries of the table.  FP64: the value.  FP32: the filter's margin is a thousand times an FP32 rounding,
// so the value in fixed point, 2^-25 each (half the bytes, exact sums); kFixBad: not positive definite
// or below -64.
constexpr double kFixScale = 33554432.0;                // 2^25 (values inside +-kFixMax)
constexpr int32_t kFixBad = 0x7fffffff;
template <bool F32>
struct TableOf { typedef double T; };
template <>
struct TableOf<true> { typedef int32_t T; };
template <bool F32>
using Tab = typename TableOf<F32>::T;

__device__ __forceinline__ void encode(double ld, double& e) { e = ld; }
__device__ __forceinline__ void encode(double ld, int32_t& e)
{
    e = ld > -kFixMax && ld < kFixMax ? __double2int_rn(ld * kFixScale) : kFixBad;
}
__device__ __forceinline__ double decode(double e) { return e; }
__device__ __forceinline__ double decode(int32_t e) { return e == kFixBad ? __builtin_nan("") : (double)e * (1.0 / kFixScale); }

// 1/x, two Newton steps on the hardware estimate for the last bit or so, one (about 1e-14) for the fixed
// point table; the caller tests x.
template <bool F32>
__device__ __forceinline__ double fast_rcp(double x)
{
    double y = __builtin_amdgcn_rcp(x);
    y = __builtin_fma(__builtin_fma(-x, y, 1.0), y, y);
    if constexpr (!F32) y = __builtin_fma(__builtin_fma(-x, y, 1.0), y, y);
    return y;
}

// log x for a pivot x (in (0, 1] up to rounding); NaN for x <= 0.  x = m 2^e with m in [sqrt(1/2),
// sqrt(2)), log m = 2 atanh(s) with s = (m - 1) / (m + 1), |s| < 0.1716: the series to s^21 leaves less
// than 1e-18 relative (to s^11, 2e-11, for the fixed point table), and m - 1 is exact, so pivots close to 1
// keep their relative accuracy.  21 of the library's logarithms were a third of the row's instructions.
template <bool F32>
__device__ __forceinline__ double pivot_log(double x)
{
    double m = __builtin_amdgcn_frexp_mant(x);
    int e = __builtin_amdgcn_frexp_exp(x);
    const bool low = m < 0.70710678118654752440;
    m = low ? m + m : m;
    e -= low ? 1 : 0;
    const double f = m - 1.0, den = m + 1.0, r = fast_rcp<F32>(den);
    double s = f * r;
    if constexpr (!F32) s = __builtin_fma(__builtin_fma(-den, s, f), r, s);   // the quotient's last bit
    const double z = s * s;
    double p = 1.0 / 11;
    if constexpr (!F32) {
        p = 1.0 / 21;
        p = __builtin_fma(p, z, 1.0 / 19);
        p = __builtin_fma(p, z, 1.0 / 17);
        p = __builtin_fma(p, z, 1.0 / 15);
        p = __builtin_fma(p, z, 1.0 / 13);
        p = __builtin_fma(p, z, 1.0 / 11);
    }
    p = __builtin_fma(p, z, 1.0 / 9);
    p = __builtin_fma(p, z, 1.0 / 7);
    p = __builtin_fma(p, z, 1.0 / 5);
    p = __builtin_fma(p, z, 1.0 / 3);
    const double s2 = s + s;
    const double lm = __builtin_fma(s2 * z, p, s2);
    const double y = __builtin_fma((double)e, kLn2, lm);
    return x > 0.0 ? y : __builtin_nan("");
}

// Subsets of suffix variables V..9 over the Schur complement s (lower triangle of variables V..9,
// row i - V): ld of every one into row[position], starting from ld and the subset m of the variables
// below V.
template <bool F32, int V>
__device__ __forceinline__ void cube_walk(const double (&s)[(kCubeSuffix - V) * (kCubeSuffix - V + 1) / 2 + 1], double ld,
                                          int m, double* __restrict__ row, const uint16_t* __restrict__ spos)
{
    if constexpr (V == kCubeSuffix) {
        row[spos[m]] = ld;
    } else {
        constexpr int n = kCubeSuffix - V;
        double x[(n - 1) * n / 2 + 1], y[(n - 1) * n / 2 + 1];
        sfor<1, n>([&](auto I) {
            sfor<1, I + 1>([&](auto J) { x[tri(I - 1, J - 1)] = s[tri(I, J)]; });
        });
        cube_walk<F32, V + 1>(x, ld, m, row, spos);
        const double p = s[0], inv = fast_rcp<F32>(p);
        sfor<1, n>([&](auto I) {
            const double t = s[tri(I, 0)] * inv;
            sfor<1, I + 1>([&](auto J) { y[tri(I - 1, J - 1)] = __builtin_fma(-t, s[tri(J, 0)], s[tri(I, J)]); });
        });
        cube_walk<F32, V + 1>(y, ld + pivot_log<F32>(p), m | (1 << V), row, spos);
    }
}

// grid (ceil(2^h / 16), datasets of the group), block kBuildThreads: rows P of the table of dataset
// d0 + blockIdx.y (those that take is null or nonzero for), kBuildRows per wavefront.  Bit h - 1 - v of P is
// variable v.  Rows with more than kmax members are not needed.
template <bool F32>
__global__ __launch_bounds__(kBuildThreads) void k_cube_build(const double* __restrict__ Sigma, int N, int64_t d0,
                                                              int kmax, const uint32_t* __restrict__ take,
                                                              Tab<F32>* __restrict__ table)
{
    if (take && !take[d0 + blockIdx.y]) return;                        // uniform
    extern __shared__ __align__(16) unsigned char smem[];
    double* sR = reinterpret_cast<double*>(smem);                      // [N][N]
    double* sIsd = sR + N * N;                                         // [N]
    double* sLogd = sIsd + N;                                          // [N]
    double* srow_w = sLogd + N;                                        // [waves][1024]
    double* scol_w = srow_w + kBuildWaves * kCubeRow;                  // [waves][2][32]
    double* ssch_w = scol_w + kBuildWaves * 64;                        // [waves][56]
    uint16_t* spos = reinterpret_cast<uint16_t*>(ssch_w + kBuildWaves * 56);
    const int h = N - kCubeSuffix;
    const int64_t d = d0 + blockIdx.y;
    for (int i = threadIdx.x; i < kCubeRow; i += kBuildThreads) spos[i] = kSuffix.pos[i];
    stage_corr<double>(Sigma + d * N * N, N, sR, sIsd, sLogd);
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    double* srow = srow_w + wv * kCubeRow;
    double* scol = scol_w + wv * 64;
    double* ssch = ssch_w + wv * 56;
    // lanes 0..9: the suffix variables; lane 10 + q: the q-th member of P (ascending).  r[m], m < 10:
    // entry against suffix variable m; r[10 + q]: against member q.
    const bool suf = lane < kCubeSuffix;
    const int q = lane - kCubeSuffix;
    for (int it = 0; it < kBuildRows; ++it) {                          // no block barrier below
        const uint32_t P = __builtin_amdgcn_readfirstlane((blockIdx.x * kBuildRows + it) * kBuildWaves + wv);
        const int p = __popc(P);
        if ((P >> h) != 0 || p > kmax) continue;
        uint32_t m = P;
        int var = suf ? h + lane : 0;
        double r[kCubeSuffix + kCubePrefix];
        const bool row_on = suf || q < p;
        for (int e = 0; e < p; ++e) {
            const int v = h - 1 - (31 - __builtin_clz(m));
            m &= ~(0x80000000u >> __builtin_clz(m));
            if (q == e) var = v;
        }
        sfor<0, kCubeSuffix>([&](auto M) {
            constexpr int c = M;
            r[c] = suf ? sR[var * N + h + c] : 0.0;
        });
        m = P;
        sfor<0, kCubePrefix>([&](auto Q) {
            constexpr int c = Q;
            r[kCubeSuffix + c] = 0.0;
            if (c < p) {
                const int v = h - 1 - (31 - __builtin_clz(m));
                m &= ~(0x80000000u >> __builtin_clz(m));
                r[kCubeSuffix + c] = row_on ? sR[var * N + v] : 0.0;
            }
        });
        // eliminate the members of P one after the other
        double piv = 1.0;
        sfor<0, kCubePrefix>([&](auto J) {
            constexpr int j = J;
            if (j < p) {
                double* cl = scol + (j & 1) * 32;
                if (lane < 32) cl[lane] = r[kCubeSuffix + j];
                cube_wave_sync();
                const double pj = cl[kCubeSuffix + j];
                piv = q == j ? pj : piv;
                const double t = r[kCubeSuffix + j] * fast_rcp<F32>(pj);
                sfor<j + 1, kCubePrefix>([&](auto Q) {
                    constexpr int c = Q;
                    if (c < p) r[kCubeSuffix + c] = __builtin_fma(-t, cl[kCubeSuffix + c], r[kCubeSuffix + c]);
                });
                sfor<0, kCubeSuffix>([&](auto M) { r[M] = __builtin_fma(-t, cl[M], r[M]); });
            }
        });
        const double lp = pivot_log<F32>(piv);
        double ld = 0.0;
        for (int e = 0; e < p; ++e) ld += __shfl(lp, kCubeSuffix + e, 64);
        // the Schur complement of the ten variables in every lane
        if (suf) {
            sfor<0, kCubeSuffix>([&](auto M) {
                constexpr int c = M;
                if (c <= lane) ssch[lane * (lane + 1) / 2 + c] = r[c];
            });
        }
        cube_wave_sync();
        double s[kTri10];
        sfor<0, kTri10>([&](auto E) { s[E] = ssch[E]; });
        sfor<0, 6>([&](auto T) {
            constexpr int t = T;
            if ((lane >> t) & 1) {
                const double pt = s[tri(t, t)], inv = fast_rcp<F32>(pt);
                ld += pivot_log<F32>(pt);
                sfor<t + 1, kCubeSuffix>([&](auto I) {
                    constexpr int i = I;
                    const double f = s[tri(i, t)] * inv;
                    sfor<t + 1, i + 1>([&](auto Jc) {
                        constexpr int c = Jc;
                        s[tri(i, c)] = __builtin_fma(-f, s[tri(c, t)], s[tri(i, c)]);
                    });
                });
            }
        });
        double s4[11];
        sfor<0, 4>([&](auto I) {
            sfor<0, I + 1>([&](auto J) { s4[tri(I, J)] = s[tri(I + 6, J + 6)]; });
        });
        cube_walk<F32, 6>(s4, ld, lane, srow, spos);
        cube_wave_sync();
        // sizes up to kmax - p are needed, a prefix of the row
        const int need = kmax - p >= kCubeSuffix ? kCubeRow : kSuffix.off[kmax - p + 1];
        Tab<F32>* out = table + ((int64_t)blockIdx.y << N) + ((int64_t)P << kCubeSuffix);
        for (int i = lane; i < need; i += 64) encode(srow[i], out[i]);
        cube_wave_sync();                                              // srow and the buffers are reused
    }
}

size_t build_lds_bytes(int N)
{
    return ((size_t)N * N + 2 * N + kBuildWaves * (kCubeRow + 64 + 56)) * 8 + kCubeRow * 2;
}

constexpr int kCubeWide = 2;                           // entries per lane of the reduction
constexpr int kCubeRun = 256;                          // at least C(10, 5)

// W consecutive entries of a row, aligned as one entry.
template <int W, typename V>
struct Entries {
    V v[W];
};
template <int W, typename V>
__device__ __forceinline__ Entries<W, V> load_entries(const V* __restrict__ p)
{
    typedef V Pack __attribute__((ext_vector_type(W), aligned(sizeof(V))));
    const Pack x = *reinterpret_cast<const Pack*>(p);
    Entries<W, V> r;
#pragma unroll
    for (int w = 0; w < W; ++w) r.v[w] = x[w];
    return r;
}

// sum_j (ld(S \ j) - ld(S)) of entries e .. e + W - 1 of row P (all of size b; len entries of
// that size, the lane's first at index i among them): the members of P (uniform in the wavefront), eight
// reads in flight, then the b members among the ten, whose positions in the row are nb[i], nb[len + i], ...
// (entries past the run repeat its last: their sums are not used).  Also mx[w] = max_j of the differences
// (log of the largest VIF, too large by at most 2^-20 |ld(S)|) and ex[w], a bound of the sum of their
// exponentials (the sum of the VIFs): the largest of each eight or five, as often as there are terms.
template <typename V>
struct OneOut;
template <>
struct OneOut<double> {
    double s = 0.0;
    // the group's largest value from the high words alone: values are <= 0 (a rounding above 0 counts as
    // the largest), and of those the largest has the smallest word
    uint32_t g;
    __device__ __forceinline__ void open() { g = 0xffffffffu; }
    __device__ __forceinline__ void add(double v)
    {
        s += v;
        const uint32_t hi = (uint32_t)__double2hiint(v);
        g = hi < g ? hi : g;
    }
    __device__ __forceinline__ float most(double t0) const { return (float)(__hiloint2double((int)g, 0) - t0); }
    __device__ __forceinline__ double sum(double t0, int k) const { return __builtin_fma(-(double)k, t0, s); }
};
template <>
struct OneOut<int32_t> {
    int64_t s = 0;
    int32_t g;
    __device__ __forceinline__ void open() { g = -kFixBad - 1; }
    __device__ __forceinline__ void add(int32_t v)
    {
        s += v;
        g = v > g ? v : g;
    }
    // (infinite where a member is bad: ex is then, too)
    __device__ __forceinline__ float most(int32_t t0) const
    {
        return g == kFixBad ? __builtin_inff() : (float)((int64_t)g - t0) * (float)(1.0 / kFixScale);
    }
    __device__ __forceinline__ double sum(int32_t t0, int k) const
    {
        return t0 == kFixBad ? __builtin_nan("") : (double)(s - (int64_t)k * t0) * (1.0 / kFixScale);
    }
};
template <int W, typename V>
struct LeaveOneOut {
    OneOut<V> o[W];
    float mx[W], ex[W];
    __device__ __forceinline__ LeaveOneOut()
    {
#pragma unroll
        for (int w = 0; w < W; ++w) { mx[w] = 0.0f; ex[w] = 0.0f; }
    }
    __device__ __forceinline__ void open()
    {
#pragma unroll
        for (int w = 0; w < W; ++w) o[w].open();
    }
    __device__ __forceinline__ void close(const Entries<W, V>& t0, int n)
    {
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const float x = o[w].most(t0.v[w]);
            mx[w] = x > mx[w] ? x : mx[w];
            ex[w] = fmaf((float)n, __builtin_amdgcn_exp2f(x * 1.442695041f), ex[w]);
        }
    }
    // the members of P
    __device__ __forceinline__ void prefix(const V* __restrict__ T, uint32_t P, int e, const Entries<W, V>& t0)
    {
        uint32_t m = P;
        while (m) {
            Entries<W, V> v[8];
            uint32_t mm = m;
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                v[u] = t0;
                if (mm) {
                    const uint32_t bit = 0x80000000u >> __builtin_clz(mm);
                    v[u] = load_entries<W, V>(T + ((int64_t)(P ^ bit) << kCubeSuffix) + e);
                    mm ^= bit;
                }
            }
            const int n = __popc(m) - __popc(mm);
            open();
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (m) {
#pragma unroll
                    for (int w = 0; w < W; ++w) o[w].add(v[u].v[w]);
                    m ^= 0x80000000u >> __builtin_clz(m);
                }
            close(t0, n);
        }
    }
    // the b members among the ten, at row[position - shift]
    __device__ __forceinline__ void suffix(const V* row, int shift, int b, int len, int i, const Entries<W, V>& t0,
                                           const uint16_t* nb)
    {
        int at_i[W];
#pragma unroll
        for (int w = 0; w < W; ++w) at_i[w] = i + w < len ? i + w : len - 1;
        for (int t = 0; t < b; t += 5) {
            int at[5][W];
            V v[5][W];
#pragma unroll
            for (int u = 0; u < 5; ++u)
#pragma unroll
                for (int w = 0; w < W; ++w) at[u][w] = nb[(t + u < b ? t + u : b - 1) * len + at_i[w]];
#pragma unroll
            for (int u = 0; u < 5; ++u)
#pragma unroll
                for (int w = 0; w < W; ++w) v[u][w] = row[at[u][w] - shift];
            open();
#pragma unroll
            for (int u = 0; u < 5; ++u)
                if (t + u < b) {                                       // uniform
#pragma unroll
                    for (int w = 0; w < W; ++w) o[w].add(v[u][w]);
                }
            close(t0, b - t < 5 ? b - t : 5);
        }
    }
};

// ------------------------------------------------------------------------------------------------
// Admission bounds before the reduction.  A workgroup that starts with empty lists inserts almost
// every value of its first iterations, at about 7,000 cycles per insertion: so kSampleGroups
// workgroups per order first evaluate n-plets spread over the order and each finds a key that its
// share of the K best reach; all groups together then hold K distinct n-plets up to the largest of
// these keys, and the reduction meets them again.  A wavefront takes the 64-entry piece of a run that
// holds an evenly spaced rank, so its reads are as coalesced as the reduction's (n-plets at single
// ranks, scattered over the table: 224 us against 85 at N = 25).  Small orders
// take fewer pieces: less than 64 ranks apart two could coincide.
// ------------------------------------------------------------------------------------------------
constexpr int kSampleThreads = 1024;
constexpr int kSamplePer = 8;                          // pieces per wavefront
constexpr int kSampleGroups = 8;
constexpr uint32_t kSamplePieces = kSampleThreads / 64 * kSamplePer * kSampleGroups;

// grid (kSampleGroups, orders, datasets of the group): sbound[dataset of the group][order][group][2].  take: by
// dataset of the group, or null.
// The values are taken at the unfavourable end of what the factorisation may make of them; FP32:
// n-plets near or above the refinement threshold are left out.
template <bool F32>
__global__ __launch_bounds__(kSampleThreads) void k_cube_sample(EvalArgs a, CubeTable tab, int K,
                                                                const uint32_t* __restrict__ take,
                                                                const Tab<F32>* __restrict__ table,
                                                                uint64_t* __restrict__ sbound)
{
    if (take && !take[blockIdx.z]) return;                             // uniform
    __shared__ uint32_t sbin[kCubeMaxN * (kCubeMaxN + 1)];
    __shared__ uint16_t snbr[kCubeSuffix * kCubeRow / 2];
    __shared__ uint32_t rh[256];
    __shared__ uint32_t sprefix;
    __shared__ int srank;
    __shared__ double sbias[3];
    const int N = a.N, h = N - kCubeSuffix;
    const int k = tab.p[blockIdx.y].k;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    uint64_t* out = sbound + (((int64_t)blockIdx.z * gridDim.y + blockIdx.y) * kSampleGroups + blockIdx.x) * 2;
    const uint32_t total = (uint32_t)kPascal.v[N][k];
    const uint32_t pieces = total / 64 < kSamplePieces ? total / 64 : kSamplePieces;
    for (int i = tid; i < N * (k + 1); i += kSampleThreads) sbin[i] = (uint32_t)kPascal.v[i / (k + 1)][i % (k + 1)];
    for (int i = tid; i < kCubeSuffix * kCubeRow / 2; i += kSampleThreads) snbr[i] = kSuffix.nbr[i];
    if (tid == 0) bias_for(a.bias, k, sbias[0], sbias[1], sbias[2]);
    __syncthreads();
    const Tab<F32>* T = table + ((int64_t)blockIdx.z << N);
    double om[kSamplePer], mu[kSamplePer];
    int nv = 0;
#pragma unroll
    for (int u = 0; u < kSamplePer; ++u) {
        const uint32_t s = ((uint32_t)u * (kSampleThreads / 64) + wv) * kSampleGroups + blockIdx.x;
        if (s >= pieces) {                             // uniform in the wavefront
            om[u] = __builtin_nan("");
            mu[u] = 0.0;
            continue;
        }
        uint32_t r = (uint32_t)((uint64_t)s * total / pieces);
        // the r-th k-subset in lexicographic order, as prefix bits and suffix bits (uniform)
        uint32_t P = 0, B = 0;
        int m = k - 1;
        for (int x = 0; x < N && m >= 0; ++x) {
            const uint32_t c = sbin[(N - 1 - x) * (k + 1) + m];
            if (r < c) {
                if (x < h) P |= 1u << (h - 1 - x);
                else B |= 1u << (x - h);
                --m;
            } else {
                r -= c;
            }
        }
        P = __builtin_amdgcn_readfirstlane(P);
        B = __builtin_amdgcn_readfirstlane(B);
        const int b = __popc(B);
        const int o0 = kSuffix.off[b], len = kSuffix.off[b + 1] - o0;
        const int i = (kSuffix.pos[B] - o0) / 64 * 64 + lane;
        const bool on = i < len;
        const int e = o0 + (on ? i : 0);
        const Entries<1, Tab<F32>> ld = load_entries<1, Tab<F32>>(T + ((int64_t)P << kCubeSuffix) + e);
        LeaveOneOut<1, Tab<F32>> lv;
        lv.prefix(T, P, e, ld);
        lv.suffix(T + ((int64_t)P << kCubeSuffix), 0, b, len, on ? i : 0, ld, snbr + kSuffix.noff[b]);
        const double t0 = decode(ld.v[0]), sa = lv.o[0].sum(ld.v[0], k);
        const double TC = -0.5 * t0 + sbias[0], DTC = 0.5 * (t0 + sa) + sbias[1];
        om[u] = on && isfinite(t0) && isfinite(sa) ? TC - DTC : __builtin_nan("");
        const Margin mg = margin_of<F32>(k, t0, lv.mx[0], lv.ex[0], a.vif_tau);
        mu[u] = mg.value(TC, DTC);
        if (mg.vif != 0 || !isfinite(mu[u])) om[u] = __builtin_nan("");
    }
#pragma unroll
    for (int u = 0; u < kSamplePer; ++u) nv += __syncthreads_count(!isnan(om[u]));
    const int want = (K + kSampleGroups - 1) / kSampleGroups;
    for (int l = 0; l < 2; ++l) {
        uint64_t key = kKeyEmpty;
        if (nv >= want) {                              // uniform
            if (tid == 0) { sprefix = 0; srank = want; }
            for (int pass = 3; pass >= 0; --pass) {
                if (tid < 256) rh[tid] = 0;
                __syncthreads();
                const uint32_t pre = sprefix;
#pragma unroll
                for (int u = 0; u < kSamplePer; ++u) {
                    const uint32_t hw = (uint32_t)(red_list_key(l, l == 0 ? om[u] - mu[u] : om[u] + mu[u]) >> 32);
                    if (!isnan(om[u]) && radix_match(hw, pre, pass)) atomicAdd(&rh[(hw >> (8 * pass)) & 255u], 1u);
                }
                __syncthreads();
                if (tid < 64) radix_pick(rh, tid, pass, sprefix, srank);
                __syncthreads();
            }
            key = ((uint64_t)sprefix << 32) | 0xffffffffull;
            __syncthreads();
        }
        if (tid == 0) out[l] = key;
    }
}

// grid (orders, datasets of the group), block 64: the bound of each list from its groups' keys.
__global__ void k_cube_bounds(CubeTable tab, RedArgs red, int64_t d0, const uint32_t* __restrict__ take,
                              const uint64_t* __restrict__ sbound)
{
    const int l = threadIdx.x;
    if (l >= 2 || (take && !take[d0 + blockIdx.y])) return;
    const uint64_t* b = sbound + ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * kSampleGroups * 2 + l;
    uint64_t worst = 0;
    for (int g = 0; g < kSampleGroups; ++g) worst = b[2 * g] > worst ? b[2 * g] : worst;
    if (worst != kKeyEmpty)
        atomicMax(red.bound + ((d0 + blockIdx.y) * (red.kmax + 1) + tab.p[blockIdx.x].k) * 2 + l, (unsigned long long)~worst);
}

constexpr int kOpenBuf = 256;                          // open n-plets a wavefront collects in LDS

// Whole wavefront: append buf[0..n) to the open list of order k.
__device__ __forceinline__ void flush_open(const CubeOpen& o, int k, const uint32_t* buf, int n, int lane)
{
    if (n == 0) return;
    cube_wave_sync();
    uint32_t at = 0;
    if (lane == 0) at = atomicAdd(&o.cnt[k], (uint32_t)n);
    at = __shfl(at, 0, 64);
    for (int i = lane; i < n; i += 64) o.list[o.off[k] + at + i] = buf[i];
    cube_wave_sync();
}

// grid (8 ceil(chunks / 8) orders), block 256: dataset d0, its table.  take: as for the build.
//
// The results are those of one factorisation per n-plet bit for bit (list values and indices, counts,
// what is refined), so the table's values only decide where the factorisation's cannot differ: an n-plet
// whose bin is the same over the whole margin and which cannot enter a list is counted; FP32: one above
// the refinement threshold is queued for it; the rest (FP32: about 1%; FP64: what may enter the lists) is
// left open and evaluated by k_cube_verify.
template <bool F32>
__global__ __launch_bounds__(256) void k_cube_filter(EvalArgs a, CubeTable tab, RedArgs red, CubeOpen opn, int64_t d0,
                                                     const uint32_t* __restrict__ take, const Tab<F32>* __restrict__ table)
{
    if (take && !take[d0]) return;                                     // uniform
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint32_t sopen[4 * kOpenBuf];
    __shared__ uint16_t smask[kCubeRow];
    __shared__ int32_t srun[F32 ? 4 * kCubeRun : 1];
    __shared__ double sbias[3];
    const int N = a.N, h = N - kCubeSuffix;
    // all orders of one chunk of rows run together on one XCD (workgroups are dealt to the 8 XCDs
    // round robin), so the rows and their neighbours are read from its L2
    const int xcd = (int)blockIdx.x % 8, loc = (int)blockIdx.x / 8;
    const int chunk = loc / tab.n * 8 + xcd;
    const CubePiece pc = tab.p[loc % tab.n];
    if (chunk >= tab.chunks) return;                                   // uniform
    const int k = pc.k;
    const int64_t d = d0;
    uint16_t* snbr = reinterpret_cast<uint16_t*>(smem);                // [5120]
    uint32_t* sbin = reinterpret_cast<uint32_t*>(snbr + kCubeSuffix * kCubeRow / 2);   // C(n, m), n < N, m <= k
    const size_t off = (kCubeSuffix * kCubeRow + (size_t)kCubeMaxN * (kCubeMaxN + 1) * 4 + 15) / 16 * 16;
    RedLds S = red_view(smem + off, 0, red.bins);
    for (int i = threadIdx.x; i < kCubeSuffix * kCubeRow / 2; i += 256) snbr[i] = kSuffix.nbr[i];
    for (int i = threadIdx.x; i < kCubeRow; i += 256) smask[i] = kSuffix.mask[i];
    for (int i = threadIdx.x; i < N * (k + 1); i += 256) sbin[i] = (uint32_t)kPascal.v[i / (k + 1)][i % (k + 1)];
    if (threadIdx.x == 0) bias_for(a.bias, k, sbias[0], sbias[1], sbias[2]);
    const double lo = red.lo[k], scale = (double)red.bins / (red.hi[k] - red.lo[k]);
    double top = -__builtin_inf(), bottom = __builtin_inf();
    RedArgs hist = red;                                                // counts only: the lists are k_cube_verify's
    hist.topk = 0;
    red_begin(S, hist, (int)d, k);                                     // ends with a barrier
    if (red.topk > 0) {
        // Omega from which the lists may take a value (every value without a bound)
        const unsigned long long* bd = red.bound + (d * (red.kmax + 1) + k) * 2;
        if (bd[0]) top = red_list_val(0, ~(uint64_t)bd[0]);
        if (bd[1]) bottom = red_list_val(1, ~(uint64_t)bd[1]);
    }
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    uint32_t* sbuf = sopen + wv * kOpenBuf;
    int32_t* run = srun + (F32 ? wv * kCubeRun : 0);
    int nbuf = 0;                                                      // uniform in the wavefront
    const Tab<F32>* T = table;
    const uint32_t nrows = 1u << h;
    const uint32_t r0 = (uint32_t)tab.row0 + (uint32_t)chunk * (uint32_t)tab.per;
    const uint32_t r1 = min(r0 + (uint32_t)tab.per, nrows);
    for (uint32_t Pw = r0 + wv; Pw < r1; Pw += 4) {
        const uint32_t P = __builtin_amdgcn_readfirstlane(Pw);
        const int p = __popc(P), b = k - p;
        if (b < 0 || b > kCubeSuffix) continue;                        // uniform in the wavefront
        const int o0 = kSuffix.off[b], len = kSuffix.off[b + 1] - o0;
        // lexicographic rank of P + {first b of the ten}: C(N, k) - 1 - sum C(N - 1 - c_i, k - i)
        // (lane v: variable v when it is a member, with its place among the members)
        uint32_t term = 0;
        if (lane < h) {
            if ((P >> (h - 1 - lane)) & 1u) term = sbin[(N - 1 - lane) * (k + 1) + k - (int)__popc(P >> (h - lane))];
        } else if (lane < h + b) {
            term = sbin[(N - 1 - lane) * (k + 1) + k - p - (lane - h)];
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) term += __shfl_xor(term, o, 64);
        const uint32_t rank0 = (uint32_t)kPascal.v[N][k] - 1u - term;
        // FP32: the row's subsets of one variable less, where those without one of the ten are, go into LDS
        // once the members of P are under way (N = 30: 31.5 ms without, 30.1 with; in FP64 the registers
        // cost a wavefront per SIMD, N = 27: 4.11 without, 4.20 with)
        const int om = b > 0 ? kSuffix.off[b - 1] : 0, lenm = b > 0 ? o0 - om : 0;
        int32_t less[kCubeRun / 64];
        if constexpr (F32) {
#pragma unroll
            for (int u = 0; u < kCubeRun / 64; ++u) {
                less[u] = 0;
                if (64 * u + lane < lenm) less[u] = T[((int64_t)P << kCubeSuffix) + om + 64 * u + lane];
            }
        }
        for (int i0 = 0; i0 < len; i0 += 64 * kCubeWide) {
            const int i = i0 + lane * kCubeWide;
            const bool on = i < len;
            const int e = o0 + (on ? i : 0);
            const Entries<kCubeWide, Tab<F32>> ld = load_entries<kCubeWide, Tab<F32>>(T + ((int64_t)P << kCubeSuffix) + e);
            LeaveOneOut<kCubeWide, Tab<F32>> lv;
            lv.prefix(T, P, e, ld);
            if constexpr (F32) {
                if (i0 == 0) {
#pragma unroll
                    for (int u = 0; u < kCubeRun / 64; ++u) run[64 * u + lane] = less[u];
                    cube_wave_sync();
                }
                lv.suffix(run, om, b, len, on ? i : 0, ld, snbr + kSuffix.noff[b]);
            } else {
                lv.suffix(T + ((int64_t)P << kCubeSuffix), 0, b, len, on ? i : 0, ld, snbr + kSuffix.noff[b]);
            }
#pragma unroll
            for (int w = 0; w < kCubeWide; ++w) {
                const bool in = i + w < len;
                const int64_t pos = pc.pos0 + rank0 + i + w;
                const double t0 = decode(ld.v[w]);
                const double TC = -0.5 * t0 + sbias[0], sa = lv.o[w].sum(ld.v[w], k);
                const double DTC = 0.5 * (t0 + sa) + sbias[1];
                const double v = TC - DTC;
                const Margin mg = margin_of<F32>(k, t0, lv.mx[w], lv.ex[w], a.vif_tau);
                const bool bad = !isfinite(t0) || !isfinite(sa) || !(lv.ex[w] < 3e38f);
                const bool refine = F32 && in && !bad && mg.vif == 2;
                // open: no value in the table, the VIF near the threshold, Omega near a bin edge or near the lists
                bool open = in && !refine && (bad || mg.vif == 1);
                const double mu = mg.value(TC, DTC);
                if (red.topk > 0) open = open || (in && !refine && (v + mu >= top || v - mu <= bottom));
                int bin = 0;
                if (red.bins > 0) {
                    // the place among the bins, and the margin there (with room for the rounding of
                    // this product against the reducer's quotient)
                    const double x = (v - lo) * scale, fx = floor(x), ms = mu * scale + 1e-9;
                    const bool under = x < -ms, over = x > (double)red.bins + ms;
                    bin = under ? red.bins : (over ? red.bins + 1 : (int)fx);
                    const bool clear = under || over || (x - fx > ms && fx + 1.0 - x > ms && x > 0.0 && bin < red.bins);
                    open = open || (in && !refine && !clear);
                }
                if (in && !refine && !open && red.bins > 0) atomicAdd(&S.hist[bin], 1u);
                if (a.flags && in && !open) a.flags[d * a.B + pos] = refine ? THOI_NPLET_REFINED : 0;
                if constexpr (F32) {
                    const uint64_t mr = __ballot(refine);
                    if (mr) {
                        const int leader = __builtin_ctzll(mr);
                        uint32_t at = 0;
                        if (lane == leader) at = atomicAdd(&a.hdr->refine_count, (uint32_t)__popcll(mr));
                        at = __shfl(at, leader, 64) + (uint32_t)__popcll(mr & __lanemask_lt());
                        if (refine) {
                            if (at < a.refine_cap) a.refine_list[at] = d * a.B + pos;
                            else raise_status(a.hdr, THOI_EWORKSPACE);
                        }
                    }
                }
                const uint64_t mo = __ballot(open);
                if (mo) {
                    if (open) sbuf[nbuf + __popcll(mo & __lanemask_lt())] = (P << kCubeSuffix) | smask[o0 + i + w];
                    nbuf += __popcll(mo);
                }
            }
            // the wavefront's buffer goes out when the next iteration may not fit
            if (nbuf > kOpenBuf - 64 * kCubeWide) {
                flush_open(opn, k, sbuf, nbuf, lane);
                nbuf = 0;
            }
        }
        if constexpr (F32) cube_wave_sync();                           // the next run overwrites the buffer
    }
    flush_open(opn, k, sbuf, nbuf, lane);
    red_end(S, hist, a.hdr, (int)d, k);
}

size_t filter_lds_bytes(const RedArgs& red)
{
    return (kCubeSuffix * kCubeRow + (size_t)kCubeMaxN * (kCubeMaxN + 1) * 4 + 15) / 16 * 16 + red_lds_bytes(0, red.bins);
}

// Chunks of rows: a wavefront spends about as long on the start of a (row, size) run as on two of its
// 64-entry iterations, so the work of a launch is the sum over its runs of 2 + iterations; about 128 per
// workgroup, a power of two of at least 16 rows, at most kMaxChunks chunks.
constexpr int64_t kMaxChunks = 4096;

CubeTable cube_table(int N, int kmin, int kmax, int64_t rows)
{
    CubeTable t{};
    const int h = N - kCubeSuffix;
    int64_t pos = 0, work = 0;
    for (int k = kmin; k <= kmax; ++k) {
        for (int p = 0; p <= h; ++p) {
            const int b = k - p;
            if (b >= 0 && b <= kCubeSuffix)
                work += (int64_t)binom_u64(h, p) * (2 + ((int64_t)binom_u64(kCubeSuffix, b) + 63) / 64);
        }
        t.p[t.n++] = CubePiece{k, 0, pos};
        pos += (int64_t)binom_u64(N, k);
    }
    work = work / ((int64_t(1) << h) / rows);
    const int64_t want = work / (128 * t.n);
    int64_t chunks = 8;
    while (chunks < want && chunks < kMaxChunks) chunks *= 2;
    while (rows / chunks < 16) chunks /= 2;
    t.chunks = (int32_t)chunks;
    t.per = (int32_t)(rows / chunks);
    return t;
}

int64_t cube_blocks(const CubeTable& t) { return (int64_t)(t.chunks + 7) / 8 * 8 * t.n; }

// Datasets whose tables are held at a time: up to 256 MB together, at least one dataset's.
int64_t cube_group(int32_t N, int64_t D, bool f32)
{
    const int64_t g = (int64_t(1) << 28) >> (N + (f32 ? 2 : 3));
    return g < 1 ? 1 : (g < D ? g : D);
}

// Rows filtered in one launch.  A block of rows is evaluated while the next one is filtered, and its lists
// tighten the bounds of those after that; the fork and join cost about 45 us a block (N = 25: one block
// 1.26 ms, two 1.32, four 1.50; N = 30, FP32: four blocks 31.4 ms, eight 31.9).
constexpr int kFilterBits = 18;
int filter_bits(int N) { return N - kCubeSuffix < kFilterBits ? N - kCubeSuffix : kFilterBits; }
// The largest number of n-plets of order k in such an aligned block of rows: the high prefix bits fix c
// members, the rest is free.
int64_t open_cap(int N, int k)
{
    const int free_vars = filter_bits(N) + kCubeSuffix;
    int64_t most = 0;
    for (int c = 0; c <= N - free_vars && c <= k; ++c) {
        const int64_t n = (int64_t)binom_u64(free_vars, k - c);
        most = n > most ? n : most;
    }
    return most;
}

struct CubeMem {
    size_t sample, cnt, list[2], total;                // behind the tables; a list for every other block
    CubeOpen open;
};
CubeMem cube_mem(int N, int64_t D, int kmin, int kmax, bool f32)
{
    CubeMem m{};
    const int64_t g = cube_group(N, D, f32);
    size_t off = (size_t)g << (N + (f32 ? 2 : 3));
    m.sample = off;
    off = align_up(off + (size_t)g * (N + 1) * kSampleGroups * 16, 256);
    m.cnt = off;
    off += 512;
    int64_t o = 0;
    for (int k = kmin; k <= kmax; ++k) {
        m.open.off[k] = o;
        o += open_cap(N, k);
    }
    const int lists = filter_bits(N) < N - kCubeSuffix || D > 1 ? 2 : 1;
    for (int i = 0; i < 2; ++i) {
        m.list[i] = i < lists ? off : m.list[0];
        if (i < lists) off = align_up(off + (size_t)o * 4, 256);
    }
    m.total = off;
    return m;
}

}  // namespace

int cube_kmax(bool f32, int kmax) { return f32 && kmax > kF32LaneMax ? kF32LaneMax : kmax; }

// Estimated times in ns, FP32 + refinement.  A factorisation per n-plet: 0.05 up to order 12, 0.07 above.  The
// table: 6 per row of up to kmax members, whatever sizes are needed, 0.027 per n-plet, 40,000 for the
// additional launches; 1.3 times its share for an open n-plet, which is evaluated by itself.  Measured, a
// factorisation per n-plet / the table, ms (orders, D datasets):
//   26 (3..26) 3.76 / 1.92   26 (3..12) 1.25 / 1.18   26 (3..10) 0.55 / 1.02   26 (18..26) 0.53 / 1.04
//   28 (3..28) 14.5 / 6.80   28 (3..12) 2.74 / 3.48   28 (12..14) 4.68 / 2.84  D = 4: 26 (3..26) 13.6 / 7.42
CubeCost cube_cost(int32_t N, int kmin, int kmax)
{
    CubeCost c{};
    const int h = N - kCubeSuffix;
    double table = 4e4;
    for (int k = kmin; k <= kmax; ++k) {
        const double n = (double)binom_u64(N, k), per = k <= 12 ? 0.05 : 0.07;
        c.factor[k] = (float)(n * per);
        c.open[k] = (float)(n * 1.3 * per);
        table += n * 0.027;
    }
    for (int p = 0; p <= h && p <= kmax; ++p) table += 6.0 * (double)binom_u64(h, p);
    c.table = (float)table;
    return c;
}

// The same for D datasets in FP64, fitted to 369 pairs of timings (21..30 variables, D = 1, 4 and 16, single orders
// and ranges).  A factorisation per n-plet: up to order 12 (prefix sharing, the better the more tails a prefix
// has) 0.036 + 0.13 e with e = 2^-((N - 21) / 2.5), a tenth more at 12; then 0.077 + 0.19 e; from 15 on 0.22, from 19
// on (two per wavefront) 2.9; 50,000 a call, with orders above 18 another 350,000, the latency of their lanes.
// The table: 4.6 per row and 0.53 for each order that passes over it, and 4 for each order that kmin lies above
// h (the rows of many members, which hold the n-plets, are then few and close together), 0.011 per n-plet,
// 95,000 per dataset (they are filtered one after the other) and 155,000 a call.  A factorisation per
// n-plet / the table, ms; the choice is the slower one of the two by 5% at most in 4 of the 369:
//   21 (3..21) 0.74 / 0.35   21 (3..10) 0.19 / 0.30   24 (3..9) 0.30 / 0.40    24 (3..10) 0.52 / 0.46
//   25 (3..25) 4.16 / 1.08   25 (12..12) 0.45 / 0.46  27 (3..10) 1.03 / 1.52   30 (3..12) 8.94 / 11.9
//   D = 4:   21 (3..21) 1.59 / 0.83   25 (3..10) 2.36 / 2.43   25 (19..25) 3.20 / 3.75   27 (21..27) 5.92 / 7.66
//   D = 16:  21 (3..21) 6.11 / 2.91   21 (3..9) 1.61 / 1.97    24 (3..9) 4.04 / 4.78     23 (14..23) 7.44 / 4.13
bool cube_faster_f64(int32_t N, int64_t D, int kmin, int kmax)
{
    const int h = N - kCubeSuffix;
    const double e = std::exp2(-(N - 21) / 2.5), low = 0.036 + 0.13 * e, mid = 0.077 + 0.19 * e;
    double n = 0.0, factor = (5e4 + (kmax > kF64LaneMax ? 3.5e5 : 0.0)) / (double)D;
    for (int k = kmin; k <= kmax; ++k) {
        const double c = (double)binom_u64(N, k);
        n += c;
        factor += c * (k < 12 ? low : k == 12 ? 1.1 * low : k <= 14 ? mid : k <= kF64LaneMax ? 0.22 : 2.9);
    }
    const double row = 4.6 + 0.53 * (kmax - kmin + 1) + (kmin > h ? 4.0 * (kmin - h) : 0.0);
    const double table = 1.55e5 / (double)D + 9.5e4 + row * (double)(int64_t(1) << h) + 0.011 * n;
    return factor > 1.04 * table;
}

bool cube_wanted(int32_t N, int64_t D, const thoi_nplets* sel, const thoi_eval_opts* opts)
{
    if (sel->mode != THOI_SEL_RANGE || !opts->reduce || D < 1) return false;
    const bool f32 = opts->precision == THOI_FP32_REFINE;
    if (!f32 && opts->precision != THOI_FP64) return false;
    // orders 1 and 2 have Omega = 0 up to rounding: their lists would be ordered by other rounding
    if (sel->kmin < 3) return false;
    if (opts->engine != THOI_ENGINE_AUTO || N < (f32 ? kCubeMinN32 : kCubeMinN) || N > kCubeMaxN) return false;
    // whole orders only
    int64_t all = 0;
    for (int k = sel->kmin; k <= sel->kmax; ++k) all += (int64_t)binom_u64(N, k);
    if (sel->g_begin != 0 || sel->g_count != all) return false;
    if (!f32) return cube_faster_f64(N, D, sel->kmin, sel->kmax);
    const int kmax = cube_kmax(true, sel->kmax);
    const CubeCost c = cube_cost(N, sel->kmin, kmax);
    double factor = 0.0;
    for (int k = sel->kmin; k <= kmax; ++k) factor += (double)c.factor[k];
    return factor > 1.15 * (double)c.table;
}

size_t cube_bytes(int32_t N, int64_t D, int kmin, int kmax, bool f32) { return cube_mem(N, D, kmin, kmax, f32).total; }

int64_t cube_segments(int32_t N, int kmin, int kmax, bool f32)
{
    // a workgroup of the evaluation without an open n-plet leaves none
    const int64_t blocks = int64_t(1) << (N - kCubeSuffix - filter_bits(N));
    int64_t n = 0;
    for (int k = kmin; k <= kmax; ++k) {
        const int64_t per = f32 || k <= kF64LaneMax ? kTile : kTile / 32, most = (open_cap(N, k) + per - 1) / per;
        n += blocks * (most < kVerifyBlocks ? most : kVerifyBlocks);
    }
    return n;
}

namespace {

template <bool F32>
void launch(const EvalArgs& a, const RedArgs& red, int kmin, int kmax, bool serial, const CubeGate& gate, void* mem,
            const std::function<void(hipStream_t)>& beside, const std::function<void(const FanScope&)>& rest, hipStream_t s)
{
    static_assert(sizeof(kSuffixHost.nbr) == kCubeSuffix * kCubeRow, "one neighbour per element");
    const int64_t rows = int64_t(1) << (a.N - kCubeSuffix);
    const int64_t step = int64_t(1) << filter_bits(a.N);
    CubeTable tab = cube_table(a.N, kmin, kmax, step);
    const int64_t blocks = cube_blocks(tab);
    const int64_t group = cube_group(a.N, a.D, F32);
    CubeMem m = cube_mem(a.N, a.D, kmin, kmax, F32);
    char* base = static_cast<char*>(mem);
    Tab<F32>* table = static_cast<Tab<F32>*>(mem);
    uint64_t* sbound = reinterpret_cast<uint64_t*>(base + m.sample);
    CubeOpen open[2] = {m.open, m.open};
    for (int i = 0; i < 2; ++i) {
        open[i].list = reinterpret_cast<uint32_t*>(base + m.list[i]);
        open[i].cnt = reinterpret_cast<uint32_t*>(base + m.cnt + 256 * i);
    }
    if (gate.take) cube_gate_launch(a, tab, red, gate, cube_cost(a.N, kmin, kmax), s);
    for (int64_t d0 = 0; d0 < a.D; d0 += group) {
        const int64_t nd = d0 + group < a.D ? group : a.D - d0;
        {
            const bool two = d0 == 0 && beside;
            FanScope fan(s, two && !serial ? 2 : 1);
            if (two) beside(fan.stream(1));
            const int64_t nb = (rows + kBuildWaves * kBuildRows - 1) / (kBuildWaves * kBuildRows);
            hipLaunchKernelGGL(k_cube_build<F32>, dim3((unsigned)nb, (unsigned)nd), dim3(kBuildThreads), build_lds_bytes(a.N),
                               fan.stream(0), a.Sigma, a.N, d0, kmax, gate.take, table);
        }
        if (red.topk > 0) {
            hipLaunchKernelGGL(k_cube_sample<F32>, dim3(kSampleGroups, (unsigned)tab.n, (unsigned)nd), dim3(kSampleThreads), 0, s, a, tab,
                               red.topk, gate.take ? gate.take + d0 : nullptr, table, sbound);
            hipLaunchKernelGGL(k_cube_bounds, dim3((unsigned)tab.n, (unsigned)nd), dim3(64), 0, s, tab, red, d0, gate.take, sbound);
        }
        // one dataset at a time, block of rows after block of rows, each evaluated beside the next filter
        const int64_t steps = nd * (rows / step);
        for (int64_t i = 0; i <= steps; ++i) {
            FanScope fan(s, serial ? 1 : 6);
            if (i < steps) {
                const int64_t e = i / (rows / step);
                tab.row0 = (int32_t)(i % (rows / step) * step);
                ws_clear(open[i & 1].cnt, 256, fan.stream(0));
                hipLaunchKernelGGL(k_cube_filter<F32>, dim3((unsigned)blocks), dim3(256), filter_lds_bytes(red), fan.stream(0), a, tab, red,
                                   open[i & 1], d0 + e, gate.take, table + (e << a.N));
            }
            // (the last block has the caller's stream as well)
            if (i > 0) cube_verify_launch(a, tab, open[(i - 1) & 1], red, d0 + (i - 1) / (rows / step), F32, fan, i < steps ? 1 : 0);
            if (rest && i == steps && d0 + group >= a.D) rest(fan);
        }
    }
}

}  // namespace

void cube_launch(const EvalArgs& a, const RedArgs& red, int kmin, int kmax, bool f32, bool serial, const CubeGate& gate, void* mem,
                 const std::function<void(hipStream_t)>& beside, const std::function<void(const FanScope&)>& rest, hipStream_t s)
{
    if (f32) launch<true>(a, red, kmin, kmax, serial, gate, mem, beside, rest, s);
    else launch<false>(a, red, kmin, kmax, serial, gate, mem, beside, rest, s);
}

}  // namespace thoi
