// Subset-table ("cube") engine: FP64 streaming reductions over whole orders of 21..30 variables.
//
// An exhaustive enumeration meets every subset of S as an n-plet of its own, so the leave-one-out
// determinants need no inverse: with ld(S) = log det R_S in a table over all 2^N subsets,
//   log a_j = log (R_S^-1)_jj = ld(S \ j) - ld(S)
// (the cofactor identity), and an n-plet costs one pivot and k table reads instead of a factorisation
// and an inversion of order k ("The combinatorial explosion": the number of subsets stays, the k^3
// per subset goes).
//
// A subset is a prefix P (of the first h = N - 10 variables) and one of the 1024 subsets of the last
// ten; row P of the table holds the latter ordered by size and, within a size, lexicographically.
//  - k_cube_build, one wavefront per row: the prefix is eliminated from the matrix of P and the ten
//    variables (right-looking, one matrix row per lane), then every lane eliminates its subset of the
//    first six variables from its own copy of the 10 x 10 Schur complement and walks the 16 subsets
//    of the last four.  ld of a subset is ld of the subset without its last variable plus the log of
//    the pivot, in ascending order of the variables whatever the split, so exchangeable n-plets (equal
//    sub-matrices) get equal values and ties stay ordered by index.
//  - k_cube_reduce, one wavefront per (row, size): the n-plets P + (subsets of one size) have
//    consecutive global indices and read consecutive entries of the rows of P without one member;
//    removing one of the ten variables stays inside the row (a table of neighbours in LDS).
// Bound by the latency and bandwidth of the table reads (k + 1 of 8 bytes per n-plet; 67% of the wave
// cycles wait).  N = 25, orders 3..25, top-100 and 256 bins: 4.7 ms with a factorisation per n-plet and
// prefix sharing, 1.2 ms so (build 0.27, bounds 0.09, reduction 0.84); with the orders one after the
// other in the grid, instead of all orders of a chunk of rows together, the reduction took 1.46 ms.
#include "nplets_cube.hpp"
#include "radix_pick.hpp"

namespace thoi {
namespace {

constexpr int kBuildThreads = 256;                    // four rows
constexpr int kBuildWaves = kBuildThreads / 64;
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

// 1/x to the last bit or so (two Newton steps on the hardware estimate); the caller tests x.
__device__ __forceinline__ double fast_rcp(double x)
{
    double y = __builtin_amdgcn_rcp(x);
    y = __builtin_fma(__builtin_fma(-x, y, 1.0), y, y);
    return __builtin_fma(__builtin_fma(-x, y, 1.0), y, y);
}

// Subsets of suffix variables V..9 over the Schur complement s (lower triangle of variables V..9,
// row i - V): ld of every one into row[position], starting from ld and the subset m of the variables
// below V.
template <int V>
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
        cube_walk<V + 1>(x, ld, m, row, spos);
        const double p = s[0], inv = fast_rcp(p);
        sfor<1, n>([&](auto I) {
            const double t = s[tri(I, 0)] * inv;
            sfor<1, I + 1>([&](auto J) { y[tri(I - 1, J - 1)] = __builtin_fma(-t, s[tri(J, 0)], s[tri(I, J)]); });
        });
        cube_walk<V + 1>(y, ld + log(p), m | (1 << V), row, spos);
    }
}

// grid (ceil(2^h / 4), datasets of the group), block kBuildThreads: row P of the table of dataset
// d0 + blockIdx.y.  Bit h - 1 - v of P is variable v.  Rows with more than kmax members are not needed.
__global__ __launch_bounds__(kBuildThreads) void k_cube_build(const double* __restrict__ Sigma, int N, int64_t d0,
                                                              int kmax, double* __restrict__ table)
{
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
    const uint32_t P = __builtin_amdgcn_readfirstlane(blockIdx.x * kBuildWaves + wv);
    const int p = __popc(P);
    if ((P >> h) != 0 || p > kmax) return;                             // no block barrier below
    double* srow = srow_w + wv * kCubeRow;
    double* scol = scol_w + wv * 64;
    double* ssch = ssch_w + wv * 56;
    // lanes 0..9: the suffix variables; lane 10 + q: the q-th member of P (ascending).  r[m], m < 10:
    // entry against suffix variable m; r[10 + q]: against member q.
    const bool suf = lane < kCubeSuffix;
    const int q = lane - kCubeSuffix;
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
            const double t = r[kCubeSuffix + j] * fast_rcp(pj);
            sfor<j + 1, kCubePrefix>([&](auto Q) {
                constexpr int c = Q;
                if (c < p) r[kCubeSuffix + c] = __builtin_fma(-t, cl[kCubeSuffix + c], r[kCubeSuffix + c]);
            });
            sfor<0, kCubeSuffix>([&](auto M) { r[M] = __builtin_fma(-t, cl[M], r[M]); });
        }
    });
    const double lp = log(piv);
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
            const double pt = s[tri(t, t)], inv = fast_rcp(pt);
            ld += log(pt);
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
    cube_walk<6>(s4, ld, lane, srow, spos);
    cube_wave_sync();
    // sizes up to kmax - p are needed, a prefix of the row
    const int need = kmax - p >= kCubeSuffix ? kCubeRow : kSuffix.off[kmax - p + 1];
    double* out = table + ((int64_t)blockIdx.y << N) + ((int64_t)P << kCubeSuffix);
    for (int i = lane; i < need; i += 64) out[i] = srow[i];
}

size_t build_lds_bytes(int N)
{
    return ((size_t)N * N + 2 * N + kBuildWaves * (kCubeRow + 64 + 56)) * 8 + kCubeRow * 2;
}

// The orders of a call: block (chunk c, order i) of the reduction takes order p[i].k of the rows
// [c * per, (c + 1) * per).
struct CubePiece {
    int32_t k, pad;
    int64_t pos0;                                      // position of the order's first n-plet
};
struct CubeTable {
    int32_t n, per, chunks, pad;
    CubePiece p[kCubeMaxN + 1];
};

// sum_j (ld(S \ j) - ld(S)) of entry e of row P (size b, len entries of that size), j ascending: the
// members of P (uniform in the wavefront), eight reads in flight, then the b members among the ten,
// whose positions in the row are nb[0], nb[len], ...
__device__ __forceinline__ double cube_leave_one_out(const double* __restrict__ T, uint32_t P, int b, int len, int e,
                                                     double t0, const uint16_t* nb)
{
    double sa = 0.0;
    uint32_t m = P;
    while (m) {
        double v[8];
        uint32_t mm = m;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            v[u] = t0;
            if (mm) {
                const uint32_t bit = 0x80000000u >> __builtin_clz(mm);
                v[u] = T[((int64_t)(P ^ bit) << kCubeSuffix) + e];
                mm ^= bit;
            }
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (m) {
                sa += v[u] - t0;
                m ^= 0x80000000u >> __builtin_clz(m);
            }
    }
    const double* row = T + ((int64_t)P << kCubeSuffix);
    for (int t = 0; t < b; t += 5) {
        int at[5];
        double v[5];
#pragma unroll
        for (int u = 0; u < 5; ++u) at[u] = nb[(t + u < b ? t + u : b - 1) * len];
#pragma unroll
        for (int u = 0; u < 5; ++u) v[u] = row[at[u]];
#pragma unroll
        for (int u = 0; u < 5; ++u) sa += t + u < b ? v[u] - t0 : 0.0;
    }
    return sa;
}

// ------------------------------------------------------------------------------------------------
// Admission bounds before the reduction.  A workgroup that starts with empty lists inserts almost
// every value of its first iterations, at about 7,000 cycles per insertion: so kSampleGroups
// workgroups per order first evaluate n-plets spread over the order and each finds a key that its
// share of the K best reach; all groups together then hold K distinct n-plets up to the largest of
// these keys, and the reduction meets them again.  A wavefront takes the 64-entry piece of a run that
// holds an evenly spaced rank, so its reads are as coalesced as the reduction's (n-plets at single
// ranks, scattered over the table: 224 us against 85 at N = 25).  Orders with
// fewer n-plets than kSampleMin have no bound: below 64 ranks apart two pieces could coincide.
// ------------------------------------------------------------------------------------------------
constexpr int kSampleThreads = 1024;
constexpr int kSamplePer = 8;                          // pieces per wavefront
constexpr int kSampleGroups = 8;
constexpr uint32_t kSamplePieces = kSampleThreads / 64 * kSamplePer * kSampleGroups;
constexpr uint32_t kSampleMin = kSamplePieces * 64;

// grid (kSampleGroups, orders, datasets of the group): sbound[dataset of the group][order][group][2].
__global__ __launch_bounds__(kSampleThreads) void k_cube_sample(EvalArgs a, CubeTable tab, int K, int64_t d0,
                                                                const double* __restrict__ table,
                                                                uint64_t* __restrict__ sbound)
{
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
    if (total < kSampleMin) {                          // uniform
        if (tid < 2) out[tid] = kKeyEmpty;
        return;
    }
    for (int i = tid; i < N * (k + 1); i += kSampleThreads) sbin[i] = (uint32_t)kPascal.v[i / (k + 1)][i % (k + 1)];
    for (int i = tid; i < kCubeSuffix * kCubeRow / 2; i += kSampleThreads) snbr[i] = kSuffix.nbr[i];
    if (tid == 0) bias_for(a.bias, k, sbias[0], sbias[1], sbias[2]);
    __syncthreads();
    const double* T = table + ((int64_t)blockIdx.z << N);
    double om[kSamplePer];
    int nv = 0;
#pragma unroll
    for (int u = 0; u < kSamplePer; ++u) {
        const uint32_t s = ((uint32_t)u * (kSampleThreads / 64) + wv) * kSampleGroups + blockIdx.x;
        uint32_t r = (uint32_t)((uint64_t)s * total / kSamplePieces);
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
        const double t0 = T[((int64_t)P << kCubeSuffix) + e];
        const double sa = cube_leave_one_out(T, P, b, len, e, t0, snbr + kSuffix.noff[b] + (on ? i : 0));
        const double TC = -0.5 * t0 + sbias[0], DTC = 0.5 * (t0 + sa) + sbias[1];
        om[u] = on && isfinite(t0) && isfinite(sa) ? TC - DTC : __builtin_nan("");
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
                    const uint32_t hw = (uint32_t)(red_list_key(l, om[u]) >> 32);
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
__global__ void k_cube_bounds(CubeTable tab, RedArgs red, int64_t d0, const uint64_t* __restrict__ sbound)
{
    const int l = threadIdx.x;
    if (l >= 2) return;
    const uint64_t* b = sbound + ((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * kSampleGroups * 2 + l;
    uint64_t worst = 0;
    for (int g = 0; g < kSampleGroups; ++g) worst = b[2 * g] > worst ? b[2 * g] : worst;
    if (worst != kKeyEmpty)
        atomicMax(red.bound + ((d0 + blockIdx.y) * (red.kmax + 1) + tab.p[blockIdx.x].k) * 2 + l, (unsigned long long)~worst);
}

// grid (8 ceil(chunks / 8) orders, datasets of the group), block 256.
__global__ __launch_bounds__(256) void k_cube_reduce(EvalArgs a, CubeTable tab, RedArgs red, int64_t d0,
                                                     const double* __restrict__ table)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double sbias[3];
    const int N = a.N, h = N - kCubeSuffix;
    // all orders of one chunk of rows run together on one XCD (workgroups are dealt to the 8 XCDs
    // round robin), so the rows and their neighbours are read from its L2
    const int xcd = (int)blockIdx.x % 8, loc = (int)blockIdx.x / 8;
    const int chunk = loc / tab.n * 8 + xcd;
    const CubePiece pc = tab.p[loc % tab.n];
    if (chunk >= tab.chunks) return;                                   // uniform
    const int k = pc.k;
    const int64_t d = d0 + blockIdx.y;
    uint16_t* snbr = reinterpret_cast<uint16_t*>(smem);                // [5120]
    uint32_t* sbin = reinterpret_cast<uint32_t*>(snbr + kCubeSuffix * kCubeRow / 2);   // C(n, m), n < N, m <= k
    const size_t off = (kCubeSuffix * kCubeRow + (size_t)kCubeMaxN * (kCubeMaxN + 1) * 4 + 15) / 16 * 16;
    RedLds S = red_view(smem + off, red.topk, red.bins);
    for (int i = threadIdx.x; i < kCubeSuffix * kCubeRow / 2; i += 256) snbr[i] = kSuffix.nbr[i];
    for (int i = threadIdx.x; i < N * (k + 1); i += 256) sbin[i] = (uint32_t)kPascal.v[i / (k + 1)][i % (k + 1)];
    if (threadIdx.x == 0) bias_for(a.bias, k, sbias[0], sbias[1], sbias[2]);
    red_begin(S, red, (int)d, k);                                      // ends with a barrier
    const int wv = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const double* T = table + ((int64_t)blockIdx.y << N);
    const uint32_t nrows = 1u << h;
    const uint32_t r0 = (uint32_t)chunk * (uint32_t)tab.per;
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
        for (int i0 = 0; i0 < len; i0 += 64) {
            const int i = i0 + lane;
            const bool on = i < len;
            const int e = o0 + (on ? i : 0);
            const double t0 = T[((int64_t)P << kCubeSuffix) + e];
            const double sa = cube_leave_one_out(T, P, b, len, e, t0, snbr + kSuffix.noff[b] + (on ? i : 0));
            FactorOut<double> f;
            f.ld = t0;
            f.sa = sa;
            f.vmax = 1.0;
            f.ok = true;                                               // a pivot <= 0 leaves NaN or -inf in ld
            double omega = 0.0;
            const int64_t pos = pc.pos0 + rank0 + i;
            bool valid = false;
            if (on)
                valid = store_result<double>(a, true, (int)d, pos, k, f, 0.0, sbias[0], sbias[1], sbias[2], true, omega);
            red_push(S, red, k, valid, omega, a.g_begin + pos);
        }
    }
    red_end(S, red, a.hdr, (int)d, k);
}

size_t reduce_lds_bytes(const RedArgs& red)
{
    return (kCubeSuffix * kCubeRow + (size_t)kCubeMaxN * (kCubeMaxN + 1) * 4 + 15) / 16 * 16 + red_lds_bytes(red.topk, red.bins);
}

// Chunks of rows: a wavefront spends about as long on the start of a (row, size) run as on two of its
// 64-entry iterations, so the work of a call is the sum over its runs of 2 + iterations; about 128 per
// workgroup, a power of two of at least 16 rows, at most 512 chunks (each workgroup leaves a segment to
// merge).
CubeTable cube_table(int N, int kmin, int kmax)
{
    CubeTable t{};
    const int h = N - kCubeSuffix;
    const int64_t rows = int64_t(1) << h;
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
    const int64_t want = work / (128 * t.n);
    int64_t chunks = 8;
    while (chunks < want && chunks < 512) chunks *= 2;
    while (rows / chunks < 16) chunks /= 2;
    t.chunks = (int32_t)chunks;
    t.per = (int32_t)(rows / chunks);
    return t;
}

int64_t cube_blocks(const CubeTable& t) { return (int64_t)(t.chunks + 7) / 8 * 8 * t.n; }

}  // namespace

bool cube_wanted(int32_t N, int64_t D, const thoi_nplets* sel, const thoi_eval_opts* opts)
{
    if (sel->mode != THOI_SEL_RANGE || opts->precision != THOI_FP64 || !opts->reduce || D < 1) return false;
    // orders 1 and 2 have Omega = 0 up to rounding: their lists would be ordered by other rounding
    if (sel->kmin < 3) return false;
    if (opts->engine != THOI_ENGINE_AUTO || N < kCubeMinN || N > kCubeMaxN) return false;
    // whole orders only, and enough of the subsets that the table holds
    int64_t all = 0, need = 0;
    for (int k = sel->kmin; k <= sel->kmax; ++k) all += (int64_t)binom_u64(N, k);
    for (int k = 0; k <= sel->kmax; ++k) need += (int64_t)binom_u64(N, k);
    if (sel->g_begin != 0 || sel->g_count != all) return false;
    return sel->kmax >= 8 && all >= need / 8;
}

int64_t cube_group(int32_t N, int64_t D)
{
    // tables of up to 256 MB together, at least one dataset's
    const int64_t g = (int64_t(1) << 28) >> (N + 3);
    return g < 1 ? 1 : (g < D ? g : D);
}

size_t cube_table_bytes(int32_t N, int64_t D)
{
    // the tables, then the sample keys of every order
    return (size_t)cube_group(N, D) * (((size_t)8 << N) + (size_t)(N + 1) * kSampleGroups * 16);
}

int64_t cube_segments(int32_t N, int kmin, int kmax)
{
    return cube_blocks(cube_table(N, kmin, kmax));
}

void cube_launch(const EvalArgs& a, const RedArgs& red, int kmin, int kmax, double* table, hipStream_t s)
{
    static_assert(sizeof(kSuffixHost.nbr) == kCubeSuffix * kCubeRow, "one neighbour per element");
    const CubeTable tab = cube_table(a.N, kmin, kmax);
    const int64_t blocks = cube_blocks(tab);
    const int64_t rows = int64_t(1) << (a.N - kCubeSuffix);
    const int64_t group = cube_group(a.N, a.D);
    for (int64_t d0 = 0; d0 < a.D; d0 += group) {
        const int64_t nd = d0 + group < a.D ? group : a.D - d0;
        hipLaunchKernelGGL(k_cube_build, dim3((unsigned)((rows + kBuildWaves - 1) / kBuildWaves), (unsigned)nd),
                           dim3(kBuildThreads), build_lds_bytes(a.N), s, a.Sigma, a.N, d0, kmax, table);
        if (red.topk > 0) {
            uint64_t* sbound = reinterpret_cast<uint64_t*>(table + (group << a.N));
            hipLaunchKernelGGL(k_cube_sample, dim3(kSampleGroups, (unsigned)tab.n, (unsigned)nd), dim3(kSampleThreads), 0, s,
                               a, tab, red.topk, d0, table, sbound);
            hipLaunchKernelGGL(k_cube_bounds, dim3((unsigned)tab.n, (unsigned)nd), dim3(64), 0, s, tab, red, d0, sbound);
        }
        hipLaunchKernelGGL(k_cube_reduce, dim3((unsigned)blocks, (unsigned)nd), dim3(256), reduce_lds_bytes(red), s, a, tab,
                           red, d0, table);
    }
}

}  // namespace thoi
