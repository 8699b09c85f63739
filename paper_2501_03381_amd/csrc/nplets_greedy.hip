// Greedy growth run on the device (Methods, "Heuristics", "Greedy Algorithm"): from the kappa
// best n-plets of one order, every solution is extended by every variable it lacks, all
// candidates of the next order are evaluated, and the kappa best are kept; the orders follow one
// another with no host round trip (two launches per order).  The objective is one measure (TC,
// DTC, O-information or S-information) in one dataset, or its mean or paired effect size over D
// datasets (Discussion: functions of the measures optimised across datasets).
//
// Candidate (p, v) is solution p extended by variable v.  A candidate reached from several parents
// is evaluated once, from the first of them (the lowest p whose solution is a subset of it).  One
// 64-lane workgroup per candidate and dataset factors its correlation block (FP64), taking the
// sums of the logs in variable order, so candidates that differ only by which independent
// variable they hold get bit-identical values.  One workgroup then forms each candidate's
// objective, sorts the candidates of the order by it and, among equal values, by the n-plet in
// lexicographic order (the smaller first), and keeps the first kappa.
#include "thoi_internal.hpp"
#include "nplets_common.hpp"
#include "objective_common.hpp"
#include "pair_factor_lat.hpp"
#include "radix_pick.hpp"
#include "search_mask.hpp"

namespace thoi {
namespace {

constexpr int kSelThreads = 1024;
// Wavefronts of an order up to which the evaluation is latency-bound, two per SIMD.  N = 100, 16
// solutions, orders 4..32, ms plain / arranged for latency: 800 wavefronts 2.58 / 2.45, 1600 2.65 / 2.64,
// 2400 2.77 / 2.90, 6400 3.55 / 3.70, 12,800 4.92 / 5.22.
constexpr int kLatWaves = 2048;
constexpr int kSelMax = 4096;           // candidates of one order that the selection sorts in LDS

__device__ __forceinline__ bool has(const Mask& m, int v) { return (m.w[v >> 6] >> (v & 63)) & 1ull; }

__device__ __forceinline__ bool subset(const Mask& a, const Mask& b)
{
    return (a.w[0] & ~b.w[0]) == 0 && (a.w[1] & ~b.w[1]) == 0;
}

// a before b in lexicographic order of the sorted index tuples (equal orders): the lowest variable
// in which they differ belongs to a
__device__ __forceinline__ bool lex_less(const Mask& a, const Mask& b)
{
    const uint64_t x0 = a.w[0] ^ b.w[0];
    if (x0) return (a.w[0] >> __builtin_ctzll(x0)) & 1ull;
    const uint64_t x1 = a.w[1] ^ b.w[1];
    if (x1) return (a.w[1] >> __builtin_ctzll(x1)) & 1ull;
    return false;
}

// total order on doubles as uint64 (-0.0 folded onto +0.0)
__device__ __forceinline__ uint64_t okey(double x)
{
    if (x == 0.0) x = 0.0;
    const uint64_t u = (uint64_t)__double_as_longlong(x);
    return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}

struct GreedyArgs {
    const double* Sigma;    // [D][N][N]
    int D;
    int N;
    int kappa;
    int measure;            // 0 TC, 1 DTC, 2 Omega, 3 S
    int kind;               // THOI_OBJ_MEAN or THOI_OBJ_PAIRED_EFFECT over the D datasets
    double sign;            // +1: keep the largest objective, -1: the smallest
    Mask* sols;             // [steps + 1][kappa]; slot 0 holds the first order's solutions
    double* vals;           // [steps + 1][kappa]
    int32_t* count;         // [steps + 1]
    Mask* cmask;            // [kappa * N] candidates of the current step
    double* meas;           // [D][kappa * N] their measure (NaN: not a candidate or not positive definite)
};

// grid (kappa * N, D), block 64: candidate (p, v) = blockIdx.x / N, % N of step s (order k + 1)
// in dataset blockIdx.y.  Dynamic LDS: the factorisation block, kc rows of stride kc + 1 for the
// step's order kc (sized per step, so that short orders leave room for more wavefronts per CU).
__global__ __launch_bounds__(64) void k_greedy_eval(GreedyArgs g, int s, int kc)
{
    extern __shared__ double sM[];
    const int ks = kc + 1;
    __shared__ double sInv[64], sIsd[64], sSeq[128];
    __shared__ int cidx[64];
    const int N = g.N;
    const int p = blockIdx.x / N, v = blockIdx.x % N;
    const int lane = threadIdx.x;
    const int d = blockIdx.y;
    const int64_t slot = blockIdx.x;
    double* meas = g.meas + (int64_t)d * g.kappa * N;
    const double* Sig = g.Sigma + (int64_t)d * N * N;
    const int cnt = g.count[s];
    const Mask* sol = g.sols + (int64_t)s * g.kappa;
    // uniform in the workgroup: a parent that exists, a variable it lacks, and no earlier parent
    // reaching the same n-plet
    bool use = p < cnt && !has(sol[p], v);
    Mask C{};
    if (use) {
        C = sol[p];
        C.w[v >> 6] |= 1ull << (v & 63);
        for (int q = lane; q < p; q += 64) use = use && !subset(sol[q], C);
        use = __all(use);                      // __all over the wavefront: every earlier parent checked
        use = use && popc(C) <= kc;            // the step's order by construction; the block holds no more
    }
    if (!use) {
        if (lane == 0) meas[slot] = __builtin_nan("");
        return;
    }
    int k = popc(C);
    k = k < 64 ? k : 64;
    int ci = 0;
    if (lane < k) {
        ci = nth_set(C, lane);                 // lane j takes the (j+1)-th member
        cidx[lane] = ci;
        const double dj = Sig[(int64_t)ci * N + ci];
        sIsd[lane] = dj > 0.0 ? 1.0 / sqrt(dj) : __builtin_nan("");
    }
    __syncthreads();
    if (lane < k) gather_row(Sig + (int64_t)ci * N, cidx, sIsd, lane, sM + lane * ks);
    __syncthreads();
    const FactorOut<double> f = wave_factor_core(k, sM, ks, sInv, sSeq);
    if (lane == 0) {
        const bool ok = f.ok && isfinite(f.ld) && isfinite(f.sa);
        const double TC = -0.5 * f.ld, DTC = 0.5 * (f.ld + f.sa);
        const double m = g.measure == 0 ? TC : g.measure == 1 ? DTC : g.measure == 2 ? TC - DTC : TC + DTC;
        if (d == 0) g.cmask[slot] = C;
        meas[slot] = ok ? m : __builtin_nan("");
    }
}

// grid (ceil(kappa * N / 2), D), block 64: two candidate slots per wavefront (half-wave h takes
// slot 2 blockIdx.x + h), factored with the rows in registers; for steps whose order is at most
// kW2Max.  The same candidates, measures and sums in variable order as k_greedy_eval.  LAT: the
// factorisation arranged for latency, for up to kLatWaves wavefronts; with more of them its
// registers cost more than it gains (also 200 datasets of 40 variables, 32 solutions, orders
// 4..30: 22.3 ms against 20.2).
template <bool LAT>
__global__ __launch_bounds__(64) void k_greedy_eval_pair(GreedyArgs g, int s)
{
    __shared__ double scol[2 * 2 * kW2Max], swrow[2 * 2 * kW2Max];
    __shared__ int sch[2 * kW2Max];
    const int N = g.N;
    const int lane = threadIdx.x, h = lane >> 5, i = lane & 31;
    const int64_t slot = 2 * (int64_t)blockIdx.x + h;
    const int64_t nslot = (int64_t)g.kappa * N;
    const int d = blockIdx.y;
    double* meas = g.meas + (int64_t)d * nslot;
    const double* Sig = g.Sigma + (int64_t)d * N * N;
    const int cnt = g.count[s];
    const Mask* sol = g.sols + (int64_t)s * g.kappa;
    const int p = slot < nslot ? (int)(slot / N) : 0, v = slot < nslot ? (int)(slot % N) : 0;
    // uniform in the half-wave: a slot that exists, a parent that exists, a variable it lacks, and
    // no earlier parent reaching the same n-plet
    bool use = slot < nslot && p < cnt && !has(sol[p], v);
    Mask C{};
    if (use) {
        C = sol[p];
        C.w[v >> 6] |= 1ull << (v & 63);
    }
    bool lane_ok = true;
    if (use)
        for (int q = i; q < p; q += 32) lane_ok = lane_ok && !subset(sol[q], C);
    const uint64_t bad = __ballot(!lane_ok);               // whole wavefront active
    use = use && ((bad >> (32 * h)) & 0xffffffffull) == 0;
    int kh = use ? popc(C) : 0;
    kh = kh < kW2Max ? kh : kW2Max;
    int* ch = sch + h * kW2Max;
    if (i < kh) ch[i] = nth_set(C, i);
    wave_sync();
    const int k0 = __shfl(kh, 0), k1 = __shfl(kh, 32);
    const int ku = k0 > k1 ? k0 : k1;
    double* col = scol + h * 2 * kW2Max;
    double* wrow = swrow + h * 2 * kW2Max;
    FactorOut<double> f;
    if constexpr (LAT) f = pair_factor_lat<PairSource::Global, true>(Sig, N, ch, ku, kh, col, wrow);
    else f = pair_factor<true, true>(Sig, N, ch, ku, kh, col, wrow);
    if (i == 0 && slot < nslot) {
        if (!use) {
            meas[slot] = __builtin_nan("");
        } else {
            const bool ok = f.ok && isfinite(f.ld) && isfinite(f.sa);
            const double TC = -0.5 * f.ld, DTC = 0.5 * (f.ld + f.sa);
            const double m = g.measure == 0 ? TC : g.measure == 1 ? DTC : g.measure == 2 ? TC - DTC : TC + DTC;
            if (d == 0) g.cmask[slot] = C;
            meas[slot] = ok ? m : __builtin_nan("");
        }
    }
}

constexpr int kSelChunk = 128;         // entries one wavefront sorts on its own (two per lane)

// Entry (kx, ix) goes before entry (ky, iy): the smaller key, or equal valid keys and the
// lexicographically smaller n-plet (valid slots hold distinct n-plets, so the order is strict there).
__device__ __forceinline__ bool sel_before(uint64_t kx, int ix, uint64_t ky, int iy, const Mask* msk)
{
    if (kx != ky) return kx < ky;
    return ky != ~0ull && lex_less(msk[ix], msk[iy]);
}

// grid 1, block kSelThreads: the objective of each of the ncand = kappa * N slots of step s, then
// the kappa best distinct n-plets in order as step s + 1.
//
// Selection before sorting: a radix selection over the upper key words (four passes of 8 bits) finds a
// key that kappa slots reach, and only the slots up to it (kappa and the ties of that word) are
// sorted.  1600 slots: 12 us; sorting all of them took 19.6 us, most of it the sort.
//
// The sort: bitonic in LDS of the P >= n (a power of two) keys and slots.  Thread
// 1024 j + 64 w + r of a stage with stride <= 64 exchanges entries of the 128-entry chunk
// 2048 j + 128 w only, so between two such stages wavefront w waits for itself alone; a stage that
// follows or precedes one with a wider stride (or the fill) waits for the block.  When kappa <= 128
// only the best 128 entries are needed: once every chunk is sorted (chunk c ascending when c is
// even, else descending), pairs of chunks are merged keeping the lower half only.  Entry-wise
// minimum of an ascending and a descending chunk is the 128 smallest of the two as a bitonic
// sequence; one wavefront sorts it (strides 64..1) ascending or descending as the next merge needs,
// and the number of chunks halves, until chunk 0 holds the best 128 in order.
__global__ __launch_bounds__(kSelThreads) void k_greedy_select(GreedyArgs g, int s)
{
    __shared__ uint64_t key[kSelMax];
    __shared__ int idx[kSelMax];            // entry (into msk) ...
    __shared__ Mask msk[kSelMax];           // ... its n-plet, read for the lexicographic ties
    __shared__ int slot_of[kSelMax];        // ... and its candidate slot
    __shared__ uint32_t rh[256];
    __shared__ uint32_t sprefix;
    __shared__ int srank, sn;
    constexpr int kPer = kSelMax / kSelThreads;
    const int ncand = g.kappa * g.N;
    const int tid = threadIdx.x;
    uint64_t kk[kPer];
    int nv = 0;
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        const int i = tid + u * kSelThreads;
        const double o = i < ncand ? objective_of<double>(g.meas, g.D, ncand, i, g.kind) : __builtin_nan("");
        // ascending key = better first; invalid slots are left out
        kk[u] = isnan(o) ? ~0ull : (g.sign > 0.0 ? ~okey(o) : okey(o));
    }
    if (tid == 0) { sprefix = 0; srank = g.kappa; sn = 0; }
#pragma unroll
    for (int u = 0; u < kPer; ++u) nv += __syncthreads_count(kk[u] != ~0ull);
    uint32_t upto = 0xffffffffu;
    if (nv > g.kappa) {                     // uniform
        for (int pass = 3; pass >= 0; --pass) {
            if (tid < 256) rh[tid] = 0;
            __syncthreads();
            const uint32_t pre = sprefix;
#pragma unroll
            for (int u = 0; u < kPer; ++u) {
                const uint32_t h = (uint32_t)(kk[u] >> 32);
                if (kk[u] != ~0ull && radix_match(h, pre, pass))
                    atomicAdd(&rh[(h >> (8 * pass)) & 255u], 1u);
            }
            __syncthreads();
            if (tid < 64) radix_pick(rh, tid, pass, sprefix, srank);
            __syncthreads();
        }
        upto = sprefix;
    }
#pragma unroll
    for (int u = 0; u < kPer; ++u) {
        if (kk[u] != ~0ull && (uint32_t)(kk[u] >> 32) <= upto) {
            const int e = atomicAdd(&sn, 1);
            const int i = tid + u * kSelThreads;
            key[e] = kk[u];
            idx[e] = e;
            msk[e] = g.cmask[i];
            slot_of[e] = i;
        }
    }
    __syncthreads();
    const int nsel = sn;
    int P = 1;
    while (P < nsel) P <<= 1;
    for (int i = nsel + tid; i < P; i += kSelThreads) { key[i] = ~0ull; idx[i] = -1; }
    const bool topk = g.kappa <= kSelChunk && P > kSelChunk;
    const int top = topk ? kSelChunk : P;
    bool wide = true;
    for (int size = 2; size <= top; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            const bool w = stride > 64;
            if (w || wide) __syncthreads();
            else wave_sync();
            wide = w;
            for (int i = threadIdx.x; i < (P >> 1); i += kSelThreads) {
                const int lo = 2 * i - (i & (stride - 1)), hi = lo + stride;
                const bool asc = (lo & size) == 0;
                const uint64_t ka = key[lo], kb = key[hi];
                const int ia = idx[lo], ib = idx[hi];
                if (sel_before(kb, ib, ka, ia, msk) == asc) { key[lo] = kb; key[hi] = ka; idx[lo] = ib; idx[hi] = ia; }
            }
        }
    }
    if (topk) {
        // P / 128 <= 32 chunks; merge r pairs chunk 2^r w (ascending) with chunk 2^r w + 2^(r-1)
        // (descending) in wavefront w, for w below the number of chunks left
        const int wv = threadIdx.x >> 6, ln = threadIdx.x & 63;
        const int nch = P / kSelChunk;
        for (int r = 1; (1 << r) <= nch; ++r) {
            __syncthreads();
            if (wv < (nch >> r)) {
                const int a = (wv << r) * kSelChunk, b = a + (1 << (r - 1)) * kSelChunk;
                const bool asc = (wv & 1) == 0;
                for (int j = ln; j < kSelChunk; j += 64) {
                    const uint64_t ka = key[a + j], kb = key[b + j];
                    const int ia = idx[a + j], ib = idx[b + j];
                    if (sel_before(kb, ib, ka, ia, msk)) { key[a + j] = kb; idx[a + j] = ib; }
                }
                for (int stride = 64; stride > 0; stride >>= 1) {
                    wave_sync();
                    const int lo = a + 2 * ln - (ln & (stride - 1)), hi = lo + stride;
                    const uint64_t ka = key[lo], kb = key[hi];
                    const int ia = idx[lo], ib = idx[hi];
                    if (sel_before(kb, ib, ka, ia, msk) == asc) {
                        key[lo] = kb; key[hi] = ka; idx[lo] = ib; idx[hi] = ia;
                    }
                }
            }
        }
    }
    __syncthreads();
    // the valid slots come first and are distinct n-plets: the first min(kappa, valid) are kept,
    // one thread each
    const int t = threadIdx.x;
    const int n = nsel < g.kappa ? nsel : g.kappa;
    if (t < n) {
        const int i = idx[t];
        g.sols[(int64_t)(s + 1) * g.kappa + t] = msk[i];
        g.vals[(int64_t)(s + 1) * g.kappa + t] = objective_of<double>(g.meas, g.D, ncand, slot_of[i], g.kind);
    }
    if (t == 0) g.count[s + 1] = n;
}

}  // namespace

size_t greedy_ws_bytes(int64_t D, int32_t N, int32_t kappa)
{
    return (size_t)kappa * N * (sizeof(Mask) + 8 * (size_t)D) + 256;
}

int greedy_select_max() { return kSelMax; }

thoi_status launch_greedy(const double* Sigma, int64_t D, int32_t N, int32_t k_first, int32_t kappa, int32_t steps,
                          int32_t measure, int32_t kind, int32_t maximize, uint64_t* sols, double* vals, int32_t* count,
                          void* ws, hipStream_t s)
{
    GreedyArgs g{};
    g.Sigma = Sigma;
    g.D = (int)D;
    g.N = N;
    g.kappa = kappa;
    g.measure = measure;
    g.kind = kind;
    g.sign = maximize ? 1.0 : -1.0;
    g.sols = reinterpret_cast<Mask*>(sols);
    g.vals = vals;
    g.count = count;
    char* base = static_cast<char*>(ws);
    g.cmask = reinterpret_cast<Mask*>(base);
    g.meas = reinterpret_cast<double*>(base + (size_t)kappa * N * sizeof(Mask));
    const int64_t waves = ((int64_t)kappa * N + 1) / 2 * D;
    const auto eval_pair = waves <= kLatWaves ? k_greedy_eval_pair<true> : k_greedy_eval_pair<false>;
    for (int32_t t = 0; t < steps; ++t) {
        // step t builds order k_first + t + 1
        if (k_first + t + 1 <= kW2Max)
            hipLaunchKernelGGL(eval_pair, dim3((unsigned)((kappa * N + 1) / 2), (unsigned)D), dim3(64), 0, s, g, (int)t);
        else {
            const int kc = k_first + t + 1;
            const size_t lds = (size_t)kc * (size_t)(kc + 1) * sizeof(double);
            hipLaunchKernelGGL(k_greedy_eval, dim3((unsigned)(kappa * N), (unsigned)D), dim3(64), lds, s, g, (int)t, kc);
        }
        hipLaunchKernelGGL(k_greedy_select, dim3(1), dim3(kSelThreads), 0, s, g, (int)t);
    }
    return hip_status(hipGetLastError());
}

}  // namespace thoi
