// Gaussian-copula transform on gfx950 (Supplementary, "Estimation of entropy via Gaussian
// copulas", Eq. gaussian_copula_covariance_estimator): every variable of every dataset is
// replaced by Phi^{-1}(r / (T+1)), r its 1-based ordinal rank, equal values ranked by sample
// index.
//
// Design: a column is cut into chunks of kChunk samples.  One workgroup of kChunk threads sorts
// one chunk of (orderable key, sample index) pairs with a bitonic network held in registers:
// partners inside a wavefront are exchanged by cross-lane shuffles, larger distances through LDS.
// With a single chunk the sorted position is the rank.  Otherwise the sorted chunks go to the
// workspace and a merge workgroup per chunk adds, for each of its elements, the number of entries
// before it in every chunk of the column (its own included).
// Every kernel issues its global loads in batches, all in flight together: at these sizes the
// cost is round trips to memory, not bandwidth.
#include "thoi_internal.hpp"

#include <type_traits>

namespace thoi {
namespace {

constexpr int kChunk = 1024;                       // samples per sorted chunk
constexpr int kSortThreads = 1024;
constexpr int kSortReg = kChunk / kSortThreads;    // elements per thread in the sort (one)
constexpr int kMergeThreads = 1024;
constexpr int kMergeReg = kChunk / kMergeThreads;  // elements per thread in the merge
constexpr int kMergeStage = 16;                    // chunks staged in LDS at a time (128 KB of values)

// Monotone map of a double onto uint64 (total order; -0.0 is folded onto +0.0).
__device__ __forceinline__ uint64_t order_key(double x)
{
    if (x == 0.0) x = 0.0;
    uint64_t u = (uint64_t)__double_as_longlong(x);
    return (u >> 63) ? ~u : (u | 0x8000000000000000ull);
}

// Phi^{-1}(r/(T+1)); the upper half uses the exact integer complement, so score(r) = -score(T+1-r).
// One call per score (lanes of a wave would otherwise run both inlined copies).
__device__ __forceinline__ double normal_score(int64_t r, int64_t T)
{
    const int64_t den = T + 1;
    const bool lower = 2 * r <= den;
    const double z = normcdfinv((double)(lower ? r : den - r) / (double)den);
    return lower ? z : -z;
}

template <typename ZT>
__device__ __forceinline__ void store_z(void* Z, int64_t off, double z)
{
    static_cast<ZT*>(Z)[off] = (ZT)z;
}

__device__ __forceinline__ bool pair_less(uint64_t ka, uint32_t ia, uint64_t kb, uint32_t ib)
{
    return ka < kb || (ka == kb && ia < ib);
}

__device__ __forceinline__ uint64_t shfl_xor_u64(uint64_t v, int m)
{
    const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)v, m);
    const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(v >> 32), m);
    return ((uint64_t)hi << 32) | lo;
}

// One stage (block size SIZE, partner distance S) of the bitonic network over the kChunk elements
// of a workgroup, element i = kSortReg * tid + e.  Partners at distance below kSortReg sit in the
// same thread; up to a wavefront's span they are exchanged by cross-lane shuffles; beyond it through
// LDS.
template <int SIZE, int S>
__device__ __forceinline__ void bitonic_stage(uint64_t (&k)[kSortReg], uint32_t (&x)[kSortReg], int tid,
                                              uint64_t* skey, uint32_t* sidx)
{
    if constexpr (S < kSortReg) {
#pragma unroll
        for (int e = 0; e < kSortReg; ++e) {
            if ((e & S) == 0) {
                const bool asc = (((tid * kSortReg) | e) & SIZE) == 0;
                const bool swap = pair_less(k[e | S], x[e | S], k[e], x[e]) == asc;
                const uint64_t ka = k[e], kb = k[e | S];
                const uint32_t ia = x[e], ib = x[e | S];
                k[e] = swap ? kb : ka; k[e | S] = swap ? ka : kb;
                x[e] = swap ? ib : ia; x[e | S] = swap ? ia : ib;
            }
        }
    } else {
        constexpr int m = S / kSortReg;
        uint64_t pk[kSortReg];
        uint32_t px[kSortReg];
        if constexpr (m < 64) {
#pragma unroll
            for (int e = 0; e < kSortReg; ++e) {
                pk[e] = shfl_xor_u64(k[e], m);
                px[e] = (uint32_t)__shfl_xor((int)x[e], m);
            }
        } else {
            __syncthreads();                       // earlier readers of the exchange buffer are done
#pragma unroll
            for (int e = 0; e < kSortReg; ++e) {
                skey[tid * kSortReg + e] = k[e];
                sidx[tid * kSortReg + e] = x[e];
            }
            __syncthreads();
#pragma unroll
            for (int e = 0; e < kSortReg; ++e) {
                pk[e] = skey[(tid ^ m) * kSortReg + e];
                px[e] = sidx[(tid ^ m) * kSortReg + e];
            }
        }
        const bool lower = (tid & m) == 0;
#pragma unroll
        for (int e = 0; e < kSortReg; ++e) {
            const bool asc = (((tid * kSortReg) | e) & SIZE) == 0;
            // the lower element of the pair keeps the smaller one when ascending
            const bool keep = pair_less(k[e], x[e], pk[e], px[e]) == (lower == asc);
            k[e] = keep ? k[e] : pk[e];
            x[e] = keep ? x[e] : px[e];
        }
    }
    if constexpr (S > 1) bitonic_stage<SIZE, S / 2>(k, x, tid, skey, sidx);
}

template <int SIZE>
__device__ __forceinline__ void bitonic_sort(uint64_t (&k)[kSortReg], uint32_t (&x)[kSortReg], int tid,
                                             uint64_t* skey, uint32_t* sidx)
{
    bitonic_stage<SIZE, SIZE / 2>(k, x, tid, skey, sidx);
    if constexpr (SIZE < kChunk) bitonic_sort<SIZE * 2>(k, x, tid, skey, sidx);
}

// grid (nchunks, N, D), block kSortThreads: sorts chunk q of column (d, c).
template <typename ZT>
__global__ __launch_bounds__(kSortThreads) void k_copula_sort(const double* __restrict__ X, int64_t T, int64_t N,
                                                              void* __restrict__ Z, uint64_t* __restrict__ wkey,
                                                              uint32_t* __restrict__ widx,
                                                              int32_t* __restrict__ nanflag, WsHeader* hdr)
{
    __shared__ uint64_t skey[kChunk];
    __shared__ uint32_t sidx[kChunk];
    const int tid = threadIdx.x;
    const int64_t q = blockIdx.x, c = blockIdx.y, d = blockIdx.z;
    const int64_t nchunks = gridDim.x;
    const int64_t t0 = q * kChunk;
    const int n = (int)min<int64_t>(kChunk, T - t0);

    // load: register e of thread j takes sample t0 + kSortThreads e + j (consecutive threads read
    // consecutive rows); all loads are issued before the first use
    const double* Xd = X + d * T * N;
    double v[kSortReg];
#pragma unroll
    for (int e = 0; e < kSortReg; ++e) {
        const int i = kSortThreads * e + tid;
        v[e] = i < n ? Xd[(t0 + i) * N + c] : 0.0;
    }
    uint64_t k[kSortReg];
    uint32_t x[kSortReg];
    int has_nan = 0;
#pragma unroll
    for (int e = 0; e < kSortReg; ++e) {
        const int i = kSortThreads * e + tid;
        const bool in = i < n;
        has_nan |= in && isnan(v[e]);
        k[e] = in ? order_key(v[e]) : ~0ull;
        x[e] = in ? (uint32_t)(t0 + i) : 0xffffffffu;
    }
    const bool bad = __syncthreads_or(has_nan) != 0;
    bitonic_sort<2>(k, x, tid, skey, sidx);

    if (nchunks == 1) {
        if (bad && tid == 0) raise_status(hdr, THOI_EINVAL_DATA);
#pragma unroll
        for (int e = 0; e < kSortReg; ++e) {
            const int p = tid * kSortReg + e;
            if (p < n) store_z<ZT>(Z, (d * T + x[e]) * N + c, bad ? __builtin_nan("") : normal_score(p + 1, T));
        }
    } else {
        // the merge raises the status, after this kernel: clear the header here
        if (q == 0 && c == 0 && d == 0 && tid < (int)(kWsHeader / 4)) reinterpret_cast<int32_t*>(hdr)[tid] = 0;
        const int64_t base = ((d * N + c) * nchunks + q) * (int64_t)kChunk + tid * kSortReg;
#pragma unroll
        for (int e = 0; e < kSortReg; ++e) {
            wkey[base + e] = k[e];      // padding slots too: the merge searches whole chunks
            widx[base + e] = x[e];
        }
        if (tid == 0) nanflag[(d * N + c) * nchunks + q] = bad ? 1 : 0;   // every chunk writes its own flag
    }
}

// grid (nchunks, N*D), block kMergeThreads: the rank of element j of sorted chunk q of column (d, c)
// is its position in chunk q plus, for every other chunk o, the number of entries of o before it.
// Chunks hold contiguous ranges of samples, so an entry of o with an equal value comes before it
// exactly when o < q: the count is a search on the values alone (no sample indices in LDS).
// Chunks are staged kMergeStage at a time in LDS (all loads of a stage in flight together) and
// every element does a branchless fixed-step search in every staged chunk; the searches are
// independent, so a thread keeps many LDS reads in flight.
template <typename ZT>
__global__ __launch_bounds__(kMergeThreads) void k_copula_merge(int64_t T, int64_t N, int nchunks,
                                                                void* __restrict__ Z,
                                                                const uint64_t* __restrict__ wkey,
                                                                const uint32_t* __restrict__ widx,
                                                                const int32_t* __restrict__ nanflag, WsHeader* hdr)
{
    __shared__ uint64_t okey[kMergeStage][kChunk];
    const int tid = threadIdx.x;
    // XCD-aware order: workgroups are dealt round-robin to the 8 XCDs; give consecutive work items
    // (the chunks of one column, which read the same staged chunks) to the same XCD
    const int64_t G = (int64_t)gridDim.x * gridDim.y, b = blockIdx.x + (int64_t)gridDim.x * blockIdx.y;
    const int64_t xcd = b % 8, q8 = G / 8, r8 = G % 8;
    const int64_t w = xcd * q8 + (xcd < r8 ? xcd : r8) + b / 8;
    const int q = (int)(w % nchunks);
    const int64_t cd = w / nchunks;
    const int64_t c = cd % N, d = cd / N;
    const int64_t col = (d * N + c) * nchunks;
    const int nq = (int)min<int64_t>(kChunk, T - (int64_t)q * kChunk);
    // the flags, the thread's own entries and the first stage's chunks are loaded together
    int f = 0;
    for (int o = tid; o < nchunks; o += kMergeThreads) f |= nanflag[col + o];
    bool bad = false;

    const int p0 = tid * kMergeReg;
    uint64_t mk[kMergeReg];
    uint32_t mi[kMergeReg];
    uint32_t rank[kMergeReg];
#pragma unroll
    for (int e = 0; e < kMergeReg; ++e) {
        mk[e] = wkey[(col + q) * (int64_t)kChunk + p0 + e];
        mi[e] = widx[(col + q) * (int64_t)kChunk + p0 + e];
        rank[e] = p0 + e;                                  // entries of its own chunk before it
    }
    for (int o0 = 0; o0 < nchunks; o0 += kMergeStage) {
        // stage chunks o0 .. o0+kMergeStage-1 other than q; slots past the last chunk and chunk q
        // itself are neither loaded nor searched (uniform branches)
        uint64_t lk[kMergeStage][kChunk / kMergeThreads];
#pragma unroll
        for (int s = 0; s < kMergeStage; ++s) {
            if (o0 + s < nchunks && o0 + s != q) {
                const int64_t src = (col + o0 + s) * (int64_t)kChunk;
#pragma unroll
                for (int e = 0; e < kChunk / kMergeThreads; ++e) lk[s][e] = wkey[src + e * kMergeThreads + tid];
            }
        }
        if (o0 == 0) bad = __syncthreads_or(f) != 0;     // uniform
        else __syncthreads();                      // the previous stage's searches are done
#pragma unroll
        for (int s = 0; s < kMergeStage; ++s) {
            if (o0 + s < nchunks && o0 + s != q) {
#pragma unroll
                for (int e = 0; e < kChunk / kMergeThreads; ++e) okey[s][e * kMergeThreads + tid] = lk[s][e];
            }
        }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < kMergeStage; ++s) {
            if (o0 + s >= nchunks || o0 + s == q) continue;
            const bool le = o0 + s < q;           // equal values of an earlier chunk come first
#pragma unroll
            for (int e = 0; e < kMergeReg; ++e) {
                // count of entries before x (v < x, or v <= x for an earlier chunk: v < x + 1; a
                // real key is below ~0, and the padding slots' ranks are never stored): binary
                // digits from the top, then the last entry
                const uint64_t xs = le ? mk[e] + 1 : mk[e];
                int pos = 0;
#pragma unroll
                for (int b = kChunk / 2; b >= 1; b >>= 1) pos += okey[s][pos + b - 1] < xs ? b : 0;
                pos += okey[s][pos] < xs ? 1 : 0;
                rank[e] += pos;
            }
        }
    }
    if (bad && q == 0 && tid == 0) raise_status(hdr, THOI_EINVAL_DATA);
#pragma unroll
    for (int e = 0; e < kMergeReg; ++e) {
        if (p0 + e < nq) {
            const double z = bad ? __builtin_nan("") : normal_score((int64_t)rank[e] + 1, T);
            store_z<ZT>(Z, (d * T + (int64_t)mi[e]) * N + c, z);
        }
    }
}

// ------------------------------------------------------------------------------------------------
// One workgroup per column (kChunk < T <= kColMax, enough columns to fill the chip): the column
// stays in LDS and every sample is ranked by a sample sort.  kSplit samples (one at a jittered
// place of every kSplit-th of the column) are sorted and cut the column into buckets; a sample's
// bucket is a 10-step search, and its rank is the bucket's first position plus the smaller entries
// of the bucket (about T / kSplit of them): some 10 + T / kSplit LDS reads per sample where the
// chunk sort and merge need 55 exchanges and 10 (nchunks - 1) search steps.
//
// Samples are compared by 32-bit codes: the position in [min, max] of the column in units of
// 2^-32 of the range, a monotone map, and by the next 20 bits of that position where codes are
// equal.  What the sorted splitter samples show of a column decides:
//  - hardly any equal codes (continuous values): as above.
//  - equal codes that are equal values (ties): a bucket per splitter as before, but the samples
//    equal to one of r equal splitters are dealt to their buckets by index, which is their order.
//  - many equal codes of different values (an outlier that squeezes the rest), no codes
//    (infinities, a constant column): splitters of the full (key, index) pairs, which are
//    distinct, and the key's two words as code.
// Where equal codes were taken for equal values, or the next bits were equal too, the sorted keys
// are checked at the end, and a column that does not ascend is ranked again by full keys.
//
// 64 datasets of 10,000 x 20, us, chunk sort and merge 827-852 for all of them: continuous 338 (367
// with the bucket read one entry at a time), rounded to one decimal 394 and to three 460 (with full
// keys for every tied column 730 and 727), binary 339 (576), one outlier 449.  About 150 us of it are
// the strided column reads and writes (a 128-byte line for 8 bytes each), the rest LDS latency.  160
// columns of 10,000: chunk path 124, continuous 70, one decimal 80, three 94 (155), binary 68 (123),
// outlier 95.  Telling ties apart costs continuous columns 2 to 3%.  Two workgroups share a CU up to
// 4096 samples: 1280 columns of 3000 take 90 against 125 one by one (and 210 by the chunk path).
// Squeezed columns, fewer than 300 of them, stay slower than the chunk path from 2,049 to 5,000
// samples (160 of 3,000: 44 against 36).
// ------------------------------------------------------------------------------------------------
constexpr int kColMax = 12288;
constexpr int kSplit = 1024;
// Columns from which this path is taken, T up to 2048 and above: fewer take about as long as a
// round of 256, and the chunk path's time grows with them (T = 2048: 21 us up to 128 columns, then
// 34; T = 10,000: 77 for 96, 95 for 128, 124 for 160).  Below the line tied or squeezed columns
// lose more than continuous ones gain.
constexpr int kColMinShort = 144, kColMin = 128;
// equal neighbours among the sorted splitter samples above which ties and shared codes are told
// apart, and above which columns of shared codes get full keys
constexpr int kColTies = 2, kColShared = 16;
static_assert(kSplit == kSortThreads && kSplit == kChunk, "one splitter per thread");

// LDS: base u32 [kSplit + 2] | wave scratch 4 x f64 [16] | bucket heads u64 [T / 64 + 2] | then codes u32 [T],
// lower key words u32 [T] and indices u16 [T]; before those are written, the splitters u64 [kSplit],
// u32 [kSplit]; after them, the ranks u16 [T].
constexpr size_t kColFixed = ((kSplit + 2) * 4 + 15) / 16 * 16 + 4 * 16 * 8;
inline size_t col_lds_bytes(int64_t T)
{
    const size_t body = (size_t)T * 10 > kSplit * 12 ? (size_t)T * 10 : kSplit * 12;
    return kColFixed + (size_t)(T / 64 + 2) * 8 + (body + 15) / 16 * 16 + 16;
}

// the scores of ranks 1..T, once per call, and the cleared header
__global__ __launch_bounds__(256) void k_copula_scores(int64_t T, double* __restrict__ score, WsHeader* hdr)
{
    const int64_t r = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (blockIdx.x == 0 && threadIdx.x < kWsHeader / 4) reinterpret_cast<int32_t*>(hdr)[threadIdx.x] = 0;
    if (r < T) score[r] = normal_score(r + 1, T);
}

// Ascending bitonic sort of one 32-bit code per thread (kSplit threads), as bitonic_sort.
template <int SIZE, int S>
__device__ __forceinline__ void bitonic_stage_u32(uint32_t& k, int tid, uint32_t* sk)
{
    uint32_t o;
    if constexpr (S < 64) {
        o = (uint32_t)__shfl_xor((int)k, S);
    } else {
        __syncthreads();                           // earlier readers of the exchange buffer are done
        sk[tid] = k;
        __syncthreads();
        o = sk[tid ^ S];
    }
    const bool low = ((tid & S) == 0) == ((tid & SIZE) == 0);
    k = low ? min(k, o) : max(k, o);
    if constexpr (S > 1) bitonic_stage_u32<SIZE, S / 2>(k, tid, sk);
}
template <int SIZE>
__device__ __forceinline__ void bitonic_sort_u32(uint32_t& k, int tid, uint32_t* sk)
{
    bitonic_stage_u32<SIZE, SIZE / 2>(k, tid, sk);
    if constexpr (SIZE < kSplit) bitonic_sort_u32<SIZE * 2>(k, tid, sk);
}

// The compiler no longer knows what n holds (no instruction; the host pass has no scalar registers).
__device__ __forceinline__ void forget(int64_t& n)
{
#ifdef __HIP_DEVICE_COMPILE__
    asm volatile("" : "+s"(n));
#endif
}

// Number of the sorted splitters s below code c.
__device__ __forceinline__ int below(const uint32_t* s, uint32_t c)
{
    int pos = 0;
#pragma unroll
    for (int w = kSplit / 2; w >= 1; w >>= 1) pos += s[pos + w - 1] < c ? w : 0;
    return pos + (s[pos] < c ? 1 : 0);
}

// grid (N * D), block kSortThreads; E samples per thread, t = tid + 1024 e.
template <typename ZT, int E>
__device__ __forceinline__ void copula_col(const double* __restrict__ X, int T, int64_t N, void* __restrict__ Z,
                                           const double* __restrict__ score, WsHeader* hdr)
{
    extern __shared__ __align__(16) unsigned char smem[];
    uint32_t* base = reinterpret_cast<uint32_t*>(smem);
    double* wred = reinterpret_cast<double*>(smem + kColFixed - 4 * 16 * 8);
    uint64_t* heads = reinterpret_cast<uint64_t*>(smem + kColFixed);
    unsigned char* body = smem + kColFixed + (size_t)(T / 64 + 2) * 8;
    uint64_t* spk = reinterpret_cast<uint64_t*>(body);
    uint32_t* spi = reinterpret_cast<uint32_t*>(spk + kSplit);
    uint32_t* spc = reinterpret_cast<uint32_t*>(body);
    uint64_t* skey = reinterpret_cast<uint64_t*>(spc + kSplit);
    uint16_t* send = reinterpret_cast<uint16_t*>(skey);
    uint32_t* code = reinterpret_cast<uint32_t*>(body);
    uint32_t* klo = code + T;
    uint16_t* bi = reinterpret_cast<uint16_t*>(klo + T);
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    // XCD-aware order: the columns of one dataset, which share its cache lines, go to one XCD
    const int64_t G = gridDim.x, b = blockIdx.x;
    const int64_t xcd = b % 8, q8 = G / 8, r8 = G % 8;
    const int64_t w = xcd * q8 + (xcd < r8 ? xcd : r8) + b / 8;
    const int64_t c = w % N, d = w / N;
    const double* Xd = X + d * T * N + c;

    // the samples and the thread's splitter candidate (a place in its stratum of the column from a
    // multiplicative hash of the thread index), all loads in flight together
    double v[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int t = tid + kSortThreads * e;
        v[e] = Xd[(int64_t)(t < T ? t : T - 1) * N];
    }
    const int lo_t = (int)((int64_t)tid * T / kSplit), hi_t = (int)((int64_t)(tid + 1) * T / kSplit);
    const int ts = lo_t + (int)(((uint32_t)tid * 2654435761u >> 16) % (uint32_t)(hi_t - lo_t));
    const double vs = Xd[(int64_t)ts * N];
    base[tid] = 0;
    if (tid < 2) base[kSplit + tid] = 0;
    for (int i = tid; i < T / 64 + 2; i += kSortThreads) heads[i] = 0;
    int has_nan = 0;
    double mn = v[0], mx = v[0];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        has_nan |= isnan(v[e]);
        mn = v[e] < mn ? v[e] : mn;
        mx = v[e] > mx ? v[e] : mx;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double y = __shfl_xor(mn, o, 64), z = __shfl_xor(mx, o, 64);
        mn = y < mn ? y : mn;
        mx = z > mx ? z : mx;
    }
    if (lane == 0) { wred[wv] = mn; wred[16 + wv] = mx; }
    const bool bad = __syncthreads_or(has_nan) != 0;
    if (bad) {                                     // uniform
        if (tid == 0) raise_status(hdr, THOI_EINVAL_DATA);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int t = tid + kSortThreads * e;
            if (t < T) store_z<ZT>(Z, (d * T + t) * N + c, __builtin_nan(""));
        }
        return;
    }
    for (int u = 0; u < kSortThreads / 64; ++u) {
        mn = wred[u] < mn ? wred[u] : mn;
        mx = wred[16 + u] > mx ? wred[16 + u] : mx;
    }
    const double scale = 4294967295.0 / (mx - mn);
    // the position plus 2^32, a number in [2^32, 2^33): its mantissa is 32 bits before the point (the code)
    // and 20 after it
    auto place = [&](double x) { return (uint64_t)__double_as_longlong(fma(x - mn, scale, 4294967296.0)); };
    auto code_of = [&](double x) { return (uint32_t)(place(x) >> 20); };
    auto next_bits = [&](double x) { return (uint32_t)place(x); };
    // a constant column, an infinite range or a denormal one has no codes
    bool full = !(mx > mn) || !(scale > 0.0) || !isfinite(scale), tied = false;
    if (!full) {
        const uint32_t own = code_of(vs);
        uint32_t sc = own;
        bitonic_sort_u32<2>(sc, tid, spc);
        __syncthreads();
        spc[tid] = sc;
        __syncthreads();
        const bool first = tid == 0 || spc[tid - 1] != sc;
        const int equal = __syncthreads_count(!first);
        if (equal > kColTies) {
            // ties, or different values that share a code?
            const int a = below(spc, own);
            skey[a] = order_key(vs);
            __syncthreads();
            tied = __syncthreads_or(skey[a] != order_key(vs)) == 0;     // (every lane has read skey)
            full = !tied && equal > kColShared;
            if (tied) {                            // one past the last of the equal splitters
                if (first) send[tid] = (uint16_t)(sc == 0xffffffffu ? kSplit : below(spc, sc + 1));
                __syncthreads();
            }
        }
    }
    uint16_t* srank = reinterpret_cast<uint16_t*>(body);
    // ranks of the samples v into srank; whether equal codes have to be looked at
    auto rank_samples = [&](const double (&v)[E], bool full, bool tied) {
    // bucket = number of splitters before the sample (full keys: at or before) and, of the splitters
    // equal to it (ties), the share that its index is of T
    int bkt[E];
    // code and the next 20 bits, or the key's two words: made together, they let the samples' registers
    // go (with ten samples and more that spills)
    constexpr bool kWords = E <= 8;
    uint32_t cd[E], cl[kWords ? E : 1];
    if (!full) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            cd[e] = code_of(v[e]);
            if constexpr (kWords) cl[e] = next_bits(v[e]);
        }
#pragma unroll
        for (int e = 0; e < E; ++e) bkt[e] = below(spc, cd[e]);
        if (tied) {
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const int pos = bkt[e] < kSplit ? bkt[e] : kSplit - 1;
                if (spc[pos] == cd[e]) {
                    const int r = (int)send[pos] - pos;
                    const int q = (int)((float)((tid + kSortThreads * e) * (r + 1)) / (float)T);
                    bkt[e] += q < r ? q : r;
                }
            }
        }
    } else {
        uint64_t sk[1] = {order_key(vs)};
        uint32_t si[1] = {(uint32_t)ts};
        bitonic_sort<2>(sk, si, tid, spk, spi);
        __syncthreads();
        spk[tid] = sk[0];
        spi[tid] = si[0];
        __syncthreads();
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const uint32_t t = tid + kSortThreads * e;
            const uint64_t key = order_key(v[e]);
            int pos = 0;
#pragma unroll
            for (int s = kSplit / 2; s >= 1; s >>= 1)
                pos += pair_less(spk[pos + s - 1], spi[pos + s - 1], key, t + 1) ? s : 0;
            pos += pair_less(spk[pos], spi[pos], key, t + 1) ? 1 : 0;
            bkt[e] = pos;
            cd[e] = (uint32_t)(key >> 32);
            if constexpr (kWords) cl[e] = (uint32_t)key;
        }
    }
    // counting sort by bucket
#pragma unroll
    for (int e = 0; e < E; ++e)                    // place in the bucket << 11 | bucket (at most kSplit)
        if (tid + kSortThreads * e < T) bkt[e] |= (int)(atomicAdd(&base[bkt[e]], 1u) << 11);
    __syncthreads();
    {
        uint32_t* wsum = reinterpret_cast<uint32_t*>(wred);
        const uint32_t own = base[tid];
        uint32_t incl = own;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) { const uint32_t y = __shfl_up(incl, o, 64); incl += lane >= o ? y : 0u; }
        if (lane == 63) wsum[wv] = incl;
        __syncthreads();
        uint32_t before = 0;
        for (int u = 0; u < wv; ++u) before += wsum[u];
        const uint32_t first = before + incl - own;
        base[tid] = first;                         // first position of bucket tid
        auto mark = [&](uint32_t p) {
            atomicOr(reinterpret_cast<unsigned long long*>(&heads[p >> 6]), 1ull << (p & 63));
        };
        if (own) mark(first);
        if (tid == kSplit - 1) {
            base[kSplit] = before + incl;
            mark(before + incl);                   // the last bucket, or the end when it is empty
            if (before + incl < (uint32_t)T) mark((uint32_t)T);
        }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int t = tid + kSortThreads * e;
        if (t < T) {
            const uint32_t p = base[bkt[e] & 2047] + ((uint32_t)bkt[e] >> 11);
            code[p] = cd[e];
            bi[p] = (uint16_t)t;
            if constexpr (kWords) klo[p] = cl[e];
            else klo[p] = full ? (uint32_t)order_key(v[e]) : next_bits(v[e]);
        }
    }
    __syncthreads();
    // positions in bucket order: the lanes of a wavefront read the same few buckets.  The wavefront's
    // 64 positions share one word of bucket heads; the bucket that reaches into it and the one that
    // reaches out end in the neighbouring words.
    uint32_t rk[E];                                // rank << 16 | index
    bool check = tied;                             // equal codes were taken for equal values
    auto rank_buckets = [&](auto ties) {
    constexpr bool TIED = decltype(ties)::value;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int p = tid + kSortThreads * e;
        rk[e] = 0;
        if (p < T) {
            int wd = p >> 6;
            const uint64_t hw = heads[wd];
            const uint64_t below = hw & ((2ull << lane) - 1ull), above = lane < 63 ? hw >> (lane + 1) : 0ull;
            int lo, hi;
            if (below) {
                lo = (wd << 6) + 63 - __builtin_clzll(below);
            } else {
                int q = wd - 1;                    // bit 0 of word 0 is set
                while (heads[q] == 0) --q;
                lo = (q << 6) + 63 - __builtin_clzll(heads[q]);
            }
            if (above) {
                hi = p + 1 + __builtin_ctzll(above);
            } else {
                int q = wd + 1;                    // bit T is set
                while (heads[q] == 0) ++q;
                hi = (q << 6) + __builtin_ctzll(heads[q]);
            }
            const uint32_t mine = code[p];
            const int t = bi[p];
            uint32_t less = 0, eq = 0, alike = 0;
            if constexpr (TIED) {                  // most codes have equals
                const uint32_t ml = klo[p];
#pragma unroll 2
                for (int q = lo; q < hi; ++q) {
                    const uint32_t o = code[q], ol = klo[q];
                    const int ot = bi[q];
                    const bool same = o == mine && ol == ml;
                    less += (o < mine || (o == mine && ol < ml) || (same && ot < t)) ? 1u : 0u;
                }
            } else {
#pragma unroll 4
                for (int q = lo; q < hi; ++q) {
                    const uint32_t o = code[q];
                    less += o < mine ? 1u : 0u;
                    eq += o == mine ? 1u : 0u;
                }
                if (eq > 1) {
                    const uint32_t ml = klo[p];
                    for (int q = lo; q < hi; ++q)
                        if (code[q] == mine) {
                            const uint32_t ol = klo[q];
                            less += (ol < ml || (ol == ml && (int)bi[q] < t)) ? 1u : 0u;
                            alike += ol == ml ? 1u : 0u;
                        }
                }
            }
            check = check || alike > 1;
            rk[e] = ((uint32_t)lo + less) << 16 | (uint32_t)t;
        }
    }
    };
    if (tied) rank_buckets(std::true_type{});      // uniform
    else rank_buckets(std::false_type{});
    check = __syncthreads_or(check && !full) != 0;
    // back in sample order, so that consecutive lanes store consecutive rows
#pragma unroll
    for (int e = 0; e < E; ++e)
        if (tid + kSortThreads * e < T) srank[rk[e] & 0xffffu] = (uint16_t)(rk[e] >> 16);
    __syncthreads();
    return check;
    };
    if (rank_samples(v, full, tied)) {             // uniform
        // the keys in the order of the ranks ascend where equal codes were equal values (the samples
        // are read again: held, they would cost the registers of every column)
        uint64_t* sorted = reinterpret_cast<uint64_t*>(body + ((size_t)T * 2 + 7) / 8 * 8);
        double y[E];
        int64_t n = N;
        forget(n);                                 // nor are the addresses held
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int t = tid + kSortThreads * e;
            y[e] = Xd[(int64_t)(t < T ? t : T - 1) * n];
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int t = tid + kSortThreads * e;
            if (t < T) sorted[srank[t]] = order_key(y[e]);
        }
        __syncthreads();
        bool wrong = false;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int t = tid + kSortThreads * e;
            if (t < T) {
                const int r = srank[t];
                wrong = wrong || (r > 0 && sorted[r - 1] > order_key(y[e]));
            }
        }
        if (__syncthreads_or(wrong)) {             // uniform
            base[tid] = 0;
            if (tid < 2) base[kSplit + tid] = 0;
            for (int i = tid; i < T / 64 + 2; i += kSortThreads) heads[i] = 0;
            __syncthreads();
            rank_samples(y, true, false);
        }
    }
    double z[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int t = tid + kSortThreads * e;
        z[e] = score[srank[t < T ? t : T - 1]];
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int t = tid + kSortThreads * e;
        if (t < T) store_z<ZT>(Z, (d * T + t) * N + c, z[e]);
    }
}

template <typename ZT, int E>
__global__ __launch_bounds__(kSortThreads) void k_copula_col(const double* __restrict__ X, int T, int64_t N,
                                                             void* __restrict__ Z, const double* __restrict__ score,
                                                             WsHeader* hdr)
{
    copula_col<ZT, E>(X, T, N, Z, score, hdr);
}
// Up to four samples per thread: 64 vector registers let two workgroups of 16 wavefronts share a
// CU, and the scalar ones have to let them too.
template <typename ZT, int E>
__global__ __launch_bounds__(kSortThreads) __attribute__((amdgpu_waves_per_eu(8), amdgpu_num_sgpr(80))) void
k_copula_col2(const double* __restrict__ X, int T, int64_t N, void* __restrict__ Z, const double* __restrict__ score,
              WsHeader* hdr)
{
    copula_col<ZT, E>(X, T, N, Z, score, hdr);
}

template <typename ZT>
void launch_col(const double* X, int64_t D, int64_t T, int64_t N, void* Z, const double* score, WsHeader* hdr,
                hipStream_t s)
{
    typedef void (*ColKernel)(const double*, int, int64_t, void*, const double*, WsHeader*);
    static const ColKernel kern[] = {k_copula_col2<ZT, 2>, k_copula_col2<ZT, 4>, k_copula_col<ZT, 6>,
                                     k_copula_col<ZT, 8>, k_copula_col<ZT, 10>, k_copula_col<ZT, 12>};
    const int e = (int)((T + kSortThreads - 1) / kSortThreads);
    hipLaunchKernelGGL(kern[(e + 1) / 2 - 1], dim3((unsigned)(N * D)), dim3(kSortThreads), col_lds_bytes(T), s, X, (int)T,
                       N, Z, score, hdr);
}

__global__ void k_zero_i32(int32_t* p, int64_t n)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

struct CopulaWs {
    size_t key_off, idx_off, nan_off, total;
};

CopulaWs copula_layout(int64_t D, int64_t T, int64_t N)
{
    CopulaWs w{};
    const int64_t nchunks = (T + kChunk - 1) / kChunk;
    size_t off = kWsHeader;
    if (nchunks > 1) {
        const size_t slots = (size_t)D * N * nchunks * kChunk;
        w.key_off = off; off = align_up(off + slots * 8, 256);
        w.idx_off = off; off = align_up(off + slots * 4, 256);
        w.nan_off = off; off = align_up(off + (size_t)D * N * nchunks * 4, 256);
    }
    w.total = off;
    return w;
}

}  // namespace

size_t copulize_ws_bytes(int64_t D, int64_t T, int64_t N) { return copula_layout(D, T, N).total; }

thoi_status launch_copulize(const double* X, int64_t D, int64_t T, int64_t N, int32_t z_dtype, void* Z, void* ws,
                            hipStream_t s)
{
    const CopulaWs w = copula_layout(D, T, N);
    char* base = static_cast<char*>(ws);
    WsHeader* hdr = reinterpret_cast<WsHeader*>(base);
    const int64_t nchunks = (T + kChunk - 1) / kChunk;
    uint64_t* wkey = nchunks > 1 ? reinterpret_cast<uint64_t*>(base + w.key_off) : nullptr;
    uint32_t* widx = nchunks > 1 ? reinterpret_cast<uint32_t*>(base + w.idx_off) : nullptr;
    int32_t* nanf = nchunks > 1 ? reinterpret_cast<int32_t*>(base + w.nan_off) : nullptr;

    if (nchunks > 1 && T <= kColMax && D * N >= (T <= 2 * kChunk ? kColMinShort : kColMin)) {
        // the score table takes the place of the sorted keys (12 bytes per slot of every column)
        double* score = reinterpret_cast<double*>(base + w.key_off);
        hipLaunchKernelGGL(k_copula_scores, dim3((unsigned)((T + 255) / 256)), dim3(256), 0, s, T, score, hdr);
        if (z_dtype == THOI_DTYPE_F64) launch_col<double>(X, D, T, N, Z, score, hdr, s);
        else launch_col<float>(X, D, T, N, Z, score, hdr, s);
        return hip_status(hipGetLastError());
    }

    // the header starts at zero: a fill kernel where the sort itself raises the status (one chunk),
    // else the sort clears it and the merge raises (no memset node, so the call can be captured)
    if (nchunks <= 1 || D * N == 0)
        hipLaunchKernelGGL(k_zero_i32, dim3(1), dim3(64), 0, s, reinterpret_cast<int32_t*>(hdr), (int64_t)(kWsHeader / 4));
    if (D * N == 0 || T == 0) return hip_status(hipGetLastError());

    dim3 g1((unsigned)nchunks, (unsigned)N, (unsigned)D);
    if (z_dtype == THOI_DTYPE_F64)
        hipLaunchKernelGGL(k_copula_sort<double>, g1, dim3(kSortThreads), 0, s, X, T, N, Z, wkey, widx, nanf, hdr);
    else
        hipLaunchKernelGGL(k_copula_sort<float>, g1, dim3(kSortThreads), 0, s, X, T, N, Z, wkey, widx, nanf, hdr);
    if (nchunks > 1) {
        dim3 g2((unsigned)nchunks, (unsigned)(N * D));
        if (z_dtype == THOI_DTYPE_F64)
            hipLaunchKernelGGL(k_copula_merge<double>, g2, dim3(kMergeThreads), 0, s, T, N, (int)nchunks, Z, wkey, widx,
                               nanf, hdr);
        else
            hipLaunchKernelGGL(k_copula_merge<float>, g2, dim3(kMergeThreads), 0, s, T, N, (int)nchunks, Z, wkey, widx,
                               nanf, hdr);
    }
    return hip_status(hipGetLastError());
}

}  // namespace thoi
