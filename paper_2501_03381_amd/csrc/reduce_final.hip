// Final merge of the streaming reduction, one workgroup of kFinThreads per (order, dataset, list):
// the accumulated list of earlier calls, every segment of this call and the FP64-refined values
// become the top-K (bottom-K) list.
//
// Latency-bound (a few hundred kept entries out of thousands of sorted segments), so the work is
// selection first: a threshold that at least K entries reach is taken from the segments' heads,
// only entries up to it are collected, and they are sorted once.  Merging the segments one after
// the other (two dependent global reads and two barriers each) took 285 us for the 236 segments
// of an objective over 60,458 n-plets with K = 100; the whole call of 64 datasets and that objective
// went from 482 to 215 us, the FP64 reduction of 25 variables from 4.70 to 4.31 ms.  The threshold is a
// (key, index) pair: by the key alone every entry of equal values was collected and sorted (a million
// equal values, K = 100: 8.66 ms, 0.39 so; distinct ones 0.27).
#include "radix_pick.hpp"
#include "reduce_common.hpp"

namespace thoi {
namespace {

constexpr int kFinThreads = 512;
constexpr int kFinWaves = kFinThreads / 64;
constexpr int kFinBuf = 2048;                    // collected entries sorted at a time
constexpr int kFinSegs = 2048;                   // segments considered at a time
static_assert(kFinBuf >= kFinWaves * kRedMaxK && kFinBuf >= kFinThreads, "one round of appends fits the buffer");

struct RedFinal {
    RedItem list[2][kRedMaxK];                   // the running list, double-buffered
    RedItem buf[kFinBuf];                        // collected entries
    uint64_t head[kFinSegs];                     // matching segments: the first key of each ...
    int64_t head_g[kFinSegs];                    // ... its index ...
    uint32_t seg[kFinSegs];                      // ... and the segment's slot
    uint32_t rh[256];                            // radix selection
    uint64_t thr;                                // entries behind (thr, thr_g) are not needed
    int64_t thr_g;
    uint32_t prefix;
    int cur, nbuf, nseg, rank;
};

// Whole workgroup: sort the collected entries, merge them into the running list (keeping K), empty
// the buffer and tighten the threshold.
__device__ __forceinline__ void red_final_flush(RedFinal& S, int K)
{
    __syncthreads();
    const int n = S.nbuf;
    const int c = S.cur;
    __syncthreads();                             // every thread has read them before the next append
    if (n == 0) return;                          // uniform
    int P = 1;
    while (P < n) P <<= 1;
    for (int i = n + (int)threadIdx.x; i < P; i += kFinThreads) S.buf[i] = RedItem{kKeyEmpty, kGEmpty};
    for (int size = 2; size <= P; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            __syncthreads();
            for (int i = threadIdx.x; i < (P >> 1); i += kFinThreads) {
                const int lo = 2 * i - (i & (stride - 1)), hi = lo + stride;
                const bool asc = (lo & size) == 0;
                const RedItem a = S.buf[lo], b = S.buf[hi];
                if (red_less(b, a) == asc) { S.buf[lo] = b; S.buf[hi] = a; }
            }
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < K; i += kFinThreads)
        S.list[c ^ 1][i] = red_merge_at(S.list[c], K, S.buf, n < K ? n : K, i);
    __syncthreads();
    if (threadIdx.x == 0) {
        const RedItem t = S.list[c ^ 1][K - 1];
        if (red_less(t.k, t.g, S.thr, S.thr_g)) { S.thr = t.k; S.thr_g = t.g; }
        S.cur = c ^ 1;
        S.nbuf = 0;
    }
    __syncthreads();
}

// Whole wavefront: append the entries of the lanes with `want` to the buffer (room is the caller's
// business).
__device__ __forceinline__ void red_final_append(RedFinal& S, bool want, uint64_t key, int64_t g)
{
    const uint64_t m = __ballot(want);
    if (m == 0) return;
    const int lane = (int)(threadIdx.x & 63);
    const int leader = __builtin_ctzll(m);
    int base = 0;
    if (lane == leader) base = atomicAdd(&S.nbuf, __popcll(m));
    base = __shfl(base, leader, 64);
    if (want) S.buf[base + __popcll(m & ((1ull << lane) - 1))] = RedItem{key, g};
}

// Whole workgroup: an upper bound of the K-th smallest of S.head[0..n) (n >= K >= 1) that at least
// K heads reach, exact in the upper 32 bits: four passes over 8 bits each.
__device__ __forceinline__ uint64_t red_final_select(RedFinal& S, int n, int K)
{
    if (threadIdx.x == 0) { S.prefix = 0; S.rank = K; }
    for (int pass = 3; pass >= 0; --pass) {
        for (int i = threadIdx.x; i < 256; i += kFinThreads) S.rh[i] = 0;
        __syncthreads();
        const uint32_t pre = S.prefix;
        for (int i = threadIdx.x; i < n; i += kFinThreads) {
            const uint32_t h = (uint32_t)(S.head[i] >> 32);
            if (radix_match(h, pre, pass)) atomicAdd(&S.rh[(h >> (8 * pass)) & 255u], 1u);
        }
        __syncthreads();
        if (threadIdx.x < 64) radix_pick(S.rh, (int)threadIdx.x, pass, S.prefix, S.rank);
        __syncthreads();
    }
    return ((uint64_t)S.prefix << 32) | 0xffffffffull;
}

// Whole workgroup: the segments [r, n) whose head can still enter, moved to the front; their number.
__device__ __forceinline__ int red_final_repack(RedFinal& S, int r, int n)
{
    constexpr int kU = kFinSegs / kFinThreads;
    uint64_t h[kU];
    int64_t g[kU];
    uint32_t s[kU];
    bool on[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
        const int j = r + (int)threadIdx.x + u * kFinThreads;
        on[u] = j < n;
        h[u] = on[u] ? S.head[j] : 0;
        g[u] = on[u] ? S.head_g[j] : 0;
        s[u] = on[u] ? S.seg[j] : 0;
        on[u] = on[u] && !red_less(S.thr, S.thr_g, h[u], g[u]);
    }
    if (threadIdx.x == 0) S.nseg = 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kU; ++u)
        if (on[u]) {
            const int j = atomicAdd(&S.nseg, 1);
            S.head[j] = h[u];
            S.head_g[j] = g[u];
            S.seg[j] = s[u];
        }
    __syncthreads();
    return S.nseg;
}

__global__ __launch_bounds__(kFinThreads) void k_red_final(RedArgs red, WsHeader* hdr)
{
    __shared__ RedFinal S;
    const int k = blockIdx.x, d = blockIdx.y, l = blockIdx.z;
    const int K = red.topk;
    if (K <= 0) return;
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    double* tv = red.top_val + (((int64_t)d * (red.kmax + 1) + k) * 2 + l) * K;
    int64_t* tg = red.top_g + (((int64_t)d * (red.kmax + 1) + k) * 2 + l) * K;
    for (int i = tid; i < K; i += kFinThreads) {
        const bool has = tg[i] >= 0;
        S.list[0][i] = has ? RedItem{red_list_key(l, tv[i]), tg[i]} : RedItem{kKeyEmpty, kGEmpty};
    }
    if (tid == 0) { S.cur = 0; S.nbuf = 0; S.nseg = 0; }
    __syncthreads();
    if (tid == 0) {
        S.thr = S.list[0][K - 1].k;
        S.thr_g = S.list[0][K - 1].g;
        if (red.bound) {
            // the tightest K-th key that a segment of this (d, k) has published
            const uint64_t b = ~(uint64_t)red.bound[((int64_t)d * (red.kmax + 1) + k) * 2 + l];
            if (b < S.thr) { S.thr = b; S.thr_g = kGEmpty; }
        }
    }
    __syncthreads();
    const uint32_t nseg = min(hdr->seg_next, red.seg_cap);
    for (uint32_t s0 = 0; s0 < nseg;) {
        // the next segments of this (d, k) whose head can still enter, up to kFinSegs of them
        const uint64_t thr = S.thr;
        const int64_t thr_g = S.thr_g;
        constexpr int kU = kFinSegs / kFinThreads;
        SegHdr h[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const uint32_t s = s0 + tid + u * kFinThreads;
            h[u] = s < nseg ? red.seg_hdr[s] : SegHdr{-1, -1};
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const uint32_t s = s0 + tid + u * kFinThreads;
            if (h[u].d == d && h[u].k == k) {
                const uint64_t key = red.seg_key[((int64_t)s * 2 + l) * K];
                const int64_t g = red.seg_g[((int64_t)s * 2 + l) * K];
                if (key != kKeyEmpty && !red_less(thr, thr_g, key, g)) {
                    const int j = atomicAdd(&S.nseg, 1);
                    S.head[j] = key;
                    S.head_g[j] = g;
                    S.seg[j] = s;
                }
            }
        }
        s0 += kFinSegs;
        __syncthreads();
        int n = S.nseg;
        if (n >= K && n > kFinWaves) {
            // K heads reach this key, so K entries do: a larger one is not needed, nor is a segment
            // with a larger head
            const uint64_t t = red_final_select(S, n, K);
            if (tid == 0 && t < S.thr) { S.thr = t; S.thr_g = kGEmpty; }
        } else if (n > kFinWaves) {
            // fewer segments than K: the j-th entries of all of them with n * j >= K
            const int j = (K + n - 1) / n;
            uint64_t worst = 0;
            for (int i = tid; i < n; i += kFinThreads) {
                const uint64_t e = red.seg_key[((int64_t)S.seg[i] * 2 + l) * K + j - 1];
                worst = e > worst ? e : worst;
            }
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) { const uint64_t y = __shfl_xor(worst, o, 64); worst = y > worst ? y : worst; }
            if (tid == 0) S.head[0] = 0;         // the heads are not used on this path
            __syncthreads();
            if (lane == 0) atomicMax(reinterpret_cast<unsigned long long*>(&S.head[0]), (unsigned long long)worst);
            __syncthreads();
            if (tid == 0 && S.head[0] < S.thr) { S.thr = S.head[0]; S.thr_g = kGEmpty; }
        }
        __syncthreads();
        const bool sel = n >= K && n > kFinWaves;
        // one segment per wavefront and round; a flush when the next round may not fit
        for (int r = 0; r < n; r += kFinWaves) {
            const int nb = S.nbuf;
            __syncthreads();                     // every thread has read nbuf before the next append
            if (nb + kFinWaves * K > kFinBuf) {
                red_final_flush(S, K);
                if (sel) {
                    n = red_final_repack(S, r, n);
                    r = 0;
                    if (n == 0) break;           // uniform
                }
            }
            const uint64_t t = S.thr;
            const int j = r + wave;
            if (j < n && !(sel && S.head[j] > t)) {
                const int64_t e0 = ((int64_t)S.seg[j] * 2 + l) * K;
                for (int i0 = 0; i0 < K; i0 += 64) {
                    const int i = i0 + lane;
                    const uint64_t key = i < K ? red.seg_key[e0 + i] : kKeyEmpty;
                    bool want = key != kKeyEmpty && key <= t;
                    const bool all = __ballot(want) == ~0ull;
                    const int64_t g = want ? red.seg_g[e0 + i] : 0;
                    // (no wait for the index where no key ties with the threshold's)
                    if (__ballot(want && key == t)) want = want && (key < t || g <= S.thr_g);
                    red_final_append(S, want, key, g);
                    if (!all) break;                         // sorted: nothing further on is smaller
                }
            }
            __syncthreads();
        }
        red_final_flush(S, K);
        if (tid == 0) S.nseg = 0;
        __syncthreads();
    }
    // the FP64-refined values, kU per thread and round with their loads in flight together
    constexpr int kU = kFinBuf / kFinThreads;
    const uint32_t nlate = min(hdr->late_next, red.late_cap);
    for (uint32_t b0 = 0; b0 < nlate; b0 += kFinBuf) {
        red_final_flush(S, K);
        const uint64_t t = S.thr;
        const int64_t thr_g = S.thr_g;
        LateEntry e[kU];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const uint32_t i = b0 + tid + u * kFinThreads;
            e[u] = i < nlate ? red.late[i] : LateEntry{-1, -1, 0, 0.0};
        }
#pragma unroll
        for (int u = 0; u < kU; ++u) {
            const uint64_t key = red_list_key(l, e[u].v);
            red_final_append(S, e[u].d == d && e[u].k == k && !red_less(t, thr_g, key, e[u].g), key, e[u].g);
        }
    }
    red_final_flush(S, K);
    __syncthreads();
    for (int i = tid; i < K; i += kFinThreads) {
        const RedItem e = S.list[S.cur][i];
        const bool has = e.k != kKeyEmpty;
        tv[i] = has ? red_list_val(l, e.k) : __builtin_nan("");
        tg[i] = has ? e.g : -1;
    }
}

}  // namespace

void red_final_launch(const RedArgs& red, WsHeader* hdr, int kmax, int64_t D, hipStream_t s)
{
    hipLaunchKernelGGL(k_red_final, dim3((unsigned)(kmax + 1), (unsigned)D, 2), dim3(kFinThreads), 0, s, red, hdr);
}

}  // namespace thoi
