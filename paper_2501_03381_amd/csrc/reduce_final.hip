// Final merge of the streaming reduction, one workgroup of kFinThreads per (order, dataset, list) (where there
// are many lists of few segments: k_red_final_many):
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
    uint64_t head[kFinSegs];                     // matching segments: one key of each ...
    uint32_t seg[kFinSegs];                      // ... and its slot
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

// Whether a segment of this head may hold an entry that is needed; the index is read where the keys tie.
__device__ __forceinline__ bool red_final_enters(uint64_t thr, int64_t thr_g, uint64_t head, const int64_t* __restrict__ g)
{
    return head < thr || (head == thr && (thr_g == kGEmpty || *g <= thr_g));
}

// Whole workgroup: the segments [r, n) whose head can still enter, moved to the front; their number.
__device__ __forceinline__ int red_final_repack(RedFinal& S, const RedArgs& red, int l, int K, int r, int n)
{
    constexpr int kU = kFinSegs / kFinThreads;
    uint64_t h[kU];
    uint32_t s[kU];
    bool on[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) {
        const int j = r + (int)threadIdx.x + u * kFinThreads;
        on[u] = j < n;
        h[u] = on[u] ? S.head[j] : 0;
        s[u] = on[u] ? S.seg[j] : 0;
        on[u] = on[u] && red_final_enters(S.thr, S.thr_g, h[u], red.seg_g + ((int64_t)s[u] * 2 + l) * K);
    }
    if (threadIdx.x == 0) S.nseg = 0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kU; ++u)
        if (on[u]) {
            const int j = atomicAdd(&S.nseg, 1);
            S.head[j] = h[u];
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
                if (key != kKeyEmpty && red_final_enters(thr, thr_g, key, red.seg_g + ((int64_t)s * 2 + l) * K)) {
                    const int j = atomicAdd(&S.nseg, 1);
                    S.head[j] = key;
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
                    n = red_final_repack(S, red, l, K, r, n);
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

// ------------------------------------------------------------------------------------------------
// The same where there are many lists of few segments each: one workgroup of 256 threads and 21 KB of LDS per
// (order, dataset) for both lists, so seven share a CU and the headers are read once for both; the
// segments that still beat the running lists are merged one after the other.
// ------------------------------------------------------------------------------------------------
struct RedMany {
    uint64_t key[2][2][kRedMaxK];
    int64_t g[2][2][kRedMaxK];
    uint64_t ck[256];
    int64_t cg[256];
    int cur[2];
    int nc;
};

// Whole workgroup: merge the sorted run (bk, bg)[0..nb) into list `l`, keeping K.
__device__ __forceinline__ void red_many_merge(RedMany& S, int l, int K, const uint64_t* bk, const int64_t* bg, int nb)
{
    const int c = S.cur[l];
    const uint64_t* ak = S.key[l][c];
    const int64_t* ag = S.g[l][c];
    uint64_t* ok = S.key[l][c ^ 1];
    int64_t* og = S.g[l][c ^ 1];
    const int na = K;
    for (int i = threadIdx.x; i < K; i += blockDim.x) {
        int lo = i - nb > 0 ? i - nb : 0, hi = i < na ? i : na;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (red_less(ak[mid], ag[mid], bk[i - 1 - mid], bg[i - 1 - mid])) lo = mid + 1; else hi = mid;
        }
        const int a = lo, b = i - a;
        const bool takeA = (b >= nb) || (a < na && red_less(ak[a], ag[a], bk[b], bg[b]));
        ok[i] = takeA ? ak[a] : bk[b];
        og[i] = takeA ? ag[a] : bg[b];
    }
    __syncthreads();
    if (threadIdx.x == 0) S.cur[l] = c ^ 1;
    __syncthreads();
}

// Whole workgroup (blockDim <= 256): offer one (key, g) per thread (valid == false: nothing) to
// list l; the candidates are compacted, sorted (bitonic) and merged.
__device__ __forceinline__ void red_many_offer(RedMany& S, int l, int K, bool valid, uint64_t key, int64_t g)
{
    const int c = S.cur[l];
    const bool cand = valid && red_less(key, g, S.key[l][c][K - 1], S.g[l][c][K - 1]);
    if (!__syncthreads_or(cand)) return;
    if (threadIdx.x == 0) S.nc = 0;
    __syncthreads();
    if (cand) {
        const int slot = atomicAdd(&S.nc, 1);
        S.ck[slot] = key;
        S.cg[slot] = g;
    }
    __syncthreads();
    const int nc = S.nc;
    int P = 1;
    while (P < nc) P <<= 1;
    for (int i = nc + threadIdx.x; i < P; i += blockDim.x) { S.ck[i] = kKeyEmpty; S.cg[i] = kGEmpty; }
    for (int size = 2; size <= P; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            __syncthreads();
            for (int i = threadIdx.x; i < (P >> 1); i += blockDim.x) {
                const int lo = 2 * i - (i & (stride - 1)), hi = lo + stride;
                const bool asc = (lo & size) == 0;
                const uint64_t ka = S.ck[lo], kb = S.ck[hi];
                const int64_t ga = S.cg[lo], gb = S.cg[hi];
                if (red_less(kb, gb, ka, ga) == asc) { S.ck[lo] = kb; S.ck[hi] = ka; S.cg[lo] = gb; S.cg[hi] = ga; }
            }
        }
    }
    __syncthreads();
    red_many_merge(S, l, K, S.ck, S.cg, nc < K ? nc : K);
}

__global__ __launch_bounds__(256) void k_red_final_many(RedArgs red, WsHeader* hdr)
{
    __shared__ RedMany S;
    const int k = blockIdx.x, d = blockIdx.y;
    const int K = red.topk;
    if (K <= 0) return;
    double* tv = red.top_val + ((int64_t)d * (red.kmax + 1) + k) * 2 * K;
    int64_t* tg = red.top_g + ((int64_t)d * (red.kmax + 1) + k) * 2 * K;
    for (int i = threadIdx.x; i < 2 * K; i += blockDim.x) {
        const int l = i / K, j = i % K;
        const bool has = tg[i] >= 0;
        S.key[l][0][j] = has ? red_list_key(l, tv[i]) : kKeyEmpty;
        S.g[l][0][j] = has ? tg[i] : kGEmpty;
    }
    if (threadIdx.x == 0) { S.cur[0] = S.cur[1] = 0; }
    __syncthreads();
    // Segments in batches of one per thread: each thread tests its segment's two list heads
    // against the current K-th entries, the candidates are compacted, and only those are merged
    // (tested again against the threshold as it tightens).  After the first batches almost no
    // segment beats the running lists, so a batch costs one round of parallel loads.
    __shared__ uint32_t cand[2][256];
    __shared__ int ncand[2];
    const uint32_t nseg = min(hdr->seg_next, red.seg_cap);
    for (uint32_t s0 = 0; s0 < nseg; s0 += blockDim.x) {
        if (threadIdx.x < 2) ncand[threadIdx.x] = 0;
        __syncthreads();
        const uint32_t s = s0 + threadIdx.x;
        if (s < nseg) {
            const SegHdr h = red.seg_hdr[s];
            if (h.d == d && h.k == k) {
                for (int l = 0; l < 2; ++l) {
                    const int64_t e = ((int64_t)s * 2 + l) * K;
                    const int c = S.cur[l];
                    if (red_less(red.seg_key[e], red.seg_g[e], S.key[l][c][K - 1], S.g[l][c][K - 1]))
                        cand[l][atomicAdd(&ncand[l], 1)] = s;
                }
            }
        }
        __syncthreads();
        for (int l = 0; l < 2; ++l) {
            const int nc = ncand[l];
            for (int j = 0; j < nc; ++j) {
                const int64_t e = ((int64_t)cand[l][j] * 2 + l) * K;
                const uint64_t* bk = red.seg_key + e;
                const int64_t* bg = red.seg_g + e;
                const int c = S.cur[l];
                if (!red_less(bk[0], bg[0], S.key[l][c][K - 1], S.g[l][c][K - 1])) continue;   // uniform
                red_many_merge(S, l, K, bk, bg, K);
            }
        }
        __syncthreads();                         // every thread has read ncand before the reset
    }
    const uint32_t nlate = min(hdr->late_next, red.late_cap);
    for (uint32_t b0 = 0; b0 < nlate; b0 += blockDim.x) {
        const uint32_t i = b0 + threadIdx.x;
        bool mine = false;
        double v = 0.0;
        int64_t g = 0;
        if (i < nlate) {
            const LateEntry e = red.late[i];
            mine = e.d == d && e.k == k;
            v = e.v;
            g = e.g;
        }
        red_many_offer(S, 0, K, mine, red_list_key(0, v), g);
        red_many_offer(S, 1, K, mine, red_list_key(1, v), g);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 2 * K; i += blockDim.x) {
        const int l = i / K, j = i % K;
        const uint64_t key = S.key[l][S.cur[l]][j];
        const bool has = key != kKeyEmpty;
        tv[i] = has ? red_list_val(l, key) : __builtin_nan("");
        tg[i] = has ? S.g[l][S.cur[l]][j] : -1;
    }
}

// The second form where a list has a few segments on average, or there are more lists than the first form's
// workgroups (two per CU) get through in about four rounds.  Whole calls, FP64, K = 100, second / first form, ms:
//   orders 3..12 of 12 variables (1.4 segments per list): 1 dataset 0.098 / 0.105, 128 0.164 / 0.212, 2000 3.40 / 5.30
//   orders 3..16 of 16 (15): 1 dataset 0.176 / 0.131, 32 0.465 / 0.442, 128 2.45 / 2.38, 512 9.40 / 10.2
//   orders 3..6 of 18 (14): 1 dataset 0.156 / 0.096, 128 0.529 / 0.500, 256 0.914 / 0.940
constexpr int64_t kFewSegments = 4, kManyLists = 1500;

}  // namespace

void red_final_launch(const RedArgs& red, WsHeader* hdr, int kmax, int64_t D, hipStream_t s)
{
    const int64_t lists = (int64_t)(kmax + 1) * D;
    if (lists > kManyLists || (int64_t)red.seg_cap <= kFewSegments * lists)
        hipLaunchKernelGGL(k_red_final_many, dim3((unsigned)(kmax + 1), (unsigned)D), dim3(256), 0, s, red, hdr);
    else
        hipLaunchKernelGGL(k_red_final, dim3((unsigned)(kmax + 1), (unsigned)D, 2), dim3(kFinThreads), 0, s, red, hdr);
}

}  // namespace thoi
