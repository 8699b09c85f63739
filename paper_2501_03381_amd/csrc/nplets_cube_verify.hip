// The n-plets that the cube engine's filter leaves open (nplets_cube.hip): the lane engine's
// factorisation, or the pair engine's above its orders (the same operations), result handling and reducer,
// on lists of n-plets by order, so that a filtered reduction is theirs bit for bit.
#include "nplets_cube.hpp"
#include "pair_factor.hpp"

namespace thoi {
namespace {

// Factor the n-plet of row P and suffix subset B; term: C(N, k) - 1 - its lexicographic rank.
template <typename F, int K, int KHI>
__device__ __forceinline__ FactorOut<F> verify_factor(int k, uint32_t P, uint32_t B, int N, const F* sR,
                                                      const uint32_t* sbin, uint32_t& term)
{
    if (k == K) {
        const int h = N - kCubeSuffix;
        int c[K];
        term = 0;
#pragma unroll
        for (int i = 0; i < K; ++i) {
            if (P) {
                const int lz = __builtin_clz(P);
                c[i] = h - 1 - (31 - lz);
                P &= ~(0x80000000u >> lz);
            } else {
                c[i] = h + __builtin_ctz(B);
                B &= B - 1;
            }
            term += sbin[(N - 1 - c[i]) * (K + 1) + K - i];
        }
        return lane_factor<F, K>(c, sR, N);
    }
    if constexpr (K < KHI) return verify_factor<F, K + 1, KHI>(k, P, B, N, sR, sbin, term);
    return FactorOut<F>{};
}

// grid (kVerifyBlocks, orders of the class), block kTile.
template <typename F, int KLO, int KHI>
__global__ __launch_bounds__(kTile) void k_cube_verify(EvalArgs a, CubeTable tab, CubeOpen open, RedArgs red, int64_t d,
                                                       int first)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double sbias[3];
    const CubePiece pc = tab.p[first + (int)blockIdx.y];
    const int k = pc.k, N = a.N;
    const int64_t n = open.cnt[k];
    if ((int64_t)blockIdx.x * kTile >= n) return;                      // uniform
    F* sR = reinterpret_cast<F*>(smem);
    const size_t off = ((size_t)N * N * sizeof(F) + 15) / 16 * 16;
    double* sIsd = reinterpret_cast<double*>(smem + off);
    double* sLogd = sIsd + N;
    uint32_t* sbin = reinterpret_cast<uint32_t*>(sLogd + N);           // C(n, m), n < N, m <= k
    const size_t roff = (off + 16 * (size_t)N + (size_t)N * (KHI + 1) * 4 + 15) / 16 * 16;
    RedLds S = red_view(smem + roff, red.topk, red.bins);
    for (int i = threadIdx.x; i < N * (k + 1); i += kTile) sbin[i] = (uint32_t)kPascal.v[i / (k + 1)][i % (k + 1)];
    if (threadIdx.x == 0) bias_for(a.bias, k, sbias[0], sbias[1], sbias[2]);
    stage_corr<F>(a.Sigma + d * N * N, N, sR, sIsd, sLogd);
    red_begin(S, red, (int)d, k);
    const uint32_t* list = open.list + open.off[k];
    const uint32_t last = (uint32_t)kPascal.v[N][k] - 1u;
    for (int64_t t = (int64_t)blockIdx.x * kTile; t < n; t += (int64_t)kVerifyBlocks * kTile) {
        const int64_t i = t + threadIdx.x;
        double omega = 0.0;
        int64_t pos = 0;
        bool valid = false;
        if (i < n) {
            const uint32_t m = list[i];
            uint32_t term = 0;
            const FactorOut<F> f =
                verify_factor<F, KLO, KHI>(k, m >> kCubeSuffix, m & (kCubeRow - 1), N, sR, sbin, term);
            pos = pc.pos0 + (int64_t)(last - term);
            valid = store_result<F>(a, true, (int)d, pos, k, f, 0.0, sbias[0], sbias[1], sbias[2], sizeof(F) == 8, omega);
        }
        red_push(S, red, k, valid, omega, a.g_begin + pos);
    }
    red_end(S, red, a.hdr, (int)d, k);
}

// The same for orders above the lane engine's, two n-plets per wavefront (FP64).
__global__ __launch_bounds__(kTile) void k_cube_verify_pair(EvalArgs a, CubeTable tab, CubeOpen open, RedArgs red, int64_t d,
                                                            int first)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double scol[kTile / 32 * 2 * kW2Max], swrow[kTile / 32 * 2 * kW2Max];
    __shared__ int scidx[kTile / 32 * kW2Max];
    __shared__ double sbias[3];
    const CubePiece pc = tab.p[first + (int)blockIdx.y];
    const int k = pc.k, N = a.N, h = N - kCubeSuffix;
    const int64_t n = open.cnt[k];
    constexpr int kPer = kTile / 32;                                   // n-plets per round
    if ((int64_t)blockIdx.x * kPer >= n) return;                       // uniform
    double* sR = reinterpret_cast<double*>(smem);
    double* sIsd = sR + N * N;
    double* sLogd = sIsd + N;
    uint32_t* sbin = reinterpret_cast<uint32_t*>(sLogd + N);           // C(n, m), n < N, m <= k
    const size_t roff = ((size_t)N * N * 8 + 16 * (size_t)N + (size_t)N * (kCubeMaxN + 1) * 4 + 15) / 16 * 16;
    RedLds S = red_view(smem + roff, red.topk, red.bins);
    for (int i = threadIdx.x; i < N * (k + 1); i += kTile) sbin[i] = (uint32_t)kPascal.v[i / (k + 1)][i % (k + 1)];
    if (threadIdx.x == 0) bias_for(a.bias, k, sbias[0], sbias[1], sbias[2]);
    stage_corr<double>(a.Sigma + d * N * N, N, sR, sIsd, sLogd);
    red_begin(S, red, (int)d, k);
    const int half = threadIdx.x >> 5, i = threadIdx.x & 31;
    int* ch = scidx + half * kW2Max;
    double* col = scol + half * 2 * kW2Max;
    double* wrow = swrow + half * 2 * kW2Max;
    const uint32_t* list = open.list + open.off[k];
    const uint32_t last = (uint32_t)kPascal.v[N][k] - 1u;
    for (int64_t t = (int64_t)blockIdx.x * kPer; t < n; t += (int64_t)kVerifyBlocks * kPer) {
        const bool on = t + half < n;
        const uint32_t m = list[on ? t + half : n - 1];                // a half without an entry repeats the last
        const uint32_t P = m >> kCubeSuffix, B = m & (kCubeRow - 1);
        const int p = __popc(P);
        // lane v: variable v when it is a member, at its place among the members
        uint32_t term = 0;
        const bool in = i < h ? ((P >> (h - 1 - i)) & 1u) != 0 : (i < N && ((B >> (i - h)) & 1u) != 0);
        if (in) {
            const int q = i < h ? (int)__popc(P >> (h - i)) : p + (int)__popc(B & ((1u << (i - h)) - 1u));
            ch[q] = i;
            term = sbin[(N - 1 - i) * (k + 1) + k - q];
        }
#pragma unroll
        for (int o = 16; o > 0; o >>= 1) term += __shfl_xor(term, o, 32);
        wave_sync();
        const FactorOut<double> f = pair_factor<false>(sR, N, ch, k, k, col, wrow);
        double omega = 0.0;
        const int64_t pos = pc.pos0 + (int64_t)(last - term);
        bool valid = false;
        if (on && i == 0)
            valid = store_result<double>(a, true, (int)d, pos, k, f, 0.0, sbias[0], sbias[1], sbias[2], true, omega);
        red_push(S, red, k, valid, omega, a.g_begin + pos);
    }
    red_end(S, red, a.hdr, (int)d, k);
}

// Pieces of orders KLO..KHI: the first and how many.
int pieces(const CubeTable& tab, int klo, int khi, int& first)
{
    int n = 0;
    first = -1;
    for (int i = 0; i < tab.n; ++i)
        if (tab.p[i].k >= klo && tab.p[i].k <= khi) {
            if (first < 0) first = i;
            ++n;
        }
    return n;
}

template <typename F, int KLO, int KHI>
void launch_class(const EvalArgs& a, const CubeTable& tab, const CubeOpen& open, const RedArgs& red, int64_t d,
                  hipStream_t s)
{
    int first = 0;
    const int n = pieces(tab, KLO, KHI, first);
    if (n == 0) return;
    const size_t off = ((size_t)a.N * a.N * sizeof(F) + 15) / 16 * 16;
    const size_t lds = (off + 16 * (size_t)a.N + (size_t)a.N * (KHI + 1) * 4 + 15) / 16 * 16 + red_lds_bytes(red.topk, red.bins);
    hipLaunchKernelGGL((k_cube_verify<F, KLO, KHI>), dim3(kVerifyBlocks, (unsigned)n), dim3(kTile), lds, s, a, tab, open, red,
                       d, first);
}

}  // namespace

void cube_verify_launch(const EvalArgs& a, const CubeTable& tab, const CubeOpen& open, const RedArgs& red, int64_t d,
                        bool f32, const FanScope& fan, int from)
{
    // short lists: each class is bound by the latency of its longest lane, so they run side by side
    if (f32) {
        launch_class<float, 17, 20>(a, tab, open, red, d, fan.stream(from));
        launch_class<float, 21, 24>(a, tab, open, red, d, fan.stream(from + 1));
        launch_class<float, 13, 16>(a, tab, open, red, d, fan.stream(from + 2));
        launch_class<float, 9, 12>(a, tab, open, red, d, fan.stream(from + 3));
        launch_class<float, 3, 8>(a, tab, open, red, d, fan.stream(from + 4));
        return;
    }
    launch_class<double, 15, 18>(a, tab, open, red, d, fan.stream(from));
    launch_class<double, 11, 14>(a, tab, open, red, d, fan.stream(from + 1));
    launch_class<double, 7, 10>(a, tab, open, red, d, fan.stream(from + 2));
    launch_class<double, 3, 6>(a, tab, open, red, d, fan.stream(from + 3));
    int first = 0;
    const int n = pieces(tab, kF64LaneMax + 1, kCubeMaxN, first);
    if (n > 0) {
        const size_t lds = ((size_t)a.N * a.N * 8 + 16 * (size_t)a.N + (size_t)a.N * (kCubeMaxN + 1) * 4 + 15) / 16 * 16 +
                           red_lds_bytes(red.topk, red.bins);
        hipLaunchKernelGGL(k_cube_verify_pair, dim3(kVerifyBlocks, (unsigned)n), dim3(kTile), lds, fan.stream(from + 4), a, tab, open,
                           red, d, first);
    }
}

}  // namespace thoi
