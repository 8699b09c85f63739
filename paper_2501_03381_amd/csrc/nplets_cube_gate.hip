// Whether the subset table pays for a dataset (nplets_cube.hip), decided before it is built.
//
// The filter leaves an n-plet open when its margin, which grows with the sum of its VIFs, reaches a bin edge or
// the lists, and an open n-plet costs a factorisation beside its table reads.  How many are open depends on
// the data and the bins: N = 28, FP32 + refinement, 256 bins over each order's range, AR(1) covariances of
// 0.9 / 0.97 / 0.99 took 7.9 / 9.7 / 17.1 ms with the table and 14.5 by a factorisation per n-plet, with 4096
// bins 23.7 / 25.7 / 25.9.  So a few n-plets of every order are factored in FP64 first, and the datasets
// whose estimate says so go to the factorisation engines whole: 7.9 / 9.8 / 14.7 and 14.7 / 14.8 / 14.8 ms.  FP64 has
// no such choice: its margin is too small to matter, and 25 us are a tenth of its smallest calls.
//
// Latency-bound: one workgroup per (order, dataset), one n-plet per half-wave, one round, with the
// factorisation that is arranged for latency (25 to 29 us for all orders).  The last workgroup of a
// dataset to report decides.
#include "nplets_cube.hpp"
#include "nplets_cube_margin.hpp"
#include "pair_factor_lat.hpp"

namespace thoi {
namespace {

constexpr int kGateThreads = 512;
constexpr int kGateSamples = kGateThreads / 32;

struct GateRow {
    double piv, aj;          // of the lane's row: its pivot and a_j
};
// Rows of the half-wave's n-plet cidx[0..k-1] (32 entries; those beyond the order are cleared), k <= KM.
template <int KM>
__device__ __attribute__((noinline)) GateRow gate_factor(GlobalDouble Sig, int N, LdsInt cidx, int k_in, LdsDouble col,
                                                         LdsDouble wrow)
{
    const int k = __builtin_amdgcn_readfirstlane(k_in);
    const int i = threadIdx.x & 31;
    if (i >= k) cidx[i] = 0;
    wave_sync();
    const int ci = cidx[i];
    const double si = inv_sd(Sig[(int64_t)ci * N + ci]);
    wrow[i] = si;
    wave_sync();
    double r[kW2Max];
    pair_gather_lat<PairSource::Global, KM, 4>(r, Sig, N, cidx, k, k, i, ci, si, wrow);
    wave_sync();                                          // wrow is reused below
    GateRow g{1.0, 0.0};
    pair_pivots_lat<KM>(r, k, k, i, col, wrow, g.piv, g.aj);
    wave_sync();
    return g;
}

// grid (orders, D), block kGateThreads.
__global__ __launch_bounds__(kGateThreads) void k_cube_gate(EvalArgs a, CubeTable tab, RedArgs red, CubeGate gate, CubeCost cost)
{
    __shared__ double scol[kGateSamples * 2 * kW2Max], swrow[kGateSamples * 2 * kW2Max];
    __shared__ int scidx[kGateSamples * kW2Max];
    __shared__ uint32_t sbin[kCubeMaxN * (kCubeMaxN + 1)];
    __shared__ double sv[kGateSamples], smu[kGateSamples], sbias[3];
    __shared__ float sp[kGateSamples];
    __shared__ int sin_[kGateSamples];
    const int N = a.N, h = N - kCubeSuffix;
    const int k = tab.p[blockIdx.x].k;
    const int64_t d = blockIdx.y;
    const int tid = threadIdx.x, half = tid >> 5, i = tid & 31;
    for (int e = tid; e < N * (k + 1); e += kGateThreads) sbin[e] = (uint32_t)kPascal.v[e / (k + 1)][e % (k + 1)];
    if (tid == 0) bias_for(a.bias, k, sbias[0], sbias[1], sbias[2]);
    __syncthreads();
    // evenly spaced ranks, unranked by every lane of the half-wave
    int* ch = scidx + half * kW2Max;
    {
        uint32_t r = (uint32_t)((2 * half + 1) * kPascal.v[N][k] / (2 * kGateSamples));
        int m = k - 1;
        for (int x = 0; x < N && m >= 0; ++x) {
            const uint32_t c = sbin[(N - 1 - x) * (k + 1) + m];
            if (r < c) {
                if (i == 0) ch[k - 1 - m] = x;
                --m;
            } else {
                r -= c;
            }
        }
    }
    wave_sync();
    const GlobalDouble Sig = (GlobalDouble)(a.Sigma + d * N * N);
    const LdsInt lx = (LdsInt)ch;
    const LdsDouble lc = (LdsDouble)(scol + half * 2 * kW2Max), lw = (LdsDouble)(swrow + half * 2 * kW2Max);
    GateRow g;
    if (k <= 8) g = gate_factor<8>(Sig, N, lx, k, lc, lw);             // uniform
    else if (k <= 16) g = gate_factor<16>(Sig, N, lx, k, lc, lw);
    else if (k <= 24) g = gate_factor<24>(Sig, N, lx, k, lc, lw);
    else g = gate_factor<kW2Max>(Sig, N, lx, k, lc, lw);
    const bool mine = i < k;
    const bool ok = half_sum(mine && !(g.piv > 0.0) ? 1.0 : 0.0) == 0.0;
    const double ld = half_sum(mine ? log(g.piv) : 0.0), sa = half_sum(mine ? log(g.aj) : 0.0);
    const double vmax = half_max(mine ? g.aj : 0.0);
    // the filter's bound of the sum of VIFs: the largest of each eight members of the prefix and of each
    // five of the last ten variables, as often as there are members
    const int p = __popc((uint32_t)(__ballot(mine && ch[i] < h) >> (tid & 32)));
    double* w = swrow + half * 2 * kW2Max;
    w[i] = mine ? g.aj : 0.0;
    wave_sync();
    const int g0 = i < p ? i / 8 * 8 : p + (i - p) / 5 * 5;
    const int g1 = i < p ? (g0 + 8 < p ? g0 + 8 : p) : (g0 + 5 < k ? g0 + 5 : k);
    double most = 0.0;
    if (mine)
        for (int j = g0; j < g1; ++j) most = w[j] > most ? w[j] : most;
    const double ex = half_sum(most);
    const double TC = -0.5 * ld + sbias[0], DTC = 0.5 * (ld + sa) + sbias[1], v = TC - DTC;
    const Margin mg = margin_of<true>(k, ld, (float)log(vmax), (float)ex, a.vif_tau);
    const double mu = mg.value(TC, DTC);
    const bool bad = !ok || !isfinite(ld) || !isfinite(sa) || !isfinite(mu) || !(fabs(ld) < kFixMax);
    const bool in = !bad && mg.vif == 0;                               // may enter lists and bins as FP32 has it
    float open = bad || mg.vif == 1 ? 1.0f : 0.0f;
    if (in && red.bins > 0) {
        // the chance that a bin edge is within the margin
        const double scale = (double)red.bins / (red.hi[k] - red.lo[k]), x = (v - red.lo[k]) * scale, ms = mu * scale;
        if (!(x < -ms || x > (double)red.bins + ms)) open = ms < 0.5 ? (float)(2.0 * ms) : 1.0f;
    }
    if (i == 0) {
        sv[half] = v;
        smu[half] = mu;
        sp[half] = open;
        sin_[half] = in ? 1 : 0;
    }
    __syncthreads();
    if (tid >= 64) return;                                             // the first wavefront, one lane per sample
    const bool on = tid < kGateSamples;
    const bool cand = on && sin_[on ? tid : 0] != 0 && red.topk > 0;
    const double tv = cand ? sv[tid] : 0.0, tm = cand ? smu[tid] : 0.0;
    double hi = cand ? tv - tm : -__builtin_inf(), lo = cand ? tv + tm : __builtin_inf();
    float sum = on ? sp[tid] : 0.0f;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double y = __shfl_xor(hi, o, 64), z = __shfl_xor(lo, o, 64);
        hi = y > hi ? y : hi;
        lo = z < lo ? z : lo;
        sum += __shfl_xor(sum, o, 64);
    }
    // n-plets whose margin reaches the best of the others stand for those that reach the lists
    const int top = __popcll(__ballot(cand && tv + tm >= hi)), bottom = __popcll(__ballot(cand && tv - tm <= lo));
    const float share = (sum + (float)(top > 0 ? top - 1 : 0) + (float)(bottom > 0 ? bottom - 1 : 0)) / kGateSamples;
    uint32_t before = 0;
    if (tid == 0) {
        __hip_atomic_store(&gate.share[d * 32 + k], (uint32_t)(65536.0f * (share < 1.0f ? share : 1.0f)), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        before = __hip_atomic_fetch_add(&gate.done[d], 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (__shfl(before, 0, 64) + 1 < gridDim.x) return;
    float table = 0.0f, factor = 0.0f;
    if (tid < tab.n) {
        const int q = tab.p[tid].k;
        const uint32_t s = __hip_atomic_load(&gate.share[d * 32 + q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        table = (float)s * (1.0f / 65536.0f) * cost.open[q];
        factor = cost.factor[q];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        table += __shfl_xor(table, o, 64);
        factor += __shfl_xor(factor, o, 64);
    }
    if (tid == 0) gate.take[d] = cost.table + table < factor ? 1u : 0u;
}

}  // namespace

void cube_gate_launch(const EvalArgs& a, const CubeTable& tab, const RedArgs& red, const CubeGate& gate, const CubeCost& cost,
                      hipStream_t s)
{
    hipLaunchKernelGGL(k_cube_gate, dim3((unsigned)tab.n, (unsigned)a.D), dim3(kGateThreads), 0, s, a, tab, red, gate, cost);
}

}  // namespace thoi
