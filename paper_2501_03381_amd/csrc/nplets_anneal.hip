// Batched simulated annealing run on the device (Methods, "Heuristics", "Simulated Annealing
// Algorithm").  In each iteration every chain proposes a neighbour, evaluates its O-information (Eq.
// O-info with TC and DTC from one Cholesky factorisation) and applies the Metropolis rule; a launch
// runs up to kAnnealSteps iterations, so a whole run is enqueued without a host round trip.
//
// Orders up to 32: two chains per 64-lane wavefront, each half-wave factoring its chain's
// neighbour with the rows in registers (the pair factorisation, entries from Sigma staged in LDS).
// Larger orders (up to 64): one wavefront per chain, the block gathered into LDS.  In both, every lane
// of a chain forms its neighbour from the chain's mask and draws, takes the decision and updates the
// chain's state, which stays in registers for the launch.  Masks are two 64-bit words (N <= 128).  The
// random numbers are inputs (one row of draws per iteration), so a run is reproducible bit for bit.
#include "thoi_internal.hpp"
#include "nplets_common.hpp"
#include "pair_factor_lat.hpp"
#include "search_mask.hpp"

namespace thoi {
namespace {

constexpr int64_t kAnnealSteps = 256;      // iterations per launch

struct AnnealArgs {
    const double* Sigma;
    int N;
    int kappa;
    int across;
    int kmin, kmax;
    double sign;                   // +1: maximise Omega, -1: minimise
    const double* move;            // [iters][kappa] (across orders only)
    const double* a;               // [iters][kappa] which member leaves
    const double* b;               // [iters][kappa] which outsider enters
    const double* u;               // [iters][kappa] acceptance draw
    Mask* cur;
    double* cur_om;
    Mask* best;
    double* best_om;
    int64_t* acc;
};

__device__ __forceinline__ Mask full_mask(int N)
{
    Mask f;
    f.w[0] = N >= 64 ? ~0ull : ((1ull << N) - 1ull);
    f.w[1] = N >= 128 ? ~0ull : (N > 64 ? ((1ull << (N - 64)) - 1ull) : 0ull);
    return f;
}

// The neighbour of mask `cur` (Methods, "Simulated Annealing Algorithm"): within an order a member
// is swapped for an outsider; across orders a member is added (move < 1/3), removed
// (1/3 <= move < 2/3) or swapped, a swap also replacing a move that would leave [kmin, kmax].  The
// member is the floor(a k)-th set bit and the outsider the floor(b (N - k))-th clear bit, both in
// ascending order.
__device__ __forceinline__ Mask propose(Mask cur, int N, bool across, int kmin, int kmax, double move, double a,
                                        double b)
{
    const Mask full = full_mask(N);
    const int k = popc(cur);
    const bool add = across && move < 1.0 / 3.0 && k < kmax;
    const bool rem = across && move >= 1.0 / 3.0 && move < 2.0 / 3.0 && k > kmin;
    const bool swap = !(add || rem);
    Mask out;
    out.w[0] = ~cur.w[0] & full.w[0];
    out.w[1] = ~cur.w[1] & full.w[1];
    const int drop = nth_set(cur, (int)(int64_t)(a * (double)k));
    const int take = nth_set(out, (int)(int64_t)(b * (double)(N - k)));
    Mask p = cur;
    if (swap || rem) p.w[drop >> 6] &= ~(1ull << (drop & 63));
    if (swap || add) p.w[take >> 6] |= 1ull << (take & 63);
    return p;
}

// A chain's state.
struct Chain {
    Mask cur, best;
    double om, best_om;
    int64_t acc;
};

__device__ __forceinline__ Mask start_mask(const Mask* __restrict__ masks0, int c, int N)
{
    const Mask full = full_mask(N);
    Mask p;
    p.w[0] = masks0[c].w[0] & full.w[0];
    p.w[1] = masks0[c].w[1] & full.w[1];
    return p;
}

__device__ __forceinline__ Chain load_chain(const AnnealArgs& g, int c)
{
    return Chain{g.cur[c], g.best[c], g.cur_om[c], g.best_om[c], g.acc[c]};
}

__device__ __forceinline__ void store_chain(const AnnealArgs& g, int c, const Chain& s)
{
    g.cur[c] = s.cur;
    g.cur_om[c] = s.om;
    g.best[c] = s.best;
    g.best_om[c] = s.best_om;
    g.acc[c] = s.acc;
}

// Omega = TC - DTC with TC = -ld/2 and DTC = (ld + sum_j log a_j)/2; NaN if not positive definite.
__device__ __forceinline__ double omega_of(const FactorOut<double>& f)
{
    const bool ok = f.ok && isfinite(f.ld) && isfinite(f.sa);
    const double TC = -0.5 * f.ld, DTC = 0.5 * (f.ld + f.sa);
    return ok ? TC - DTC : __builtin_nan("");
}

// The Metropolis decision on neighbour p: energy E = sign * Omega; p is taken when dE > 0, else with
// probability exp(dE / temp); a neighbour that is not positive definite is never taken.
__device__ __forceinline__ void metropolis(Chain& s, double sign, double temp, double u, const Mask& p, double om)
{
    const double E = sign * s.om;
    const double Ep = sign * om;
    const double dE = Ep - E;
    const bool take = ((dE > 0.0) || (u < exp(dE / temp))) && !isnan(Ep);
    if (take) {
        s.cur = p;
        s.om = om;
        s.acc += 1;
    }
    if (sign * s.om > sign * s.best_om) {
        s.best = s.cur;
        s.best_om = s.om;
    }
}

struct Draws {
    double move, a, b, u;
};

__device__ __forceinline__ Draws load_draws(const AnnealArgs& g, int c, int64_t t)
{
    const int64_t e = t * g.kappa + c;
    return Draws{g.across ? g.move[e] : 0.0, g.a[e], g.b[e], g.u[e]};
}

// Whole workgroup: the lower triangle of Sigma packed by rows, and 1/sqrt of its diagonal.
__device__ __forceinline__ void stage_lower(const double* __restrict__ Sigma, int N, double* __restrict__ sLow,
                                            double* __restrict__ sIsd)
{
    const int bd = (int)blockDim.x;
    for (int e0 = threadIdx.x; e0 < N * N; e0 += 8 * bd) {
        double v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = e0 + u * bd < N * N ? Sigma[e0 + u * bd] : 0.0;
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int e = e0 + u * bd, i = e / N, j = e - i * N;
            if (e < N * N && j <= i) sLow[i * (i + 1) / 2 + j] = v[u];
            if (e < N * N && j == i) sIsd[i] = inv_sd(v[u]);
        }
    }
    __syncthreads();
}

// Iterations t0 .. t0 + nt - 1 of every chain in one launch: chains are independent of each other, so
// a chain's state stays in registers and the next iteration's draws are loaded while the current
// neighbour is factored.  One launch per iteration (each starting with a cold instruction cache, the
// state and the draws in memory) took 30.9 us per iteration of 1024 chains at order 20.
// masks0 != null: the starting state is evaluated first; else it is what an earlier launch left.
//
// Orders up to kW2Max: grid (ceil(kappa / (2 W))), block 64 W, two chains per wavefront.  The
// covariance's lower triangle (N (N + 1) / 2 doubles) and the N factors 1/sqrt(Sigma_jj) stay in LDS
// for the launch: a neighbour's entries are scattered over the rows, and gathered from memory each of
// its k columns cost a cache line per row (8,300 of the 26,000 cycles of an iteration at order 20 and
// N = 100).  Dynamic LDS: the triangle, then the factors.
__global__ __launch_bounds__(256) void k_anneal_pair(AnnealArgs g, const Mask* __restrict__ masks0, int64_t t0, int nt,
                                                     double temp, double alpha)
{
    extern __shared__ double sLow[];
    __shared__ double scol_w[4][2 * 2 * kW2Max], swrow_w[4][2 * 2 * kW2Max];
    __shared__ int sch_w[4][2 * kW2Max];
    const int N = g.N;
    double* sIsd = sLow + N * (N + 1) / 2;
    stage_lower(g.Sigma, N, sLow, sIsd);
    const int wv = threadIdx.x >> 6;
    double* scol = scol_w[wv];
    double* swrow = swrow_w[wv];
    int* sch = sch_w[wv];
    const int lane = threadIdx.x & 63, h = lane >> 5, i = lane & 31;
    const int c = 2 * (int)(blockIdx.x * (blockDim.x >> 6) + wv) + h;
    const bool live = c < g.kappa;
    // a half-wave past the last chain follows it and stores nothing
    const int cc = live ? c : g.kappa - 1;
    int* ch = sch + h * kW2Max;
    Chain s{};
    const bool init = masks0 != nullptr;
    if (!init) s = load_chain(g, cc);
    Draws dr{};
    if (nt > 0) dr = load_draws(g, cc, t0);
    for (int t = init ? -1 : 0; t < nt; ++t) {
        const Mask p = t < 0 ? start_mask(masks0, cc, g.N)
                             : propose(s.cur, g.N, g.across != 0, g.kmin, g.kmax, dr.move, dr.a, dr.b);
        const double u = dr.u;
        if (t >= 0 && t + 1 < nt) dr = load_draws(g, cc, t0 + t + 1);
        int kh = popc(p);
        kh = kh < kW2Max ? kh : kW2Max;
        wave_sync();                                      // the last factorisation has read its indices
        if (i < kh) ch[i] = nth_set(p, i);
        wave_sync();
        // every shuffle runs with the whole wavefront active
        const int k0 = __shfl(kh, 0), k1 = __shfl(kh, 32);
        const FactorOut<double> f = pair_factor_lat<PairSource::Lower>(
            sLow, N, ch, k0 > k1 ? k0 : k1, kh, scol + h * 2 * kW2Max, swrow + h * 2 * kW2Max, sIsd);
        const double om = omega_of(f);
        if (t < 0) {
            s = Chain{p, p, om, om, 0};
        } else {
            metropolis(s, g.sign, temp, u, p, om);
            temp *= alpha;
        }
    }
    if (i == 0 && live) store_chain(g, c, s);
}

// Omega of the n-plet (w0, w1) by one wavefront, at most kmax members (the clamp keeps a starting mask outside the
// range of orders in bounds of the block).  A call, not inlined: inside the loop over iterations the compiler
// unrolled the factorisation's loops otherwise (500 chains of N = 100, 200 iterations, order 64 41.1 ms, 30.8 so; order
// 40 17.7 and 14.7; one launch per iteration 32.4 and 16.0).
__device__ __attribute__((noinline)) double wave_omega(GlobalDouble Sigma, int N, uint64_t w0, uint64_t w1, int kmax,
                                                       LdsDouble sM,
                                                       LdsDouble sInv, LdsDouble sIsd, LdsInt cidx)
{
    const Mask p{{w0, w1}};
    const int ks = kmax + 1, lane = threadIdx.x & 63;
    int k = popc(p);
    k = __builtin_amdgcn_readfirstlane(k < kmax ? k : kmax);
    // the block's variables and 1/sqrt of their variances, then the correlation block row by row:
    // R_ij = (Sigma_ij / sqrt(Sigma_ii)) / sqrt(Sigma_jj), unit diagonal
    int ci = 0;
    if (lane < k) {
        ci = nth_set(p, lane);
        cidx[lane] = ci;
        sIsd[lane] = inv_sd(Sigma[(int64_t)ci * N + ci]);
    }
    __syncthreads();
    if (lane < k)
        gather_row((const double*)(Sigma + (int64_t)ci * N), (const int*)cidx, (const double*)sIsd, lane, (double*)(sM + lane * ks));
    __syncthreads();
    return omega_of(wave_factor_core(k, (double*)sM, ks, (double*)sInv));
}

// grid (kappa), block 64: one wavefront per chain, orders up to 64 (otherwise as above).
// Dynamic LDS: the factorisation block, kmax rows of stride kmax + 1 (sized for the largest order a
// chain reaches, so that smaller maxima leave room for more wavefronts per CU); static: sInv [64] |
// sIsd [64] | cidx [64].
__global__ __launch_bounds__(64) void k_anneal(AnnealArgs g, const Mask* __restrict__ masks0, int64_t t0, int nt,
                                               double temp, double alpha)
{
    extern __shared__ double sM[];
    __shared__ double sInv[64], sIsd[64];
    __shared__ int cidx[64];
    const int N = g.N;
    const int c = blockIdx.x;
    const int lane = threadIdx.x;
    Chain s{};
    const bool init = masks0 != nullptr;
    if (!init) s = load_chain(g, c);
    Draws dr{};
    if (nt > 0) dr = load_draws(g, c, t0);
    for (int t = init ? -1 : 0; t < nt; ++t) {
        const Mask p = t < 0 ? start_mask(masks0, c, N)
                             : propose(s.cur, N, g.across != 0, g.kmin, g.kmax, dr.move, dr.a, dr.b);
        const double u = dr.u;
        if (t >= 0 && t + 1 < nt) dr = load_draws(g, c, t0 + t + 1);
        __syncthreads();                                  // the last factorisation is done with the LDS
        const double om = wave_omega((GlobalDouble)g.Sigma, N, p.w[0], p.w[1], g.kmax, (LdsDouble)sM, (LdsDouble)sInv,
                                     (LdsDouble)sIsd, (LdsInt)cidx);
        if (t < 0) {
            s = Chain{p, p, om, om, 0};
        } else {
            metropolis(s, g.sign, temp, u, p, om);
            temp *= alpha;
        }
    }
    if (lane == 0) store_chain(g, c, s);
}

}  // namespace

thoi_status launch_anneal(const double* Sigma, int32_t N, const uint64_t* masks0, int32_t kappa, int32_t iters,
                          const double* draw_move, const double* draw_a, const double* draw_b, const double* draw_u,
                          double T0, double alpha, int32_t maximize, int32_t across, int32_t k_min, int32_t k_max,
                          uint64_t* cur_mask, double* cur_omega, uint64_t* best_mask, double* best_omega,
                          int64_t* accepted, hipStream_t s)
{
    AnnealArgs g{};
    g.Sigma = Sigma;
    g.N = N;
    g.kappa = kappa;
    g.across = across ? 1 : 0;
    g.kmin = k_min;
    g.kmax = k_max;
    g.sign = maximize ? 1.0 : -1.0;
    g.move = draw_move;
    g.a = draw_a;
    g.b = draw_b;
    g.u = draw_u;
    g.cur = reinterpret_cast<Mask*>(cur_mask);
    g.cur_om = cur_omega;
    g.best = reinterpret_cast<Mask*>(best_mask);
    g.best_om = best_omega;
    g.acc = accepted;
    const Mask* m0 = reinterpret_cast<const Mask*>(masks0);
    // every order a chain can reach is at most k_max: the pair factorisation when it fits
    const bool pair = k_max <= kW2Max;
    // two chains per wavefront; wavefronts share a workgroup's copy of Sigma once there are more
    // than two workgroups per CU of them
    const int waves = (kappa + 1) / 2;
    const int W = !pair || waves <= 512 ? 1 : (waves <= 1024 ? 2 : 4);
    const dim3 grid(pair ? (unsigned)((waves + W - 1) / W) : (unsigned)kappa), block(64 * W);
    const size_t lds = pair ? ((size_t)N * (N + 1) / 2 + N) * sizeof(double)
                            : (size_t)k_max * (size_t)(k_max + 1) * sizeof(double);
    // at most kAnnealSteps iterations per launch keep a launch short (a few ms)
    double temp = T0;
    for (int64_t t = 0; t == 0 || t < iters; t += kAnnealSteps) {
        const int nt = (int)((int64_t)iters - t < kAnnealSteps ? (int64_t)iters - t : kAnnealSteps);
        const Mask* start = t == 0 ? m0 : nullptr;
        if (pair) hipLaunchKernelGGL(k_anneal_pair, grid, block, lds, s, g, start, t, nt, temp, alpha);
        else hipLaunchKernelGGL(k_anneal, grid, block, lds, s, g, start, t, nt, temp, alpha);
        // the temperature of iteration t is T0 multiplied by alpha t times, one product at a time
        for (int j = 0; j < nt; ++j) temp *= alpha;
    }
    return hip_status(hipGetLastError());
}

}  // namespace thoi
