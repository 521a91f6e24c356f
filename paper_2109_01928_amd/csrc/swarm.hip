// A whole particle-swarm fit in one launch: one block per material, which
// draws its swarm, then alternates evaluating every particle (the cost
// kernel's tile, one wavefront a tile, the waves sharing the material's tiles)
// and moving it, for all iterations.  Materials are independent, so no block
// waits for another.
//
// For fits too small to fill the chip.  Launched step by step, an iteration of
// 40 particles (N = 5, 50 points) took 32 us, of which the evaluation's one
// wavefront ran 15, the move 5, the counter of the replayed graph 4 and the
// gaps between them the rest; here it takes 12 us (the whole fit of 50
// iterations 1,425 -> 603 us).  24 materials of 64 particles (N = 6, 100
// points), 100 iterations: 3,185 -> 1,749 us.  What is left is one wavefront's
// chain through the cost kernel's two passes and solve, at one wavefront a
// SIMD: a block has up to 512 registers a lane, and nothing spills (at two, N >=
// 7 spilled and lost to the steps: 60 and 25 us an iteration).

#include "fit_kernel.hpp"
#include "pso.hpp"

namespace dfit {

namespace {

// lowest-index minimum over the block: (v, i) of every thread, i < 0 none
__device__ __forceinline__ void take_min(double &v, int32_t &i, double v2, int32_t i2) {
  if (i2 >= 0 && (i < 0 || v2 < v || (v2 == v && i2 < i))) {
    v = v2;
    i = i2;
  }
}

}  // namespace

// LDS of a block beyond its waves' regions: positions, velocities, personal
// bests, their costs and the last ones, and the spectra, in doubles; then a
// byte a particle
int64_t swarm_state_bytes(int64_t P, int N, int64_t F) { return 8 * (P * (3 * N + 2) + 3 * F) + ((P + 7) & ~(int64_t)7); }

// What an evaluation needs of the launch and of the block (LDS addresses as
// byte offsets).
struct Eval {
  double damping;
  int8_t *status;   // of the material's first particle, or NULL
  uint32_t flags, region, state;
  int32_t freq_split, cand_per_wave, P, F;
};

// The costs of the wave's tiles.  What it derives is hidden from the loop it
// stands in, which would keep it in registers across the iterations and spill
// the tile's passes.
template <int N> __device__ __forceinline__ void swarm_eval(Eval in, int32_t wave, int32_t waves) {
  asm volatile("" : "+s"(in.region), "+s"(in.state), "+s"(in.freq_split), "+s"(in.cand_per_wave), "+s"(in.P), "+s"(in.F));
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  FitArgs fit{};
  fit.damping = in.damping;
  fit.flags = in.flags;
  fit.freq_split = in.freq_split;
  fit.cand_per_wave = in.cand_per_wave;
  fit.status = in.status;
  auto at = [](uint32_t offset) { return (double *)(lds_ptr)offset; };
  double *const x = at(in.state), *const cost = x + in.P * (3 * N + 1), *const om = cost + in.P;
  const OwnTile own = {tid, at(in.region), in.P, in.F, x, om, om + in.F, om + 2 * in.F, cost};
  for (int32_t tile = wave; tile * in.cand_per_wave < in.P; tile += waves)
    fit_tile<N, pole_split_for(N), false, 2, false, true>(fit, tile, own);
}

template <int N>
__global__ __launch_bounds__(64 * SWARM_WAVES) __attribute__((amdgpu_waves_per_eu(N <= 5 ? 2 : 1)))
void swarm_kernel(const FitArgs fit, const PsoArgs a, const int32_t *mats, int32_t iters, int32_t lds_per_wave) {
  __shared__ double w_val[SWARM_WAVES], g_row[N];
  __shared__ int32_t w_idx[SWARM_WAVES];
  extern __shared__ double lds_block[];
  const int tid = threadIdx.x, threads = blockDim.x, waves = threads >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int m = mats[blockIdx.x];
  const int64_t c0 = a.cand_off[m], f0 = fit.f_off[m];
  const int32_t P = (int32_t)(a.cand_off[m + 1] - c0), F = (int32_t)(fit.f_off[m + 1] - f0);
  const int64_t ld = a.ld;
  const double lo = a.lb[m], hi = a.ub[m];
  double *const x = lds_block + (int64_t)waves * (lds_per_wave >> 3);
  double *const v = x + P * N, *const px = v + P * N, *const pc = px + P * N, *const cost = pc + P;
  double *const om = cost + P, *const er = om + F, *const ei = er + F;
  uint8_t *const improved = (uint8_t *)(ei + F);

  for (int32_t k = tid; k < F; k += threads) {
    om[k] = fit.omega[f0 + k];
    er[k] = fit.eps_re[f0 + k];
    ei[k] = fit.eps_im[f0 + k];
  }
  for (int32_t e = tid; e < P * N; e += threads) {
    double xi, vi;
    pso_start(a, m, e / N, e % N, lo, hi - lo, xi, vi);
    x[e] = xi;
    v[e] = vi;
    px[e] = xi;
  }
  for (int32_t p = tid; p < P; p += threads) pc[p] = INFINITY;
  double g_cost = INFINITY;
  int32_t g_idx = -1;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_ptr)lds_block;
  const Eval eval = {fit.damping, fit.status ? fit.status + c0 : nullptr, fit.flags, lds0 + (uint32_t)(wave * lds_per_wave),
                     lds0 + (uint32_t)(waves * lds_per_wave), fit.freq_split, fit.cand_per_wave, P, F};

  for (int32_t t = 1;; ++t) {
    __syncthreads();   // the positions
    swarm_eval<N>(eval, wave, waves);
    __syncthreads();   // the costs
    // personal bests (strict improvement; NaN never compares less) and the
    // lowest-index minimum of them
    double bv = INFINITY;
    int32_t bi = -1;
    for (int32_t p = tid; p < P; p += threads) {
      const double f = cost[p], old = pc[p];
      const bool better = f < old;
      improved[p] = better;
      if (better) pc[p] = f;
      take_min(bv, bi, better ? f : old, p);
    }
#pragma unroll
    for (int s = 1; s < WAVE; s <<= 1) {
      const double v2 = __shfl_xor(bv, s, WAVE);
      const int32_t i2 = __shfl_xor(bi, s, WAVE);
      take_min(bv, bi, v2, i2);
    }
    if ((tid & 63) == 0) {
      w_val[wave] = bv;
      w_idx[wave] = bi;
    }
    __syncthreads();   // the waves' minima, and which particles improved
    bv = w_val[0];
    bi = w_idx[0];
    for (int w = 1; w < waves; ++w) take_min(bv, bi, w_val[w], w_idx[w]);
    const bool take = bi >= 0 && bv < g_cost;
    if (take) {
      g_cost = bv;
      g_idx = bi;
      if (tid < N) g_row[tid] = (improved[bi] ? x : px)[bi * N + tid];
    }
    if (tid == 0 && a.history) a.history[(int64_t)m * a.hist_ld + (t - 1)] = g_cost;
    __syncthreads();   // the best row
    const bool social = g_idx >= 0, move = t <= iters;
    for (int32_t e = tid; e < P * N; e += threads) {
      const int32_t p = e / N, d = e - p * N;
      double xi = x[e];
      if (improved[p]) px[e] = xi;
      if (move) {
        double vi = v[e];
        pso_move(a, t, m, p, d, social, px[e], social ? g_row[d] : 0.0, lo, hi, xi, vi);
        v[e] = vi;
        x[e] = xi;
      }
    }
    if (!move) break;
  }
  for (int32_t e = tid; e < P * N; e += threads) {
    const int64_t at = (c0 + e / N) * ld + e % N;
    a.x[at] = x[e];
    a.v[at] = v[e];
    a.pbest_x[at] = px[e];
  }
  for (int32_t p = tid; p < P; p += threads) {
    a.pbest_cost[c0 + p] = pc[p];
    fit.cost[c0 + p] = cost[p];
  }
  if (g_idx >= 0 && tid < N) a.gbest_x[(int64_t)m * ld + tid] = g_row[tid];
  if (tid == 0) {
    a.gbest_cost[m] = g_cost;
    a.gbest_idx[m] = g_idx;
  }
}

namespace {
template <int N>
hipError_t launch_n(const FitArgs &fit, const PsoArgs &a, const int32_t *mats, int32_t n_mats, int32_t waves,
                    int32_t state_bytes, int32_t iters, hipStream_t s) {
  const int32_t per_wave = Shape<N, pole_split_for(N)>::LDS_DOUBLES * 8 * fit.cand_per_wave;
  const int32_t bytes = per_wave * waves + state_bytes;
  if (bytes > 64 * 1024) {   // beyond the default limit of dynamic LDS
    const hipError_t e = hipFuncSetAttribute((const void *)swarm_kernel<N>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, SWARM_LDS);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL((swarm_kernel<N>), dim3((unsigned)n_mats), dim3(64 * waves), (size_t)bytes, s, fit, a,
                     mats, iters, per_wave);
  return hipGetLastError();
}
template <int... Ns> struct SwarmTable {
  static hipError_t run(int n, const FitArgs &fit, const PsoArgs &a, const int32_t *mats, int32_t n_mats, int32_t waves,
                        int32_t state_bytes, int32_t iters, hipStream_t s) {
    hipError_t e = hipErrorInvalidValue;
    ((n == Ns ? (e = launch_n<Ns>(fit, a, mats, n_mats, waves, state_bytes, iters, s)) : hipSuccess), ...);
    return e;
  }
};
}  // namespace

hipError_t launch_swarm(int n, const FitArgs &fit, const PsoArgs &a, const int32_t *mats, int32_t n_mats, int32_t waves,
                        int32_t state_bytes, int32_t iters, hipStream_t s) {
  static_assert(SWARM_POLES == 11, "the instantiations below");
  return SwarmTable<1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11>::run(n, fit, a, mats, n_mats, waves, state_bytes, iters, s);
}

}  // namespace dfit
