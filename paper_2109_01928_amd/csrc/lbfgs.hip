// Gradient polish of each material's best candidate: L-BFGS (Liu & Nocedal
// 1989) with the two-loop recursion (Nocedal & Wright, Algorithm 7.4) and
// Armijo backtracking alpha = 1, 1/2, 1/4, ... inside the search box: each
// trial point is projected onto [lb, ub] and the sufficient-decrease test uses
// the projected displacement p, C(trial) <= C + c1 min(g.p, 0) (clamping can
// make g.p positive; the cost is then not allowed to rise).  The accepted step
// is the first trial (largest alpha) that passes, which is what a sequential
// halving search returns.  The trials are evaluated in a few batched cost
// launches (the stages below), each only for the materials that the earlier
// ones left undecided (the waves of decided materials exit at once).  A step
// that accepts no trial leaves the point, gradient and history as they were, so
// every later step would rebuild and reject the same trials: such a material
// is marked stalled and left out of all later evaluations.
//
// These kernels are bound by latency: a material's work is a chain of short
// dot products and a few kB of history and trials.  One wavefront a material,
// a component a lane (both halves of the wavefront hold the same), so that rows
// are read and written whole and a dot product is five lane swaps.  With a
// thread a material, 1,024 materials of 12 poles (30 trials) took 156 us a step
// for the direction and 59 for the selections and the update; now 7 and 24.

#include "common.hpp"
#include "fit_eval.hpp"

namespace dfit {

namespace {

// row of trial t of material m in the trial arrays (stage by stage)
__device__ __forceinline__ int64_t trial_row(const LbfgsArgs &a, int m, int t) {
  int lo = 0, hi = a.stage_end[0];
#pragma unroll
  for (int s = 1; s < LBFGS_STAGES; ++s) {
    if (t < hi) break;
    lo = hi;
    hi = a.stage_end[s];
  }
  return (int64_t)a.M * lo + (int64_t)m * (hi - lo) + (t - lo);
}

// component of a trial point
__device__ __forceinline__ double trial_at(double th, double alpha, double d, double lo, double hi) {
  const double v = __builtin_fma(alpha, d, th);
  return v < lo ? lo : (v > hi ? hi : v);
}

// sum over 32 lanes, the same bits in all of them
__device__ __forceinline__ double sum32(double v) {
  v += dpp_quad<QP_SWAP1>(v);
  v += dpp_quad<QP_SWAP2>(v);
  v += dpp_quad<ROW_HALF_MIRROR>(v);   // the quads hold their sums
  v += dpp_quad<ROW_ROR8>(v);
  return v + __shfl_xor(v, 16, WAVE);
}
__device__ __forceinline__ double max32(double v) {
#pragma unroll
  for (int s = 1; s < 32; s <<= 1) v = fmax(v, __shfl_xor(v, s, WAVE));
  return v;
}

// the search direction of material m and its trial points; `rows` holds the
// live history in LDS, oldest pair first: mem rows of s, then mem of y
__device__ void direction(const LbfgsArgs &a, int m, int32_t step, double *rows) {
  constexpr int AHEAD = 16;   // rows in flight
  const int lane = threadIdx.x, i = lane & 31, half = lane >> 5;
  const int N = a.n_poles[m];
  const bool on = i < N;
  const int64_t ld = a.ld, at = (int64_t)m * ld + i;
  const double C = a.cost[m];
  if (a.cost_hist && lane == 0) a.cost_hist[(int64_t)m * (a.steps + 1) + step] = C;
  if (a.stalled[m]) return;   // not evaluated any more
  const double g = on ? a.grad[at] : 0.0;
  bool skip = !(fabs(C) < INFINITY) || __ballot(!(fabs(g) < INFINITY)) != 0;
  double gd = 0.0, d = 0.0;
  if (!skip) {
    const int mem = a.mem, n = a.hist_n[m], first = a.hist_head[m] - n + mem;
    auto slot = [&](int j) { return (first + j) % mem; };
    const double *pairs = (half ? a.Y : a.S) + (int64_t)m * mem * ld + i;
    double *mine = rows + half * mem * DFIT_MAX_POLES + i;
    for (int j0 = 0; j0 < n; j0 += AHEAD) {
      double r[AHEAD];
#pragma unroll
      for (int k = 0; k < AHEAD; ++k)
        if (j0 + k < n && on) r[k] = pairs[slot(j0 + k) * ld];
#pragma unroll
      for (int k = 0; k < AHEAD; ++k)
        if (j0 + k < n && on) mine[(j0 + k) * DFIT_MAX_POLES] = r[k];
    }
    const double rho = lane < n ? a.rho[(int64_t)m * mem + slot(lane)] : 0.0;
    __syncthreads();
    auto s_at = [&](int j) { return on ? rows[j * DFIT_MAX_POLES + i] : 0.0; };
    auto y_at = [&](int j) { return on ? rows[(mem + j) * DFIT_MAX_POLES + i] : 0.0; };
    double q = g, alphas = 0.0;   // alpha of pair j in lane j
    // newest to oldest
    for (int j = n - 1; j >= 0; --j) {
      const double y = y_at(j), alpha = __shfl(rho, j, WAVE) * sum32(s_at(j) * q);
      if (lane == j) alphas = alpha;
      q -= alpha * y;
    }
    if (n > 0) {
      const double s = s_at(n - 1), y = y_at(n - 1);
      q *= sum32(s * y) / sum32(y * y);
    }
    for (int j = 0; j < n; ++j) {
      const double s = s_at(j), b = __shfl(rho, j, WAVE) * sum32(y_at(j) * q);
      q += (__shfl(alphas, j, WAVE) - b) * s;
    }
    d = -q;
    gd = sum32(g * d);
    if (n == 0 || !(gd < 0.0)) {
      // steepest descent, largest component at most one decade
      if (lane == 0) a.hist_n[m] = 0;
      const double gmax = max32(fabs(g));
      if (!(gmax > 0.0)) {
        skip = true;
      } else {
        d = -g * fmin(1.0, 1.0 / gmax);
        gd = sum32(g * d);
      }
    }
  }
  if (lane == 0) a.gd[m] = skip ? NAN : gd;
  if (!on) return;
  if (half == 0) a.dir[at] = d;
  const double th = a.theta[at], lo = a.lb[m], hi = a.ub[m];
  for (int t = half; t < a.max_trials; t += 2)
    a.trial_theta[trial_row(a, m, t) * ld + i] = skip ? th : trial_at(th, ldexp(1.0, -t), d, lo, hi);
}

}  // namespace

__global__ __launch_bounds__(WAVE) void lbfgs_direction_kernel(const LbfgsArgs a) {
  extern __shared__ double rows[];
  direction(a, blockIdx.x, a.step, rows);
}

// After the launch of a stage, trials t_lo .. t_hi (a lane each): the first of
// them that passes the sufficient-decrease test decides the step of a material
// still undecided; after the last stage, no pass is a stall.  After the first
// stage the materials that stalled earlier (their trials were not evaluated) or
// have nothing to step along (non-finite cost or gradient, zero gradient) are
// decided too: no step.
__global__ __launch_bounds__(WAVE) void lbfgs_select_kernel(const LbfgsArgs a, int32_t t_lo, int32_t t_hi) {
  const int m = blockIdx.x, lane = threadIdx.x;
  const int N = a.n_poles[m];
  const bool on = lane < N;
  const int64_t at = (int64_t)m * a.ld + lane;
  const double lo = a.lb[m], hi = a.ub[m], C = a.cost[m], gd = a.gd[m];
  const double th = on ? a.theta[at] : 0.0, g = on ? a.grad[at] : 0.0, d = on ? a.dir[at] : 0.0;
  const bool tried = t_lo + lane <= t_hi;
  const int64_t row = tried ? trial_row(a, m, t_lo + lane) : 0;
  const double cost_t = tried ? a.trial_cost[row] : 0.0;
  const bool ok_t = tried && a.trial_status[row] == ST_OK;
  bool none = false;
  if (t_lo == 0) {
    none = a.stalled[m] || !(gd == gd);
  } else if (a.done[m]) {
    return;
  }
  int pick = -1;
  if (!none) {
    const double alpha = ldexp(1.0, -(t_lo + lane));
    double gp = 0.0;
    for (int i = 0; i < N; ++i) {
      const double th_i = __shfl(th, i, WAVE);
      gp += __shfl(g, i, WAVE) * (trial_at(th_i, alpha, __shfl(d, i, WAVE), lo, hi) - th_i);
    }
    const uint64_t pass = __ballot(ok_t && cost_t <= C + a.c1 * fmin(gp, 0.0));
    if (pass) pick = __ffsll((unsigned long long)pass) - 1;
  }
  const bool stall = none || (pick < 0 && t_hi == a.max_trials - 1);
  const bool decided = pick >= 0 || stall;
  const double c = __shfl(cost_t, pick < 0 ? 0 : pick, WAVE);
  if (lane == 0) {
    a.done[m] = decided;
    if (stall) a.stalled[m] = 1;
    if (decided) {
      a.accepted[m] = pick >= 0;
      a.acc_cost[m] = pick >= 0 ? c : C;
    }
  }
  if (decided && on) a.new_theta[at] = pick >= 0 ? trial_at(th, ldexp(1.0, -(t_lo + pick)), d, lo, hi) : th;
}

// the step's outcome; with `next` the direction of the next step as well
__global__ __launch_bounds__(WAVE) void lbfgs_update_kernel(const LbfgsArgs a, bool next) {
  extern __shared__ double rows[];
  const int m = blockIdx.x, lane = threadIdx.x, i = lane & 31, half = lane >> 5;
  const bool on = i < a.n_poles[m];
  const int64_t ld = a.ld, at = (int64_t)m * ld + i;
  const double cost = a.accepted[m] ? a.acc_cost[m] : a.cost[m];   // the evaluation the acceptance test used
  if (a.accepted[m]) {
    const int mem = a.mem, n = a.hist_n[m], head = a.hist_head[m];
    // the pair is formed in registers and stored only if it is kept: with a
    // full history, slot `head` still holds the oldest live pair, which a
    // rejected pair (s.y <= 1e-300) must not overwrite
    const double th = on ? a.new_theta[at] : 0.0, g = on ? a.new_grad[at] : 0.0;
    const double s = on ? th - a.theta[at] : 0.0, y = on ? g - a.grad[at] : 0.0;
    const double sy = sum32(s * y);
    if (sy > 1e-300) {
      if (on) (half ? a.Y : a.S)[((int64_t)m * mem + head) * ld + i] = half ? y : s;
      if (lane == 0) {
        a.rho[(int64_t)m * mem + head] = 1.0 / sy;
        a.hist_head[m] = (head + 1) % mem;
        a.hist_n[m] = n < mem ? n + 1 : mem;
      }
    }
    if (on && half == 0) {
      a.theta[at] = th;
      a.grad[at] = g;
    }
    if (lane == 0) a.cost[m] = cost;
  }
  if (a.cost_hist && a.step == a.steps - 1 && lane == 0) a.cost_hist[(int64_t)m * (a.steps + 1) + a.steps] = cost;
  if (next) {
    __syncthreads();   // the stores above are read by other lanes
    direction(a, m, a.step + 1, rows);
  }
}

static uint32_t rows_bytes(const LbfgsArgs &a) { return 2u * a.mem * DFIT_MAX_POLES * sizeof(double); }

hipError_t launch_lbfgs_direction(const LbfgsArgs &a, hipStream_t s) {
  hipLaunchKernelGGL(lbfgs_direction_kernel, dim3(a.M), dim3(WAVE), rows_bytes(a), s, a);
  return hipGetLastError();
}
hipError_t launch_lbfgs_select(const LbfgsArgs &a, int32_t t_lo, int32_t t_hi, hipStream_t s) {
  hipLaunchKernelGGL(lbfgs_select_kernel, dim3(a.M), dim3(WAVE), 0, s, a, t_lo, t_hi);
  return hipGetLastError();
}
hipError_t launch_lbfgs_update(const LbfgsArgs &a, bool next, hipStream_t s) {
  hipLaunchKernelGGL(lbfgs_update_kernel, dim3(a.M), dim3(WAVE), next ? rows_bytes(a) : 0, s, a, next);
  return hipGetLastError();
}

}  // namespace dfit
