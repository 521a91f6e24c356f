// One coordinate of one particle: its start and its move (shared by the swarm
// kernels).  Every product and sum is rounded separately (contraction is off
// here, whatever the including file's) and evaluated in a fixed order, so that
// a swarm is bit-reproducible from its seed.
#pragma once

#include "common.hpp"
#include "fit_eval.hpp"
#include "rng.hpp"

namespace dfit {

// particle p of material m starts at x in [lo, lo + span] with velocity v in
// [-span, span]
__device__ __forceinline__ void pso_start(const PsoArgs &a, int m, int64_t p, int d, double lo, double span, double &x,
                                          double &v) {
#pragma clang fp contract(off)
  const U64x4 r = philox4x64((uint64_t)d, (uint64_t)p, 0, STREAM_PSO_INIT, a.seed, (uint64_t)m);
  x = lo + span * unit53(r.w[0]);
  v = span * (2.0 * unit53(r.w[1]) - 1.0);
}

// iteration t: v <- inertia v + c1 r1 (pbest - x) + c2 r2 (gbest - x), x <- x + v
// clamped to [lo, hi]
__device__ __forceinline__ void pso_move(const PsoArgs &a, int32_t t, int m, int64_t p, int d, bool social,
                                         double pbest, double gbest, double lo, double hi, double &x, double &v) {
#pragma clang fp contract(off)
  const U64x4 r = philox4x64((uint64_t)d, (uint64_t)p, (uint64_t)t, STREAM_PSO_STEP, a.seed, (uint64_t)m);
  const double r1 = unit53(r.w[0]), r2 = unit53(r.w[1]);
  double vel = a.inertia * v;
  vel = vel + (a.c1 * r1) * (pbest - x);
  if (social) vel = vel + (a.c2 * r2) * (gbest - x);
  v = vel;
  const double xn = x + vel;
  x = xn < lo ? lo : (xn > hi ? hi : xn);
}

}  // namespace dfit
