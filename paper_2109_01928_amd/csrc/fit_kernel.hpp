// Batched multi-Debye DLS cost evaluation and its variable-projection adjoint
// for gfx950 (MI355X), FP64.
//
// Method (paper Sec. III-B; Eq. 7 basis with the sign of Eq. 1):
//   tau_i = 10^theta_i, x_ki = w_k tau_i, R_ki = 1/(1+x^2), I_ki = x R_ki
//   weights: damped least squares on the loss part with Marquardt scaling,
//     (D^-1 G D^-1 + damping Id) zt = D^-1 b,  G = I^T I, b = I^T eps'', D = diag(G)^1/2,
//     z = D^-1 zt, solved by Cholesky plus one corrected-semi-normal-equations
//     step (a residual pass over the frequencies, I^T r accumulated with
//     compensation) because log-spaced Debye columns are nearly collinear;
//   flip: w = |z| (penalty for negative weights);
//   eps_inf = (sum_k eps'_k - sum_i w_i S_i) / F,  S_i = sum_k R_ki;
//   cost = sum_k (eps'_k - eps_inf - (R w)_k)^2 + (eps''_k - (I w)_k)^2.
//
// Work decomposition (one wavefront per work tile, one tile per 64-lane block):
//   - a candidate is served by SP x SF lanes: SP lanes split its poles (the
//     "ring" split below) and SF lanes split its frequency points;
//   - the 64/(SP*SF) candidates of a wave are listed by the plan (any mix of
//     materials with the same pole count);
//   - every F-reduction is a per-lane register accumulation followed by a
//     fixed butterfly over the SF lanes, so results are deterministic;
//   - passes: (1) Gram and right-hand side, (2) refinement residual (and,
//     for the adjoint, the column sums S), (3) cost; passes 1 and 2
//     recompute the basis in registers (it is never stored; four poles share
//     one reciprocal), pass 3 evaluates the model sums as rational functions
//     of w^2 (basis form as the fallback), and the adjoint adds pass 4.
//
// Gram matrix on the two-lane split (SP = 2): the NP = 2 NB (padded) poles are
// placed on a ring; lane q owns poles q*NB .. q*NB+NB-1 and accumulates, for
// each owned pole p and each offset d = 0..NP/2, the entry G(p, (p+d) mod NP).
// Every unordered pair is covered (the d = NP/2 entries twice, with
// bit-identical values), the work is balanced, and a lane only needs the basis
// values of the next NP/2 poles on the ring, which it receives from its
// neighbour by DPP quad permutes.  Padded poles get tau = 0, so their loss
// column is exactly zero and they drop out.
//
// Gram matrix on the four-lane split (SP = 4, N >= 15): 4x4 tiles of poles on
// the matrix cores, v_mfma_f64_4x4x4 (four blocks; D += A B per block, K = 4
// points).  Its lanes are numbered pole (bits 0-1), block (bits 2-3), point
// (bits 4-5) in A and in B alike, so a lane that forms the basis of poles
// q, 4 + q, 8 + q, ... at its point holds the operands of every tile as they
// are: no value moves between lanes, and the accumulators are one register
// pair a tile (15 at N = 20) where the ring held 55.  The instruction takes
// the FP64 pipe for 16 cycles (four issue slots): 60 slots a wave and point
// for the tiles at N = 20, against 75 for the ring's 55 fused multiply-adds
// and 20 moves; alone it sustained 68.6 TFLOP/s, chains of fused multiply-adds
// 62.7, the two mixed 71 to 74.  A candidate's lanes hold at least four points
// (SF >= 4), so a wave holds at most four candidates, and the solves are shared
// by 16 lanes (Coop).  Both against the ring with SF = 2 and solves run by
// every lane, forward evaluation of N = 20 on one box: F = 4096 (32,768
// candidates) 3.06 -> 2.69 ms, F = 200 (131,072) 1.18 -> 0.87 ms, F = 50 0.92
// -> 0.58 ms; N = 17 at F = 4096 3.00 -> 2.71 ms, N = 24 3.88 -> 3.35 ms; the
// adjoint at N = 20, F = 4096, 6.00 -> 5.45 ms; N = 16 (65,536 candidates of F =
// 2000) 2.08 -> 1.96 ms, (131,072 of F = 200) 0.80 -> 0.63 ms.  At N = 12 to 14
// the padding to whole tiles and the smaller reciprocal groups of a lane cost
// what the ring's moves do, or more (F = 2000: N = 12 1.45 ms on the ring, 1.46
// on tiles; N = 13 1.74 and 1.93).

#pragma once

#include <type_traits>

#include "common.hpp"
#include "fit_eval.hpp"

namespace dfit {

using lds_ptr = __attribute__((address_space(3))) double *;
using lds_cptr = const __attribute__((address_space(3))) double *;

template <int N, int SP> struct Shape {
  static_assert(SP == 1 || SP == 2 || SP == 4, "pole split must be 1, 2 or 4");
  static constexpr bool MF = SP == 4;                        // Gram on the matrix cores
  static constexpr int NB = (N + SP - 1) / SP;               // poles owned per lane
  static constexpr int NP = NB * SP;                         // padded pole count
  static constexpr int D = (SP == 2) ? NP / 2 : 0;           // ring half width
  static constexpr int NV = (SP == 2) ? NB + D : NB;         // basis values seen by a lane
  // Gram accumulators: the triangle, the tiles' upper triangle, or the ring's
  static constexpr int NG = (SP == 1) ? N * (N + 1) / 2 : MF ? NB * (NB + 1) / 2 : NB * (D + 1);
  static constexpr int NT = N * (N + 1) / 2;                 // packed triangle
  // per candidate: the parked factor (SP == 1), or the whole solve (SP > 1)
  static constexpr int LDS_DOUBLES = (SP == 1) ? N * (N + 1) / 2 : N * (N + 1) / 2 + (MF ? 6 : 5) * N;
};

constexpr __host__ __device__ int tri(int n, int i, int j) { return i * n - (i * (i - 1)) / 2 + (j - i); }

// Orders a wave's LDS accesses across its lanes: the LDS serves one wave's
// accesses in order, so only the compiler has to keep it.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// the neighbour's value on the two-lane ring
__device__ __forceinline__ double ring_fetch(double v) { return dpp_quad<QP_SWAP1>(v); }

// xor mask, in the wave's lane numbers, of bit m of a lane's index among its
// candidate's lanes: the same number, except on the four-lane split, whose
// lanes are numbered as the matrix instruction has them (pole lane in bits
// 0-1, block in bits 2-3, point in bits 4-5) and a candidate's lanes by pole
// lane, point, block
template <int SP> constexpr int lane_mask(int m) { return SP == 4 ? (m < 4 ? m : m < 16 ? m << 2 : m >> 2) : m; }

// A lane's value and that of lane ^ MASK, as a pair whose order does not matter
// (both lanes get the same two): by DPP inside a row of 16 lanes and by the
// row and half swaps across rows, all in the vector unit.  Through the LDS
// crossbar (ds_bpermute) each step of a butterfly waited for a round trip: the
// sums after the Gram pass took 2,500 of an evaluation's 21,000 cycles for 40
// candidates of 5 poles and 50 points at split 8.
struct Two {
  double a, b;
};
template <int MASK> __device__ __forceinline__ Two with_lane_xor(double v) {
  if constexpr (MASK == 1) {
    return {v, dpp_quad<QP_SWAP1>(v)};
  } else if constexpr (MASK == 2) {
    return {v, dpp_quad<QP_SWAP2>(v)};
  } else if constexpr (MASK == 4) {
    return {v, dpp_quad<QP_REV>(dpp_quad<ROW_HALF_MIRROR>(v))};   // lane ^ 7 ^ 3
  } else if constexpr (MASK == 8) {
    return {v, dpp_quad<ROW_ROR8>(v)};
  } else {
    const uint32_t lo = (uint32_t)__double2loint(v), hi = (uint32_t)__double2hiint(v);
    if constexpr (MASK == 16) {
      const auto l = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
      const auto h = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
      return {__hiloint2double((int)h[0], (int)l[0]), __hiloint2double((int)h[1], (int)l[1])};
    } else {
      const auto l = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
      const auto h = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
      return {__hiloint2double((int)h[0], (int)l[0]), __hiloint2double((int)h[1], (int)l[1])};
    }
  }
}

// step(mask) for the bits FROM .. s_lanes / 2 of a lane's index among its
// candidate's lanes
template <int SP, int FROM, class STEP> __device__ __forceinline__ void each_bit(int s_lanes, STEP &&step) {
  if constexpr (FROM < WAVE) {
    if (FROM < s_lanes) {
      step(std::integral_constant<int, lane_mask<SP>(FROM)>());
      each_bit<SP, FROM * 2>(s_lanes, step);
    }
  }
}

// sum over the SP lanes of a candidate (bit-identical in all of them)
template <int SP> __device__ __forceinline__ double group_sum(double v) {
  if constexpr (SP == 1) {
    return v;
  } else if constexpr (SP == 2) {
    return v + dpp_quad<QP_SWAP1>(v);
  } else {
    v = v + dpp_quad<QP_SWAP1>(v);
    return v + dpp_quad<QP_SWAP2>(v);
  }
}

// sums over the SF frequency lanes of a candidate (xor butterfly over the bits
// from FROM on; all lanes end with the same bits)
template <int K, int SP, int FROM> __device__ __forceinline__ void freq_sum_n(double *v, int s_lanes) {
  each_bit<SP, FROM>(s_lanes, [&](auto mask) {
#pragma unroll
    for (int e = 0; e < K; ++e) {
      const Two t = with_lane_xor<decltype(mask)::value>(v[e]);
      v[e] = t.a + t.b;
    }
  });
}
template <int SP, int FROM> __device__ __forceinline__ double freq_sum(double v, int s_lanes) {
  freq_sum_n<1, SP, FROM>(&v, s_lanes);
  return v;
}

// Compensated accumulation sum += a * b (Kahan's summation with the running
// correction c folded into the product by a fused multiply-add): the error of
// a length-F sum stays at a few units of roundoff of the terms' magnitude
// instead of growing with F.  The true sum is sum - c.
__device__ __forceinline__ void kahan_fma_acc(double &sum, double &c, double a, double b) {
  const double y = __builtin_fma(a, b, -c);
  const double t = sum + y;
  c = (t - sum) - y;
  sum = t;
}

// The same for K double-doubles (hi[e] + lo_in[e]); hi[e] receives the sum
// rounded to a double.  TwoSum's error term does not depend on the operand
// order, so all lanes end with the same bits.
template <int K, int SP, int FROM>
__device__ __forceinline__ void freq_sum_dd_n(double *hi, const double *lo_in, int s_lanes) {
  double lo[K];
#pragma unroll
  for (int e = 0; e < K; ++e) lo[e] = lo_in[e];
  each_bit<SP, FROM>(s_lanes, [&](auto mask) {
#pragma unroll
    for (int e = 0; e < K; ++e) {
      const Two h = with_lane_xor<decltype(mask)::value>(hi[e]), l = with_lane_xor<decltype(mask)::value>(lo[e]);
      const double s = h.a + h.b;
      const double bv = s - h.a;
      const double se = (h.a - (s - bv)) + (h.b - bv);
      hi[e] = s;
      lo[e] = (l.a + l.b) + se;
    }
  });
#pragma unroll
  for (int e = 0; e < K; ++e) hi[e] = hi[e] + lo[e];
}

// --------------------------------------------------------------------------
// Double-double arithmetic for the extended-precision refinement
// (FLAG_DD_REFINE).  A value is an unevaluated sum h + l.  TwoSum (Knuth)
// gives the rounding error of a sum and the fused multiply-add that of a
// product exactly, so sums and products of such pairs keep about 104 bits.
// Contraction is switched off in these routines: a product that the compiler
// fused into a later sum would no longer be the rounded product whose error
// the next operation recovers.
// --------------------------------------------------------------------------
struct ddv {
  double h, l;
};
__device__ __forceinline__ ddv two_sum(double a, double b) {
#pragma clang fp contract(off)
  const double s = a + b, bb = s - a;
  return {s, (a - (s - bb)) + (b - bb)};
}
// valid when |a| >= |b| (or a == 0)
__device__ __forceinline__ ddv quick_two_sum(double a, double b) {
#pragma clang fp contract(off)
  const double s = a + b;
  return {s, b - (s - a)};
}
__device__ __forceinline__ ddv dd_mul(ddv a, ddv b) {
#pragma clang fp contract(off)
  const double p = a.h * b.h;
  const double e = __builtin_fma(a.h, b.l, __builtin_fma(a.l, b.h, __builtin_fma(a.h, b.h, -p)));
  return quick_two_sum(p, e);
}
// sum of two pairs whose high parts do not cancel
__device__ __forceinline__ ddv dd_add(ddv a, ddv b) {
#pragma clang fp contract(off)
  const ddv s = two_sum(a.h, b.h);
  return quick_two_sum(s.h, s.l + (a.l + b.l));
}

// 10^t as a double-double, for |t| <= 30 (relative error near 2^-95).  The
// double nearest 10^t is off by up to half an ulp, which moves the weights
// of an ill-conditioned fit, and with them its cost, by more than the cost's
// tolerance; the extended-precision refinement needs the relaxation times
// to its own precision.  Steps: y = t ln 10 in double-double; y = n ln 2 + r
// with n = rint(y / ln 2), |r| <= ln 2 / 2; e^r = (e^(r/256))^256, the inner
// factor from its Taylor series to degree 9 (the first omitted term is below
// 2^-117), the power by eight squarings; then the scale 2^n.
__device__ __noinline__ ddv exp10_dd(double t) {
#pragma clang fp contract(off)
  constexpr double LN10_H = 0x1.26bb1bbb55516p+1, LN10_L = -0x1.f48ad494ea3e9p-53;
  constexpr double LN2_H = 0x1.62e42fefa39efp-1, LN2_L = 0x1.abc9e3b39803fp-56;
  const double yh = t * LN10_H;
  const double yl = __builtin_fma(t, LN10_L, __builtin_fma(t, LN10_H, -yh));
  const double n = rint(yh / LN2_H);
  // r = y - n ln 2: n * LN2_H and its rounding error exactly, then the rest
  const double ph = n * LN2_H;
  const double pe = __builtin_fma(n, LN2_H, -ph);
  ddv r = two_sum(yh, -ph);
  r = quick_two_sum(r.h, r.l + ((yl - pe) - n * LN2_L));
  r.h = ldexp(r.h, -8);
  r.l = ldexp(r.l, -8);
  // 1 + r (1 + r/2 (1 + r/3 ( ... (1 + r/9))))
  ddv p = {1.0, 0.0};
  for (int j = 9; j >= 1; --j) {
    const double dj = (double)j;
    const double qh = r.h / dj;
    const double ql = (__builtin_fma(-qh, dj, r.h) + r.l) / dj;   // the remainder r.h - qh j is exact
    p = dd_add({1.0, 0.0}, dd_mul({qh, ql}, p));
  }
  for (int s = 0; s < 8; ++s) p = dd_mul(p, p);
  const int e = (int)n;
  return {ldexp(p.h, e), ldexp(p.l, e)};
}

// The Debye basis term I = x / (1 + x^2), x = w tau, as a double-double from
// tau = th + tl: x by TwoProduct, x^2 likewise (its cross term 2 xh xl added
// to the error), 1 + x^2 by TwoSum, R = 1 / (1 + x^2) from a reciprocal of
// the high part within half an ulp and one correction r (1 + e), e = 1 - d r
// formed with fused operations, then I = x R.
__device__ __forceinline__ ddv dd_debye_I(double w, double th, double tl) {
#pragma clang fp contract(off)
  const double xh = w * th;
  const double xl = __builtin_fma(w, tl, __builtin_fma(w, th, -xh));
  const double qh = xh * xh;
  const double ql = __builtin_fma(xh + xh, xl, __builtin_fma(xh, xh, -qh));
  const ddv d = two_sum(1.0, qh);
  const double dl = d.l + ql;
  const double r = rcp_nr(d.h);
  const double rl = r * __builtin_fma(-dl, r, __builtin_fma(-d.h, r, 1.0));
  const double ih = xh * r;
  return {ih, __builtin_fma(xh, rl, __builtin_fma(xl, r, __builtin_fma(xh, r, -ih)))};
}

// --------------------------------------------------------------------------
// Debye basis of the owned poles at one frequency: R = 1/(1+x^2), I = x R.
// Every pass needs only R: with I = w tau R, the factor tau moves out of
// every frequency sum (applied once per candidate) and w out of every pole
// sum (applied once per point), and 1 + x^2 is 1 + w^2 tau^2 with w^2 shared
// by the poles and tau^2 by the points (the rounding of d is the same as
// through x = w tau: one product rounded, then a fused add).  Padded poles
// have tau = 0: R = 1, and their I columns vanish through tau.
//
// Paired form (basis_R): two poles share one reciprocal, r = 1/(d0 d1),
// R0 = d1 r, R1 = d0 r (within a few ulp).  With |log10 tau| <= 30 (larger
// values are rejected as bad input) and w < 1e45 rad/s, x < 1e75 and the
// product d0 d1 < 1e301 cannot overflow.
// --------------------------------------------------------------------------
template <int NB>
__device__ __forceinline__ void basis_R(double w2, const double *tau2, double *R) {
#pragma unroll
  for (int c = 0; c + 1 < NB; c += 2) {
    const double d0 = __builtin_fma(w2, tau2[c], 1.0), d1 = __builtin_fma(w2, tau2[c + 1], 1.0);
    const double r = rcp_nr(d0 * d1);
    R[c] = d1 * r;
    R[c + 1] = d0 * r;
  }
  if constexpr (NB & 1) R[NB - 1] = rcp_nr(__builtin_fma(w2, tau2[NB - 1], 1.0));
}

// Grouped form (the frequency passes of the cost): four poles share one
// reciprocal, r = 1/(p01 p23) with p01 = d0 d1, p23 = d2 d3, and
// 1/d0 = d1 (r p23), 1/d1 = d0 (r p23), 1/d2 = d3 (r p01), 1/d3 = d2 (r p01):
// three products and one reciprocal per four poles in place of two
// reciprocals (a reciprocal occupies the FP64 pipe for four issue cycles and
// its Newton step for three more).  Three poles beyond the last full group
// form a group too (r = 1/(p01 d2), 1/d0 = d1 (r d2), 1/d1 = d0 (r d2), 1/d2 =
// p01 r: one reciprocal in place of a pair's and a single pole's; 256
// materials, F = 2,000: 128 candidates of N = 7 448 -> 434 us, 256 of N = 13
// 1,889 -> 1,864, of N = 14 1,779 -> 1,753; not for the 11 poles of one lane,
// whose forward kernel spills more with it, 670 -> 679 us); one or two are
// taken as above.
//
// The product of four d can leave the double range (each d < 1e150), so a
// group works on d scaled by a power of two s, fixed from the bound
// w < 1e45: s^4 prod d(1e45) <= 2^990 and s >= 2^-253, so every intermediate
// product lies in [2^-1012, 2^990] at every admissible frequency and every
// reciprocal is a normal number.  With tau^2 s in place of tau^2 and s in
// place of 1, every intermediate is the unscaled value times an exact power
// of two (the same roundings, barring underflow of tiny products, which the
// scaled form suffers less); the group's basis values come out divided by
// s, and s is applied with tau after the frequency sums (a group of three, d0
// d1 d2 < 1e450, the same with s^3 and s >= 2^-169).  Any smaller s of
// the same form down to 2^-253 keeps these bounds, so a wave takes, per
// group index, the smallest s of its lanes: s is then wave-uniform and the
// fused add reads it from a scalar register (a third vector operand of a
// 64-bit FMA costs issue bandwidth), and each lane's results do not depend
// on the other lanes of its wave.
// --------------------------------------------------------------------------
constexpr double OMEGA_BOUND = 1e45;   // admissible angular frequencies: 0 < w < OMEGA_BOUND

template <int NB> struct Groups {
  static constexpr int NQ = NB / 4;              // groups of four owned poles
  static constexpr bool THREE = NB % 4 == 3 && NB < 11;   // and one of three
  static constexpr int NG = NQ + THREE;
  static constexpr int NS = NG > 0 ? NG : 1;     // (array size)
  static constexpr int POLES = 4 * NQ + 3 * THREE;
};

// the largest k >= 0 of the wave (shifts and broadcasts over the rows of 16
// lanes leave it in the last lane)
__device__ __forceinline__ int wave_max(int k) {
  auto step = [&](int o) { k = o > k ? o : k; };
  step(__builtin_amdgcn_update_dpp(0, k, 0x111, 0xF, 0xF, false));   // row_shr:1
  step(__builtin_amdgcn_update_dpp(0, k, 0x112, 0xF, 0xF, false));   // row_shr:2
  step(__builtin_amdgcn_update_dpp(0, k, 0x114, 0xF, 0xF, false));   // row_shr:4
  step(__builtin_amdgcn_update_dpp(0, k, 0x118, 0xF, 0xF, false));   // row_shr:8
  step(__builtin_amdgcn_update_dpp(0, k, 0x142, 0xA, 0xF, false));   // row_bcast:15 into rows 1 and 3
  step(__builtin_amdgcn_update_dpp(0, k, 0x143, 0xC, 0xF, false));   // row_bcast:31 into rows 2 and 3
  return __builtin_amdgcn_readlane(k, WAVE - 1);
}

// scale s = 2^-k of each group (from tau^2 of its poles), the same in every
// lane of the wave (all lanes call this together)
template <int NB>
__device__ __forceinline__ void group_scales(const double *tau2, int *kq, double *sq) {
  kq[0] = 0;
  sq[0] = 1.0;
#pragma unroll
  for (int g = 0; g < Groups<NB>::NG; ++g) {
    const int n = g < Groups<NB>::NQ ? 4 : 3;
    int e = 0;   // sum of the binary exponents: prod d(1e45) < 2^e
#pragma unroll
    for (int t = 0; t < n; ++t)
      e += __builtin_amdgcn_frexp_exp(__builtin_fma(OMEGA_BOUND * OMEGA_BOUND, tau2[4 * g + t], 1.0));
    int k = e > 990 ? (e - 990 + n - 1) / n : 0;
    // |log10 tau| <= 30 gives e <= 1996, k <= 252; the cap keeps a lane with
    // rejected input (its results are discarded) from scaling its wave's
    // valid lanes out of range
    k = k < 253 ? k : 253;
    k = wave_max(k);
    kq[g] = k;
    sq[g] = __hiloint2double((1023 - k) << 20, 0);   // 2^-k
  }
}

// scale of owned pole i (1 outside the groups)
template <int NB> __device__ __forceinline__ double pole_scale(const double *sq, int i) {
  return i < Groups<NB>::POLES ? sq[i / 4] : 1.0;
}

// x * 2^(+-k) of owned pole i's group (exact)
template <int NB> __device__ __forceinline__ double group_unscale(const int *kq, int i, double x) {
  return i < Groups<NB>::POLES ? __builtin_amdgcn_ldexp(x, kq[i / 4]) : x;
}
template <int NB> __device__ __forceinline__ double group_scale(const int *kq, int i, double x) {
  return i < Groups<NB>::POLES ? __builtin_amdgcn_ldexp(x, -kq[i / 4]) : x;
}

// R / s of the owned poles (tau2s = tau^2 s)
template <int NB>
__device__ __forceinline__ void basis_Rs(double w2, const double *tau2s, const double *sq, double *R) {
#pragma unroll
  for (int g = 0; g < Groups<NB>::NQ; ++g) {
    const int c = 4 * g;
    const double d0 = __builtin_fma(w2, tau2s[c], sq[g]), d1 = __builtin_fma(w2, tau2s[c + 1], sq[g]);
    const double d2 = __builtin_fma(w2, tau2s[c + 2], sq[g]), d3 = __builtin_fma(w2, tau2s[c + 3], sq[g]);
    const double p01 = d0 * d1, p23 = d2 * d3;
    const double r = rcp_nr(p01 * p23);
    const double r01 = r * p23, r23 = r * p01;
    R[c] = d1 * r01;
    R[c + 1] = d0 * r01;
    R[c + 2] = d3 * r23;
    R[c + 3] = d2 * r23;
  }
  constexpr int C = 4 * Groups<NB>::NQ;
  if constexpr (Groups<NB>::THREE) {
    const double s = sq[Groups<NB>::NQ];
    const double d0 = __builtin_fma(w2, tau2s[C], s), d1 = __builtin_fma(w2, tau2s[C + 1], s);
    const double d2 = __builtin_fma(w2, tau2s[C + 2], s), p01 = d0 * d1;
    const double r = rcp_nr(p01 * d2), r01 = r * d2;
    R[C] = d1 * r01;
    R[C + 1] = d0 * r01;
    R[C + 2] = p01 * r;
  } else {
    basis_R<NB - C>(w2, tau2s + C, R + C);
  }
}

// U / s with U = w R directly (the Gram pass needs no R): the factor w enters
// after the group's reciprocal is split, U0 = d1 (w (r p23)), ... (r p23 =
// 1/p01 <= 2^506, so no intermediate overflows even where the wave's scale is
// far below the lane's own and r is near 2^1012), and once per pair for the
// paired poles (U0 = d1 (w r)).
template <int NB>
__device__ __forceinline__ void basis_Us(double w, double w2, const double *tau2s, const double *sq, double *U) {
#pragma unroll
  for (int g = 0; g < Groups<NB>::NQ; ++g) {
    const int c = 4 * g;
    const double d0 = __builtin_fma(w2, tau2s[c], sq[g]), d1 = __builtin_fma(w2, tau2s[c + 1], sq[g]);
    const double d2 = __builtin_fma(w2, tau2s[c + 2], sq[g]), d3 = __builtin_fma(w2, tau2s[c + 3], sq[g]);
    const double p01 = d0 * d1, p23 = d2 * d3;
    const double r = rcp_nr(p01 * p23);
    const double r01 = w * (r * p23), r23 = w * (r * p01);
    U[c] = d1 * r01;
    U[c + 1] = d0 * r01;
    U[c + 2] = d3 * r23;
    U[c + 3] = d2 * r23;
  }
  constexpr int C = 4 * Groups<NB>::NQ;
  if constexpr (Groups<NB>::THREE) {
    const double s = sq[Groups<NB>::NQ];
    const double d0 = __builtin_fma(w2, tau2s[C], s), d1 = __builtin_fma(w2, tau2s[C + 1], s);
    const double d2 = __builtin_fma(w2, tau2s[C + 2], s), p01 = d0 * d1;
    // (r <= 2^759 at the wave's smallest scale, so w r cannot overflow)
    const double rw = w * rcp_nr(p01 * d2), r01 = rw * d2;
    U[C] = d1 * r01;
    U[C + 1] = d0 * r01;
    U[C + 2] = p01 * rw;
    return;
  }
#pragma unroll
  for (int c = C; c + 1 < NB; c += 2) {
    const double d0 = __builtin_fma(w2, tau2s[c], 1.0), d1 = __builtin_fma(w2, tau2s[c + 1], 1.0);
    const double rw = w * rcp_nr(d0 * d1);
    U[c] = d1 * rw;
    U[c + 1] = d0 * rw;
  }
  if constexpr ((NB - C) & 1) U[NB - 1] = w * rcp_nr(__builtin_fma(w2, tau2s[NB - 1], 1.0));
}

// Owned poles left over after the groups and the pairs: one (the last) or none.
template <int NB> constexpr bool odd_pole() { return ((NB - Groups<NB>::POLES) & 1) != 0; }

// The basis at two points a and b (w2 = w^2).  With an odd last pole, that
// pole's two values share one reciprocal, r = 1/(d_a d_b), R_a = d_b r,
// R_b = d_a r, as two poles of one point do (the odd pole lies outside the
// groups, so d <= 1e150 and d_a d_b cannot overflow); the other poles as in
// basis_Rs / basis_Us at each point.
template <int NB>
__device__ __forceinline__ void basis_Rs2(double w2a, double w2b, const double *tau2s, const double *sq, double *Ra,
                                          double *Rb) {
  if constexpr (odd_pole<NB>()) {
    basis_Rs<NB - 1>(w2a, tau2s, sq, Ra);
    basis_Rs<NB - 1>(w2b, tau2s, sq, Rb);
    const double da = __builtin_fma(w2a, tau2s[NB - 1], 1.0), db = __builtin_fma(w2b, tau2s[NB - 1], 1.0);
    const double r = rcp_nr(da * db);
    Ra[NB - 1] = db * r;
    Rb[NB - 1] = da * r;
  } else {
    basis_Rs<NB>(w2a, tau2s, sq, Ra);
    basis_Rs<NB>(w2b, tau2s, sq, Rb);
  }
}
template <int NB>
__device__ __forceinline__ void basis_Us2(double wa, double wb, const double *tau2s, const double *sq, double *Ua,
                                          double *Ub) {
  if constexpr (odd_pole<NB>()) {
    basis_Us<NB - 1>(wa, wa * wa, tau2s, sq, Ua);
    basis_Us<NB - 1>(wb, wb * wb, tau2s, sq, Ub);
    const double da = __builtin_fma(wa * wa, tau2s[NB - 1], 1.0), db = __builtin_fma(wb * wb, tau2s[NB - 1], 1.0);
    const double r = rcp_nr(da * db);
    Ua[NB - 1] = wa * (db * r);
    Ub[NB - 1] = wb * (da * r);
  } else {
    basis_Us<NB>(wa, wa * wa, tau2s, sq, Ua);
    basis_Us<NB>(wb, wb * wb, tau2s, sq, Ub);
  }
}

// R / s of the poles of two owner lanes (a half-candidate of the four-lane
// split, a whole candidate of the two-lane split): each owner's NQ groups of
// four at the wave's group scales (t2[0 .. 8 NQ), owner A's groups then
// owner B's, tau^2 s), then their LO leftover poles each (t2[8 NQ ..), tau^2,
// unscaled, so that d <= 1e150) in pairs sharing a reciprocal.
template <int NQ, int LO>
__device__ __forceinline__ void basis_two_owners(double w2, const double *t2, const double *sq, double *R) {
#pragma unroll
  for (int c = 0; c < 8 * NQ; c += 4) {
    const double s = sq[(c / 4) % NQ];
    const double d0 = __builtin_fma(w2, t2[c], s), d1 = __builtin_fma(w2, t2[c + 1], s);
    const double d2 = __builtin_fma(w2, t2[c + 2], s), d3 = __builtin_fma(w2, t2[c + 3], s);
    const double p01 = d0 * d1, p23 = d2 * d3;
    const double r = rcp_nr(p01 * p23);
    const double r01 = r * p23, r23 = r * p01;
    R[c] = d1 * r01;
    R[c + 1] = d0 * r01;
    R[c + 2] = d3 * r23;
    R[c + 3] = d2 * r23;
  }
#pragma unroll
  for (int c = 8 * NQ; c < 8 * NQ + 2 * LO; c += 2) {
    const double d0 = __builtin_fma(w2, t2[c], 1.0), d1 = __builtin_fma(w2, t2[c + 1], 1.0);
    const double r = rcp_nr(d0 * d1);
    R[c] = d1 * r;
    R[c + 1] = d0 * r;
  }
}

// --------------------------------------------------------------------------
// Dense solve helpers on a packed upper triangle held in registers (SP == 1)
// or in LDS (SP > 1).  A = U^T U, U upper, diagonal stored as reciprocals in uinv.
// --------------------------------------------------------------------------
template <int N, class MAT>
__device__ __forceinline__ bool equilibrate_factor(MAT &A, double *invd, double *uinv, double damping,
                                                   double tol) {
  bool ok = true;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    double g = A[tri(N, i, i)];
    ok = ok && (g > 0.0) && (g < INFINITY);
    invd[i] = rsq_nr(g);
  }
#pragma unroll
  for (int i = 0; i < N; ++i) {
#pragma unroll
    for (int j = i + 1; j < N; ++j) A[tri(N, i, j)] = A[tri(N, i, j)] * invd[i] * invd[j];
    A[tri(N, i, i)] = 1.0 + damping;
  }
#pragma unroll
  for (int j = 0; j < N; ++j) {
    double s = A[tri(N, j, j)];
#pragma unroll
    for (int l = 0; l < j; ++l) s = __builtin_fma(-A[tri(N, l, j)], A[tri(N, l, j)], s);
    ok = ok && (s > tol);
    const double ui = rsq_nr(s);   // (the pivot itself is never read)
    uinv[j] = ui;
#pragma unroll
    for (int k = j + 1; k < N; ++k) {
      double t = A[tri(N, j, k)];
#pragma unroll
      for (int l = 0; l < j; ++l) t = __builtin_fma(-A[tri(N, l, j)], A[tri(N, l, k)], t);
      A[tri(N, j, k)] = t * ui;
    }
  }
  return ok;
}

// x <- A^-1 x with A = U^T U (x overwritten)
template <int N, class MAT, class VEC>
__device__ __forceinline__ void chol_solve(const MAT &A, const double *uinv, VEC &x) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    double s = x[i];
#pragma unroll
    for (int l = 0; l < i; ++l) s = __builtin_fma(-A[tri(N, l, i)], x[l], s);
    x[i] = s * uinv[i];
  }
#pragma unroll
  for (int i = N - 1; i >= 0; --i) {
    double s = x[i];
#pragma unroll
    for (int l = i + 1; l < N; ++l) s = __builtin_fma(-A[tri(N, i, l)], x[l], s);
    x[i] = s * uinv[i];
  }
}

// The same factorisation and solves for a matrix in LDS (SP > 1).  Every
// lane of a candidate runs them on that candidate's region.  The pointers are
// typed as LDS (address space 3): through a generic pointer the calls would
// read with flat loads, whose latency each step of these serial recurrences
// waits for.  The upper triangle is packed by columns (element (i, j), i <= j,
// at j (j + 1) / 2 + i), so that every inner sum of the factorisation and of
// the forward solve reads consecutive elements: one base address and
// immediate offsets, no per-term address arithmetic.  Those sums are unrolled
// by four (their loads issued together, the additions in their order); the
// backward solve is unrolled whole (all its addresses are constants).  The
// operations and their order are those of the register form above.

constexpr __host__ __device__ int tcol(int i, int j) { return j * (j + 1) / 2 + i; }

template <int N>
__device__ __noinline__ bool lds_equilibrate_factor(lds_ptr A, lds_ptr invd, lds_ptr uinv, double damping,
                                                    double tol) {
  bool ok = true;
  double dv[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const double g = A[tcol(i, i)];
    ok = ok && (g > 0.0) && (g < INFINITY);
    dv[i] = rsq_nr(g);
    invd[i] = dv[i];
  }
#pragma unroll
  for (int j = 0; j < N; ++j) {
#pragma unroll
    for (int i = 0; i < j; ++i) A[tcol(i, j)] = A[tcol(i, j)] * dv[i] * dv[j];
    A[tcol(j, j)] = 1.0 + damping;
  }
  for (int j = 0; j < N; ++j) {
    const lds_ptr cj = A + tcol(0, j);
    double s = cj[j];
#pragma unroll 4
    for (int l = 0; l < j; ++l) s = __builtin_fma(-cj[l], cj[l], s);
    ok = ok && (s > tol);
    const double ui = rsq_nr(s);   // (the pivot itself is never read)
    uinv[j] = ui;
    for (int k = j + 1; k < N; ++k) {
      const lds_ptr ck = A + tcol(0, k);
      double t = ck[j];
#pragma unroll 4
      for (int l = 0; l < j; ++l) t = __builtin_fma(-cj[l], ck[l], t);
      ck[j] = t * ui;
    }
  }
  return ok;
}

template <int N> __device__ __noinline__ void lds_chol_solve(lds_cptr A, lds_cptr uinv, lds_ptr x) {
  double xv[N];
  for (int i = 0; i < N; ++i) {
    const lds_cptr ci = A + tcol(0, i);
    double s = x[i];
#pragma unroll 4
    for (int l = 0; l < i; ++l) s = __builtin_fma(-ci[l], x[l], s);
    x[i] = s * uinv[i];
  }
#pragma unroll
  for (int i = 0; i < N; ++i) xv[i] = x[i];
#pragma unroll
  for (int i = N - 1; i >= 0; --i) {
    double s = xv[i];
#pragma unroll
    for (int l = i + 1; l < N; ++l) s = __builtin_fma(-A[tcol(i, l)], xv[l], s);
    xv[i] = s * uinv[i];
    x[i] = xv[i];
  }
}

// The factorisation and the solves shared by 16 lanes of a candidate (the
// four-lane split, whose candidates hold 16, 32 or 64 lanes; lanes with the
// same c do the same work).  Lane c has rows and columns c and c + 16 of the
// matrix and elements c and c + 16 of the vectors; a lane without one takes
// the last.  With every lane running the whole factorisation, its N^3 / 6
// fused multiply-adds and their operands' LDS reads took as long as 200 points
// of the frequency passes at N = 20.
template <int N> struct Coop {
  static constexpr int N0 = N < 16 ? N : 16, N1 = N > 16 ? N : 0;   // rows of the first and second column
  static constexpr int NX = N1 > 0 ? N1 : 1;
  lds_ptr A, uinv;
  int k0, k1, src;   // own elements; byte address of the candidate's first lane for ds_bpermute
  __device__ __forceinline__ Coop(lds_ptr A_, lds_ptr uinv_, int c, int first_lane)
      : A(A_), uinv(uinv_), k0(c < N ? c : N - 1), k1(c + 16 < N ? c + 16 : N - 1), src(first_lane * 4) {}

  // lane c's value in all lanes of the candidate
  __device__ __forceinline__ double from(double v, int c) const {
    // (the address is formed at each use: 16 of them kept in registers across
    // the refinement pass would spill)
    int at = src;
    asm volatile("" : "+v"(at));
    at += 4 * ((c & 3) + ((c >> 2) << 4));
    return __hiloint2double(__builtin_amdgcn_ds_bpermute(at, __double2hiint(v)),
                            __builtin_amdgcn_ds_bpermute(at, __double2loint(v)));
  }

  // Equilibrates the packed triangle A (its diagonal becomes 1 + damping),
  // factors it A = U^T U in place (off-diagonal; reciprocal pivots to uinv)
  // and takes x <- U^-T D^-1 b along.  Step j: every lane posts its row-j
  // entries, reads the row back, and takes the outer product off its columns,
  // a_ik -= a_ji (a_jk / a_jj): a serial chain of N LDS round trips.
  __device__ __forceinline__ bool factor(lds_cptr b, lds_ptr invd, lds_ptr rowbuf, lds_ptr xbuf, double damping,
                                         double tol, double &x0, double &x1) const {
    double c0[N0], c1[NX];
    // own columns (entries below the diagonal are other columns', never used)
#pragma unroll
    for (int i = 0; i < N0; ++i) c0[i] = A[tcol(0, k0) + i];
#pragma unroll
    for (int i = 0; i < N1; ++i) c1[i] = A[tcol(0, k1) + i];
    const double d0 = rsq_nr(A[tcol(k0, k0)]);
    invd[k0] = d0;
    x0 = b[k0] * d0;
    double d1 = 0.0;
    x1 = 0.0;
    if constexpr (N1 > 0) {
      d1 = rsq_nr(A[tcol(k1, k1)]);
      invd[k1] = d1;
      x1 = b[k1] * d1;
    }
    wave_sync();
    bool ok = true;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const double di = invd[i];
      ok = ok && di > 0.0 && di < INFINITY;   // 0 < g_ii < inf
      if (i < N0) c0[i] = k0 == i ? 1.0 + damping : c0[i] * di * d0;
      if (i < N1) c1[i] = k1 == i ? 1.0 + damping : c1[i] * di * d1;
    }
#pragma unroll
    for (int j = 0; j < N; ++j) {
      if (j < N0) {
        rowbuf[k0] = c0[j];
        xbuf[k0] = x0;
      }
      if (j < N1) {
        rowbuf[k1] = c1[j];
        xbuf[k1] = x1;
      }
      wave_sync();
      double r[N];
#pragma unroll
      for (int i = j; i < N; ++i) r[i] = rowbuf[i];
      const double xj = xbuf[j];
      wave_sync();
      ok = ok && r[j] > tol;
      const double ri = rcp_nr(r[j]), ui = rsq_nr(r[j]);
      uinv[j] = ui;
      if (j < N0) {
        const double v = c0[j] * ri, u = c0[j] * ui;
        if (k0 > j) {
          A[tcol(0, k0) + j] = u;
          x0 = __builtin_fma(-v, xj, x0);
        }
#pragma unroll
        for (int i = j + 1; i < N0; ++i) c0[i] = __builtin_fma(-r[i], v, c0[i]);
      }
      if (j < N1) {
        const double v = c1[j] * ri, u = c1[j] * ui;
        if (k1 > j) {
          A[tcol(0, k1) + j] = u;
          x1 = __builtin_fma(-v, xj, x1);
        }
#pragma unroll
        for (int i = j + 1; i < N1; ++i) c1[i] = __builtin_fma(-r[i], v, c1[i]);
      }
    }
    wave_sync();
    x0 *= uinv[k0];
    if constexpr (N1 > 0) x1 *= uinv[k1];
    return ok;
  }

  // x <- U^-T x
  __device__ __forceinline__ void forward(double &x0, double &x1) const {
    const double u0 = uinv[k0], u1 = N1 > 0 ? uinv[k1] : 0.0;
    double c0[N0], c1[NX];   // own columns above the diagonal
#pragma unroll
    for (int l = 0; l < N0; ++l) c0[l] = l < k0 ? A[tcol(0, k0) + l] : 0.0;
#pragma unroll
    for (int l = 0; l < N1; ++l) c1[l] = l < k1 ? A[tcol(0, k1) + l] : 0.0;
#pragma unroll
    for (int l = 0; l < N - 1; ++l) {
      const double y = from(l < 16 ? x0 * u0 : x1 * u1, l & 15);
      if (l < N0) x0 = __builtin_fma(-c0[l], y, x0);
      if (l < N1) x1 = __builtin_fma(-c1[l], y, x1);
    }
    x0 *= u0;
    if constexpr (N1 > 0) x1 *= u1;
  }

  // x <- U^-1 x
  __device__ __forceinline__ void backward(double &x0, double &x1) const {
    const double u0 = uinv[k0], u1 = N1 > 0 ? uinv[k1] : 0.0;
    double r0[N], r1[N];   // own rows right of the diagonal
#pragma unroll
    for (int k = 1; k < N; ++k) r0[k] = k > k0 ? A[tcol(k0, k)] : 0.0;
#pragma unroll
    for (int k = 17; k < N; ++k) r1[k] = k > k1 ? A[tcol(k1, k)] : 0.0;
#pragma unroll
    for (int k = N - 1; k > 0; --k) {
      const double z = from(k < 16 ? x0 * u0 : x1 * u1, k & 15);
      x0 = __builtin_fma(-r0[k], z, x0);
      if (k > 16) x1 = __builtin_fma(-r1[k], z, x1);
    }
    x0 *= u0;
    if constexpr (N1 > 0) x1 *= u1;
  }

  // the lane's elements of a vector in LDS
  __device__ __forceinline__ void get(lds_cptr v, double &x0, double &x1) const {
    x0 = v[k0];
    x1 = N1 > 0 ? v[k1] : 0.0;
  }
  __device__ __forceinline__ void put(lds_ptr v, double x0, double x1) const {
    v[k0] = x0;
    if constexpr (N1 > 0) v[k1] = x1;
  }
};

// per-candidate LDS region of the SP > 1 path: packed triangle, then five
// vectors of N (scaling, reciprocal pivots, rhs, two work vectors); on the
// four-lane split a sixth (tau s)
template <int N> struct LdsLayout {
  static constexpr int NT = N * (N + 1) / 2;
  double *A, *invd, *uinv, *vb, *vz, *vw, *vt;
  __device__ __forceinline__ explicit LdsLayout(double *base)
      : A(base), invd(base + NT), uinv(base + NT + N), vb(base + NT + 2 * N), vz(base + NT + 3 * N),
        vw(base + NT + 4 * N), vt(base + NT + 5 * N) {}
};

// factor parked by the SP == 1 path: A (off-diagonal) and reciprocal pivots
template <int N>
__device__ __forceinline__ void unpark(const double *park, int cpw, int grp, double *A, double *uinv) {
#pragma unroll
  for (int i = 0; i < N; ++i)
#pragma unroll
    for (int j = i; j < N; ++j) {
      const double v = park[tri(N, i, j) * cpw + grp];
      if (i == j) uinv[i] = v;
      else A[tri(N, i, j)] = v;
    }
}

// --------------------------------------------------------------------------
// Reading a spectrum.  A lane takes points k0, k0 + stride, ... of its
// candidate's spectrum, in every pass; the passes that read one point ahead
// use the loops below.
// --------------------------------------------------------------------------
// How (WALK): 0, a lane's own 64-bit index; 1, the same, wave-uniform (split 1:
// scalar loads); 2, a wave-uniform point and a lane's own constant offset; 3,
// a lane's own index into LDS.
// point k
template <int WALK> __device__ __forceinline__ double ld(const double *p, int64_t k) {
  if constexpr (WALK == 3) return ((lds_cptr)p)[k];
  else if constexpr (WALK == 2) return *(const double *)((const char *)p + ((uint32_t)k << 3));
  else return p[k];
}
// The first point of a pass that reads one point ahead, through the constant
// address space (the spectra are read-only during a launch).  Loads from two
// address spaces are not merged, so the compiler keeps the loop's loads one
// point ahead instead of folding them with this one into a single load at the
// top of every trip (which would expose the load latency at each point).
template <int WALK> __device__ __forceinline__ double ld_first(const double *p, int64_t k) {
  using cptr = const __attribute__((address_space(4))) double *;
  if constexpr (WALK == 3) return ((lds_cptr)p)[k];
  else if constexpr (WALK == 2) return *(cptr)((const char *)p + ((uint32_t)k << 3));
  else return ((cptr)p)[k];
}
// Uniform tiles with a frequency split: the wave's lanes walk together, so a
// point is a spectrum's base (a buffer descriptor), a wave-uniform byte offset
// kept by the scalar unit, and a lane's own offset, which never changes: no
// vector instruction forms an address.  (A lane's own index, clamped to stay
// in bounds one trip ahead, and its 64-bit addresses took 9 of the 78 vector
// instructions of a pair of points in the Gram pass at N = 20, and 8 of 86 in
// the cost pass at N = 8.)
struct Reader {
  __amdgpu_buffer_rsrc_t r;
  uint32_t lane;   // the lane's byte offset
  __device__ __forceinline__ Reader(const double *p, int64_t F, int64_t k0)
      : r(__builtin_amdgcn_make_buffer_rsrc((void *)p, 0, (int)(uint32_t)(F << 3), 0x00027000)),
        lane((uint32_t)k0 << 3) {}
  // the lane's point of the trip at point u
  __device__ __forceinline__ double operator()(int32_t u) const {
    return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, (int)lane, (int)((uint32_t)u << 3), 0));
  }
};

struct Spectrum {
  const double *om, *er, *ei;
  int64_t F;
};

// body(w, eps', eps'') at points k0, k0 + stride, ... (k0 < stride)
template <int WALK, int UNROLL, class BODY>
__device__ __forceinline__ void each_point(const Spectrum &sp, int k0, int stride, BODY &&body) {
  const int64_t F = sp.F;
  int64_t k = k0;
  if constexpr (WALK == 2) {
    const int32_t n = (int32_t)F & ~(stride - 1);   // points of the trips every lane takes
    const Reader om(sp.om, F, k0), er_(sp.er, F, k0), ei_(sp.ei, F, k0);
    if (n > 0) {
      double w_n = ld_first<WALK>(sp.om, k0), er_n = ld_first<WALK>(sp.er, k0), ei_n = ld_first<WALK>(sp.ei, k0);
#pragma unroll UNROLL
      for (int32_t u = 0; u < n; u += stride) {
        const double w = w_n, er = er_n, ei = ei_n;
        const int32_t un = u + stride < n ? u + stride : u;   // in-bounds prefetch, no branch
        w_n = om(un);
        er_n = er_(un);
        ei_n = ei_(un);
        body(w, er, ei);
      }
    }
    k += n;
    if (k < F) body(ld<WALK>(sp.om, k), ld<WALK>(sp.er, k), ld<WALK>(sp.ei, k));
  } else {
    double w_n = 0, er_n = 0, ei_n = 0;
    if (k < F) {
      w_n = ld_first<WALK>(sp.om, k);
      er_n = ld_first<WALK>(sp.er, k);
      ei_n = ld_first<WALK>(sp.ei, k);
    }
#pragma unroll UNROLL
    for (; k < F; k += stride) {
      const double w = w_n, er = er_n, ei = ei_n;
      const int64_t kn = (k + stride < F) ? k + stride : k;   // in-bounds prefetch, no branch
      w_n = ld<WALK>(sp.om, kn);
      er_n = ld<WALK>(sp.er, kn);
      ei_n = ld<WALK>(sp.ei, kn);
      body(w, er, ei);
    }
  }
}

// body(a, b), a and b points (w, eps', eps''), for n_pairs pairs of points
// k0 + 2 t stride and k0 + (2 t + 1) stride that every lane has (n_pairs is
// wave-uniform); returns the index of the lane's next point
struct Point {
  double w, er, ei;
};
template <int WALK, class BODY>
__device__ __forceinline__ int64_t each_pair(const Spectrum &sp, int k0, int stride, int64_t n_pairs, BODY &&body) {
  int64_t k = k0;
  if (n_pairs <= 0) return k;
  if constexpr (WALK == 2) {
    const Reader om(sp.om, sp.F, k0), er(sp.er, sp.F, k0), ei(sp.ei, sp.F, k0);
    const int32_t n = 2 * stride * (int32_t)n_pairs;
    auto read = [&](int32_t u, Point &a, Point &b) {
      u = u < n ? u : n - 2 * stride;   // in-bounds prefetch, no branch
      a = {om(u), er(u), ei(u)};
      b = {om(u + stride), er(u + stride), ei(u + stride)};
    };
    Point an = {ld_first<WALK>(sp.om, k), ld_first<WALK>(sp.er, k), ld_first<WALK>(sp.ei, k)};
    Point bn = {ld_first<WALK>(sp.om, k + stride), ld_first<WALK>(sp.er, k + stride), ld_first<WALK>(sp.ei, k + stride)};
    // (two pairs per trip, so that the points read ahead alternate between two
    // sets of registers instead of being copied)
    int32_t u = 0;
    for (; u + 2 * stride < n; u += 4 * stride) {
      Point am, bm;
      read(u + 2 * stride, am, bm);
      body(an, bn);
      read(u + 4 * stride, an, bn);
      body(am, bm);
    }
    if (u < n) body(an, bn);
    return k + n;
  } else {
    Point an = {ld_first<WALK>(sp.om, k), ld_first<WALK>(sp.er, k), ld_first<WALK>(sp.ei, k)};
    Point bn = {ld_first<WALK>(sp.om, k + stride), ld_first<WALK>(sp.er, k + stride), ld_first<WALK>(sp.ei, k + stride)};
    for (int64_t t = 0; t < n_pairs; ++t, k += 2 * stride) {
      const Point a = an, b = bn;
      // in-bounds prefetch of the next two points, no branch
      const int64_t ka = (k + 2 * stride < sp.F) ? k + 2 * stride : k;
      const int64_t kb = (k + 3 * stride < sp.F) ? k + 3 * stride : k;
      an = {ld<WALK>(sp.om, ka), ld<WALK>(sp.er, ka), ld<WALK>(sp.ei, ka)};
      bn = {ld<WALK>(sp.om, kb), ld<WALK>(sp.er, kb), ld<WALK>(sp.ei, kb)};
      body(a, b);
    }
    return k;
  }
}

// --------------------------------------------------------------------------
// Cost pass in rational form.  With w >= 0 (the sign flip) the model sums
// over a set of NR poles are rational functions of y = w^2 with positive
// coefficients,
//   sum_i w_i R_i = P(y) / Q(y),  sum_i (w_i tau_i) R_i = P'(y) / Q(y),
//   Q(y) = prod_i (1 + y tau_i^2),  P(y) = sum_i w_i prod_{j != i} (1 + y tau_j^2),
// evaluated by Horner's rule with one reciprocal per point (no cancellation:
// every term is positive).  The variable is scaled by the largest tau^2 of
// the set (a whole candidate), so every coefficient is at most
// binomial-sized.  The lane takes points k0, k0 + stride, ... and returns its
// partial sums of squared residuals (cost) and of eps' - shift - model
// (sa).  Returns true when the wave must use the basis form instead: a
// lane's smallest coefficient would be subnormal, Q exceeds 1e280 at some
// point, or a cost is not finite (lanes that do not matter are ignored).
// --------------------------------------------------------------------------
template <int NR, int WALK>
__device__ __forceinline__ bool rational_cost_pass(const double *tau2, const double *w, const double *wt,
                                                   bool matters, int k0, int stride, const Spectrum &sp,
                                                   double shift, double &cost_out, double &sa_out) {
  double tmax = 0.0;
#pragma unroll
  for (int i = 0; i < NR; ++i) tmax = tau2[i] > tmax ? tau2[i] : tmax;
  const double isc = tmax > 0.0 ? 1.0 / tmax : 1.0;
  // coefficients built one pole at a time, every update a sum of positive
  // terms: with t the pole's scaled tau^2,
  //   P <- P (1 + y t) + w Q,  P' <- P' (1 + y t) + (w tau) Q,  Q <- Q (1 + y t)
  // (O(NR^2) fused multiply-adds; only Q, P, P' stay live)
  double qc[NR + 1], cr[NR], ci[NR];
  double pnz = 1.0;   // product of the nonzero scaled tau^2: the smallest coefficient
  qc[0] = 1.0;
#pragma unroll
  for (int k = 1; k <= NR; ++k) qc[k] = 0.0;
#pragma unroll
  for (int k = 0; k < NR; ++k) cr[k] = ci[k] = 0.0;
#pragma unroll
  for (int m = 0; m < NR; ++m) {
    const double t = tau2[m] * isc, wm = w[m], wtm = wt[m];
    pnz *= t > 0.0 ? t : 1.0;
#pragma unroll
    for (int k = m; k >= 1; --k) {
      cr[k] = __builtin_fma(wm, qc[k], __builtin_fma(t, cr[k - 1], cr[k]));
      ci[k] = __builtin_fma(wtm, qc[k], __builtin_fma(t, ci[k - 1], ci[k]));
    }
    cr[0] = __builtin_fma(wm, qc[0], cr[0]);
    ci[0] = __builtin_fma(wtm, qc[0], ci[0]);
#pragma unroll
    for (int k = m + 1; k >= 1; --k) qc[k] = __builtin_fma(t, qc[k - 1], qc[k]);
  }
  double csum = qc[NR];
#pragma unroll
  for (int k = 0; k < NR; ++k) csum += cr[k] + ci[k];
  const bool coef_ok = !matters || (pnz >= 1e-280 && fabs(csum) < INFINITY);
  if (__builtin_amdgcn_ballot_w64(!coef_ok) != 0) return true;
  double cost = 0.0, sa = 0.0, qmax = 0.0;
  // two points per trip: their Horner and reciprocal chains interleave
  each_point<WALK, 2>(sp, k0, stride, [&](double om_k, double er, double ei) {
    const double y = (om_k * om_k) * tmax;
    double hq = qc[NR], hr = cr[NR - 1], hi = ci[NR - 1];
#pragma unroll
    for (int d = NR - 1; d >= 0; --d) hq = __builtin_fma(hq, y, qc[d]);
#pragma unroll
    for (int d = NR - 2; d >= 0; --d) {
      hr = __builtin_fma(hr, y, cr[d]);
      hi = __builtin_fma(hi, y, ci[d]);
    }
    qmax = __builtin_fmax(hq, qmax);   // (a NaN shows in the cost)
    const double r = rcp_nr(hq);
    const double rr = (er - shift) - hr * r;
    const double ri = __builtin_fma(-om_k, hi * r, ei);
    sa += rr;
    cost = __builtin_fma(rr, rr, cost);
    cost = __builtin_fma(ri, ri, cost);
  });
  cost_out = cost;
  sa_out = sa;
  return __builtin_amdgcn_ballot_w64(matters && (!(qmax <= 1e280) || !(fabs(cost) + fabs(sa) < INFINITY))) != 0;
}

// --------------------------------------------------------------------------
// The kernel.  GRAD adds the adjoint (grad w.r.t. log10 tau, and per-candidate
// records for the target gradient).
// --------------------------------------------------------------------------
// target waves per SIMD: bounds the register budget of each instantiation.
// Three for the small one-lane kernels (168 registers: the forward ones of up to
// 5 poles and the adjoints of up to 4 hold all but a few of their values in
// them, the adjoints of 6 keep 44 to 76 in scratch memory); two elsewhere: the N =
// 12 two-lane kernels fit three waves with one point per trip of the Gram pass,
// but two waves with two points per trip are faster.  At two (256 registers)
// the one-lane kernels from 9 poles on and the general tiles from 17 keep 30 to
// 220 in scratch memory.
template <int N, int SP, bool GRAD, int UNI> constexpr int waves_per_simd() {
  return (SP == 1 && N <= 6) ? 3 : 2;
}

// Pole split by pole count, measured per bucket on the ragged workload (each
// pole count alone, autotuned frequency split): one lane per candidate up to
// N = 11 (at N = 9..11 its register spills cost less than the DPP traffic and
// the padded pole of the two-lane ring; at N = 12 they do not), two lanes up
// to N = 14, four above, with the Gram matrix on the matrix cores (figures at
// the top of the file; N = 14 at F = 2000 1.80 ms on two lanes, 1.95 on four).
// The adjoint of long spectra keeps two lanes up to N = 16: its third and fourth
// passes take four pole sums a point, which four lanes combine in two steps
// each (N = 16, F = 2000: 3.97 ms on two lanes, 4.22 on four); short ones are
// bound by the solves, which four lanes share (F = 200: 1.20 and 1.05 ms).  On
// two lanes and four, 16,384 candidates: N = 15 at F = 500 303 and 290 us, 700 390
// and 395, 769 419 and 431, 1,100 565 and 603; N = 16 at F = 600 355 and 342, 768
// 427 and 428, 900 487 and 499, 1,100 576 and 604.  (512 candidates, which do not
// fill the chip, are faster on four throughout: N = 15 at F = 1,100 84 and 66 us.)
constexpr int pole_split_for(int n) { return n <= 11 ? 1 : (n <= 14 ? 2 : 4); }
constexpr int pole_split_long_grad(int n) { return n <= 11 ? 1 : (n <= 16 ? 2 : 4); }

// UNI (uniform tiles; the plan checks that every active lane of every tile
// belongs to one material and that spectra hold fewer than 2^29 points):
//   1: frequency split 1, so every lane of a wave reads the same point and
//      the spectra are read with wave-uniform (scalar) loads;
//   2: frequency split > 1: wave-uniform spectrum base, per-lane 32-bit
//      byte offsets (one offset per point for the three arrays).
// XR: the refinement pass in double-double (FLAG_DD_REFINE; forward only).
// One work tile (one wavefront: the candidates the plan lists for it) of the
// cost kernel for N poles; the kernels below call it for their tiles.
// OWN: a tile of candidates 0 .. n-1 of a material in their order, by one wave
// of a block of several, outside the plan's lists; relaxation times ([n][N]
// log10 tau), spectra and costs in LDS.
struct OwnTile {
  int tid;
  double *lds;   // the wave's region
  int32_t n, F;
  const double *theta, *om, *er, *ei;
  double *cost;
};
template <int N, int SP, bool GRAD, int UNI, bool XR = false, bool OWN = false>
__device__ __forceinline__ void fit_tile(const FitArgs &a, const int64_t tile, const OwnTile own = OwnTile()) {
  static_assert(!(XR && GRAD), "the extended-precision refinement is a forward-kernel form");
  using S = Shape<N, SP>;
  constexpr bool MF = S::MF;
  constexpr int NB = S::NB, NV = S::NV, NG = S::NG, D = S::D;
  constexpr int WALK = OWN ? 3 : UNI;
  extern __shared__ double lds_block[];
  double *const lds_all = OWN ? own.lds : lds_block;

  const int lane = OWN ? own.tid & (WAVE - 1) : threadIdx.x;
  const int SF = UNI == 1 ? 1 : a.freq_split;
  const int SL = SP * SF;            // lanes per candidate
  // candidate slot in the wave, the lane's index among the candidate's lanes,
  // its pole lane and its frequency lane.  On the four-lane split (SF a
  // multiple of 4) a candidate holds SF / 4 of the wave's four blocks of 16
  // lanes, each of four pole lanes and four points (see lane_mask).
  const int grp = MF ? ((lane >> 2) & 3) / (SF >> 2) : lane / SL;
  const int sub = MF ? (lane & 3) + ((lane >> 4) << 2) + ((((lane >> 2) & 3) & ((SF >> 2) - 1)) << 4) : lane - grp * SL;
  const int first_lane = MF ? grp * (SF >> 2) * 4 : grp * SL;   // of the candidate
  const int q = sub % SP;            // pole block
  const int fl = UNI == 1 ? 0 : sub / SP; // frequency lane
  // owned pole cI: consecutive poles, or every fourth on the four-lane split
  // (lane q holds row or column q of every tile of four poles)
  auto pole_of = [](int own, int cI) -> int { return MF ? 4 * cI + own : own * NB + cI; };
  const int64_t slot = tile * a.cand_per_wave + grp;
  const int64_t cand = !OWN ? (int64_t)a.lane_cand[slot] : slot < own.n ? slot : -1;
  const bool active = cand >= 0;
  // (inactive lanes of the four-lane split take the first slot's spectrum, so
  // that their wave's point counts are those of its candidates)
  const int32_t mat = OWN ? 0 : active ? a.lane_mat[slot] : MF ? a.lane_mat[tile * a.cand_per_wave] : 0;
  const int64_t c = active ? cand : 0;
  // a wave whose candidates all belong to materials marked done exits
  // before any work (wave-uniform: a block is one wave)
  // (a wave of tiles made for fewer frequency lanes than the kernel's, or for
  // another pole split, can hold padding alone)
  if constexpr (MF || SP != pole_split_for(N))
    if (__builtin_amdgcn_ballot_w64(active) == 0) return;
  if (a.skip_mat && __builtin_amdgcn_ballot_w64(active && a.skip_mat[mat] == 0) == 0) return;

  int64_t f0 = 0, F = 0;
  if constexpr (OWN) {
    F = own.F;
  } else if constexpr (UNI != 0) {
    const int32_t mu = __builtin_amdgcn_readfirstlane(a.lane_mat[tile * a.cand_per_wave]);
    f0 = a.f_off[mu];
    F = a.f_off[mu + 1] - f0;
  } else if (active || MF) {
    f0 = a.f_off[mat];
    F = a.f_off[mat + 1] - f0;
  }
  const double *om = OWN ? own.om : a.omega + f0;
  const double *epr = OWN ? own.er : a.eps_re + f0;
  const double *epi = OWN ? own.ei : a.eps_im + f0;
  const Spectrum spec = {om, epr, epi, F};

  const double damping = a.damping;
  const bool flip = !(a.flags & FLAG_NO_SIGN_FLIP);

  // ---- relaxation times of the owned poles
  double tau[NB];
  bool bad = false;
#pragma unroll
  for (int cI = 0; cI < NB; ++cI) {
    const int p = pole_of(q, cI);
    tau[cI] = 0.0;
    if (p < N && active) {
      const double t = OWN ? ((lds_cptr)own.theta)[c * N + p] : a.theta[c * a.ld + p];
      bad = bad || !(fabs(t) <= THETA_LIMIT);
      tau[cI] = exp10(t);
    }
  }
  // Grouped basis of the frequency passes: group scales s = 2^-k, tau^2 s,
  // and tau s (the factor applied after the sums).  Only these are kept;
  // tau and tau^2 are recovered exactly where needed (ldexp by k).
  int kq[Groups<NB>::NS];
  double sq[Groups<NB>::NS], tau2s[NB], ts[NB];
  {
    double tau2[NB];
#pragma unroll
    for (int cI = 0; cI < NB; ++cI) tau2[cI] = tau[cI] * tau[cI];
    group_scales<NB>(tau2, kq, sq);
#pragma unroll
    for (int cI = 0; cI < NB; ++cI) {
      tau2s[cI] = group_scale<NB>(kq, cI, tau2[cI]);
      ts[cI] = group_scale<NB>(kq, cI, tau[cI]);
    }
  }
  auto tau_of = [&](int cI) { return group_unscale<NB>(kq, cI, ts[cI]); };
  auto tau2_of = [&](int cI) { return group_unscale<NB>(kq, cI, tau2s[cI]); };

  // ---- pass 1: Gram, right-hand side, sum of eps'.  Accumulated with
  // U / s = w R / s in place of I = tau U; the factors tau s are applied
  // after the frequency sums.  (The adjoint's column sums of R, which it needs
  // for eps_inf before its pass 3, are taken in pass 2, which forms every R
  // anyway; the forward kernels take eps_inf from the cost pass.)
  double G[NG], bv[NB], Sv[NB];
#pragma unroll
  for (int e = 0; e < NG; ++e) G[e] = 0.0;
#pragma unroll
  for (int cI = 0; cI < NB; ++cI) {
    bv[cI] = 0.0;
    Sv[cI] = 0.0;
  }
  double sum_er = 0.0;
  // one point of the Gram pass, from its basis values Iv[0 .. NB-1]
  auto gram_acc = [&](double *Iv, double er, double ei) {
#pragma unroll
    for (int cI = 0; cI < NB; ++cI) bv[cI] = __builtin_fma(Iv[cI], ei, bv[cI]);
    if constexpr (MF) {
      // tile (I, J) of four poles by four: the lane's Iv[I] is its row of A
      // (pole 4 I + q at the lane's point), Iv[J] its column of B
#pragma unroll
      for (int I = 0; I < NB; ++I)
#pragma unroll
        for (int J = I; J < NB; ++J)
          G[tri(NB, I, J)] = __builtin_amdgcn_mfma_f64_4x4x4f64(Iv[I], Iv[J], G[tri(NB, I, J)], 0, 0, 0);
    } else if constexpr (SP == 2) {
#pragma unroll
      for (int v = NB; v < NV; ++v) Iv[v] = ring_fetch(Iv[v % NB]);
#pragma unroll
      for (int cI = 0; cI < NB; ++cI)
#pragma unroll
        for (int d = 0; d <= D; ++d) G[cI * (D + 1) + d] = __builtin_fma(Iv[cI], Iv[cI + d], G[cI * (D + 1) + d]);
    } else {
#pragma unroll
      for (int i = 0; i < N; ++i)
#pragma unroll
        for (int j = i; j < N; ++j) G[tri(N, i, j)] = __builtin_fma(Iv[i], Iv[j], G[tri(N, i, j)]);
    }
    sum_er += er;
  };
  auto gram_point = [&](double w, double er, double ei) {
    double Iv[NV];
    basis_Us<NB>(w, w * w, tau2s, sq, Iv);
    gram_acc(Iv, er, ei);
  };
  // Two points per trip let the reciprocal chains of their bases interleave.
  // With no DPP in the body (SP == 1) the compiler pairs the points itself.
  // The ring's DPP moves are convergent operations, which the compiler does
  // not unroll into a loop with a remainder, so on the two-lane split the
  // pair is written out where it fits the register budget at two waves per
  // SIMD: up to N = 14 (the general-tile form from N = 13 on and N = 15, 16
  // spill with it).
  constexpr bool PAIR_RING = SP == 2 && (N == 12 || (N <= 14 && UNI != 0));
  if constexpr (MF) {
    // The matrix instruction takes every lane of the wave, so the trips are
    // counted for the whole wave: n_full of them give every lane two points of
    // its own, the rest (one, where the tile is uniform) lets a lane without
    // a point run at w = 0, whose U is 0.
    int64_t n_full = F / (2 * SF), n_all = (F + 2 * SF - 1) / (2 * SF);
    if constexpr (UNI == 0) {
#pragma unroll
      for (int m = 4; m < 16; m <<= 1) {   // over the blocks, hence the candidates
        const int64_t of = __shfl_xor(n_full, m, WAVE), oa = __shfl_xor(n_all, m, WAVE);
        n_full = of < n_full ? of : n_full;
        n_all = oa > n_all ? oa : n_all;
      }
      auto uniform = [](int64_t v) -> int64_t {
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
        const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
        return (int64_t)(((uint64_t)hi << 32) | lo);
      };
      n_full = uniform(n_full);
      n_all = uniform(n_all);
    }
    int64_t k = each_pair<WALK>(spec, fl, SF, n_full, [&](const Point &a, const Point &b) {
      double Ia[NV], Ib[NV];
      basis_Us2<NB>(a.w, b.w, tau2s, sq, Ia, Ib);
      gram_acc(Ia, a.er, a.ei);
      gram_acc(Ib, b.er, b.ei);
    });
    for (int64_t t = n_full; t < n_all; ++t, k += 2 * SF) {
      const bool va = k < F, vb = k + SF < F;
      const int64_t ka = va ? k : F - 1, kb = vb ? k + SF : F - 1;
      const double wa = va ? ld<WALK>(om, ka) : 0.0, wb = vb ? ld<WALK>(om, kb) : 0.0;
      double Ia[NV], Ib[NV];
      basis_Us2<NB>(wa, wb, tau2s, sq, Ia, Ib);
      gram_acc(Ia, va ? ld<WALK>(epr, ka) : 0.0, va ? ld<WALK>(epi, ka) : 0.0);
      gram_acc(Ib, vb ? ld<WALK>(epr, kb) : 0.0, vb ? ld<WALK>(epi, kb) : 0.0);
    }
  } else if constexpr (!PAIR_RING) {
    each_point<WALK, SP == 1 ? 2 : 1>(spec, fl, SF, gram_point);
  } else {
    // the pairs that every lane of the wave has, then the lane's own (the pole
    // lanes of a candidate share their frequency lane, hence their trip counts)
    int64_t k = fl;
    auto pair = [&](const Point &a, const Point &b) {
      double Ia[NV], Ib[NV];
      basis_Us2<NB>(a.w, b.w, tau2s, sq, Ia, Ib);
      gram_acc(Ia, a.er, a.ei);
      gram_acc(Ib, b.er, b.ei);
    };
    if constexpr (WALK == 2) k = each_pair<WALK>(spec, fl, SF, F / (2 * SF), pair);
    else if (k + SF < F) k = each_pair<WALK>(spec, fl, SF, (F - fl + SF - 1) / SF / 2, pair);
    for (; k < F; k += SF) gram_point(ld<WALK>(om, k), ld<WALK>(epr, k), ld<WALK>(epi, k));
  }
  freq_sum_n<NG, SP, MF ? 16 : SP>(G, SL);   // (the four points of a block are summed by the matrix instruction)
  if constexpr (SP == 2) {
    double tv[NV];
#pragma unroll
    for (int v = 0; v < NV; ++v) tv[v] = v < NB ? ts[v] : ring_fetch(ts[v % NB]);
#pragma unroll
    for (int cI = 0; cI < NB; ++cI)
#pragma unroll
      for (int d = 0; d <= D; ++d) G[cI * (D + 1) + d] *= ts[cI] * tv[cI + d];
  } else if constexpr (SP == 1) {
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int j = i; j < N; ++j) G[tri(N, i, j)] *= ts[i] * ts[j];
  }
  freq_sum_n<NB, SP, SP>(bv, SL);
#pragma unroll
  for (int cI = 0; cI < NB; ++cI) {
    bv[cI] = bv[cI] * ts[cI];
    bad = bad || !(fabs(bv[cI]) < INFINITY);
  }
  sum_er = freq_sum<SP, SP>(sum_er, SL);
  bad = bad || !(fabs(sum_er) < INFINITY);
  bad = group_sum<SP>(bad ? 1.0 : 0.0) != 0.0;

  // ---- DLS solve (equilibrated, damped Cholesky)
  const double tol = 8.0 * (double)(F > N ? F : N) * 0x1.0p-53;
  double zt[NB], zc[NB], invd_own[NB];
  bool ok;
  double *L = nullptr;
  double uinv_r[SP == 1 ? N : 1], invd_r[SP == 1 ? N : 1];
  if constexpr (SP == 1) {
    ok = equilibrate_factor<N>(G, invd_r, uinv_r, damping, tol);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      zt[i] = bv[i] * invd_r[i];
      invd_own[i] = invd_r[i];
    }
    chol_solve<N>(G, uinv_r, zt);
    // Park the factor in LDS (reciprocal pivots in place of its diagonal,
    // which the solves never read), element-major so that a wave's lanes touch
    // consecutive addresses.  The later solves read it back; meanwhile its
    // registers serve the frequency passes.
    {
      double *park = lds_all;
      const int cpw = WAVE / SL;
      if (fl == 0) {
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
          for (int j = i; j < N; ++j) park[tri(N, i, j) * cpw + grp] = (i == j) ? uinv_r[i] : G[tri(N, i, j)];
      }
      wave_sync();
    }
  } else {
    // assemble the packed triangle in LDS (all lanes of a candidate write the same values)
    L = lds_all + (int64_t)grp * S::LDS_DOUBLES;
    const LdsLayout<N> lay(L);
    double *A = lay.A, *invd = lay.invd, *uinv = lay.uinv, *vb = lay.vb, *vz = lay.vz;
    if constexpr (MF) {
      // the lane holds element (row lane >> 4, column q) of every tile; the
      // rows' factors tau s come through LDS
      double *st = lay.vw;
#pragma unroll
      for (int cI = 0; cI < NB; ++cI) {
        const int p = pole_of(q, cI);
        if (p < N) {
          st[p] = ts[cI];
          vb[p] = bv[cI];
        }
      }
      wave_sync();
      const int row = lane >> 4;
#pragma unroll
      for (int I = 0; I < NB; ++I) {
        const int r = 4 * I + row;
        const double tr = r < N ? st[r] : 0.0;
#pragma unroll
        for (int J = I; J < NB; ++J) {
          const int c2 = 4 * J + q;
          if (c2 < N && r <= c2) A[tcol(r, c2)] = G[tri(NB, I, J)] * (tr * ts[J]);
        }
      }
    }
#pragma unroll
    for (int cI = 0; cI < (MF ? 0 : NB); ++cI) {
      const int p1 = q * NB + cI;
#pragma unroll
      for (int d = 0; d <= D; ++d) {
        int p2 = p1 + d;
        if (p2 >= S::NP) p2 -= S::NP;
        if (p1 < N && p2 < N) {
          const int i = p1 < p2 ? p1 : p2, j = p1 < p2 ? p2 : p1;
          A[tcol(i, j)] = G[cI * (D + 1) + d];
        }
      }
      if (p1 < N) vb[p1] = bv[cI];
    }
    wave_sync();
    if constexpr (MF) {
      const Coop<N> coop((lds_ptr)A, (lds_ptr)uinv, sub & 15, first_lane);
      double x0, x1;
      ok = coop.factor((lds_cptr)vb, (lds_ptr)invd, (lds_ptr)lay.vw, (lds_ptr)vz, damping, tol, x0, x1);
      coop.backward(x0, x1);
      coop.put((lds_ptr)vz, x0, x1);
    } else {
      ok = lds_equilibrate_factor<N>((lds_ptr)A, (lds_ptr)invd, (lds_ptr)uinv, damping, tol);
      for (int i = 0; i < N; ++i) vz[i] = vb[i] * invd[i];
      lds_chol_solve<N>((lds_cptr)A, (lds_cptr)uinv, (lds_ptr)vz);
    }
    wave_sync();
#pragma unroll
    for (int cI = 0; cI < NB; ++cI) {
      const int p = pole_of(q, cI);
      zt[cI] = p < N ? vz[p] : 0.0;
      invd_own[cI] = p < N ? invd[p] : 0.0;
    }
  }
#pragma unroll
  for (int cI = 0; cI < NB; ++cI) zc[cI] = zt[cI] * invd_own[cI];

  // ---- pass 2: corrected semi-normal equations, g = I^T (eps'' - I z).
  // The residual is nearly orthogonal to the columns of I, so g is a sum with
  // heavy cancellation; it is accumulated with compensation (residual
  // refinement with the residual products summed in extra precision).
  // FLAG_NO_REFINE skips it (the forward kernels skip the whole pass; the
  // adjoint still runs it for the column sums of R that its eps_inf needs).
  const bool refine = XR || !(a.flags & FLAG_NO_REFINE);
  double gv[NB], gl[NB];
#pragma unroll
  for (int cI = 0; cI < NB; ++cI) {
    gv[cI] = 0.0;
    gl[cI] = 0.0;
  }
  if constexpr (XR) {
    // The same g = I^T (eps'' - I z) with every quantity that the rounding
    // of the FP64 pass disturbs carried in double-double: the relaxation
    // times, x = w tau, 1 + x^2, R = 1/(1 + x^2) and I = x R, the residual
    // (its pole sum by TwoSum, the low parts added plainly) and the sums of
    // I r (likewise).  Written with contraction off: every product whose
    // rounding error is recovered must stay a separate rounded product.
#pragma clang fp contract(off)
    double th[NB], tl[NB];
#pragma unroll
    for (int cI = 0; cI < NB; ++cI) {
      const int p = pole_of(q, cI);
      th[cI] = 0.0;   // padded poles: x = 0, so I = 0
      tl[cI] = 0.0;
      if (p < N && active) {
        const double t = a.theta[c * a.ld + p];
        const ddv v = exp10_dd(fabs(t) <= THETA_LIMIT ? t : 0.0);   // rejected candidates: any finite value
        th[cI] = v.h;
        tl[cI] = v.l;
      }
    }
    if (fl < F) {
      double wn = ld<WALK>(om, fl), en = ld<WALK>(epi, fl);
      for (int64_t k = fl; k < F; k += SF) {
        const double w = wn, ei = en;
        const int64_t kn = k + SF < F ? k + SF : k;   // the next point, loaded one trip ahead
        wn = ld<WALK>(om, kn);
        en = ld<WALK>(epi, kn);
        double Ih[NB], Il[NB];
        double sh = 0.0, sl = 0.0;   // sum over the owned poles of z_i I_i
#pragma unroll
        for (int cI = 0; cI < NB; ++cI) {
          const ddv I = dd_debye_I(w, th[cI], tl[cI]);
          Ih[cI] = I.h;
          Il[cI] = I.l;
          const double ih = I.h;
          const double ph = zc[cI] * ih;
          const double pl = __builtin_fma(zc[cI], Il[cI], __builtin_fma(zc[cI], ih, -ph));
          const ddv s2 = two_sum(sh, ph);
          sh = s2.h;
          sl = sl + (s2.l + pl);
        }
        if constexpr (SP > 1) {
          // over the candidate's pole lanes (TwoSum's error does not depend
          // on the operand order: every lane ends with the same pair)
          ddv s2 = two_sum(sh, dpp_quad<QP_SWAP1>(sh));
          sl = (sl + dpp_quad<QP_SWAP1>(sl)) + s2.l;
          sh = s2.h;
          if constexpr (SP == 4) {
            s2 = two_sum(sh, dpp_quad<QP_SWAP2>(sh));
            sl = (sl + dpp_quad<QP_SWAP2>(sl)) + s2.l;
            sh = s2.h;
          }
        }
        ddv rr = two_sum(ei, -sh);
        rr = two_sum(rr.h, rr.l - sl);
#pragma unroll
        for (int cI = 0; cI < NB; ++cI) {
          const double gh = Ih[cI] * rr.h;
          const double ge = __builtin_fma(Ih[cI], rr.l, __builtin_fma(Il[cI], rr.h, __builtin_fma(Ih[cI], rr.h, -gh)));
          const ddv s2 = two_sum(gv[cI], gh);
          gv[cI] = s2.h;
          gl[cI] = gl[cI] + (s2.l + ge);
        }
      }
    }
    freq_sum_dd_n<NB, SP, SP>(gv, gl, SL);
  } else if constexpr (!GRAD && (SP == 4 || (SP == 2 && NB <= 6))) {
    if (refine) {
      // The pole splits run this pass over pairs of owner lanes: lane q takes
      // the poles of owner lanes 2h and 2h + 1 (their groups of four, then
      // their leftover poles) on every other point of its frequency lane's
      // points.  On the four-lane split h = q & 1 and the point subset is
      // q >> 1, so a point's model sum needs one exchange (between the two
      // halves) instead of two; on the two-lane split h = 0, the subset is q,
      // and a lane holds the whole candidate: no exchange.  Each point's
      // basis is formed by half the lanes.  The owners' tau^2 s and tau s z
      // reach the lanes through the candidate's LDS region (its
      // right-hand-side and correction vectors are free during this pass),
      // and the sums of (R / s)(w r), added over the point subsets and
      // frequency lanes, return to the owners the same way.  (On the
      // two-lane split only up to N = 12: beyond, its 2 NB poles per lane
      // spill registers.)
      constexpr int NQ = Groups<NB>::NQ;   // groups of four per owner
      constexpr int LO = NB - 4 * NQ;      // leftover poles per owner
      static_assert(!Groups<NB>::THREE, "the owners' leftovers are taken in pairs");
      constexpr int H = 2 * NB;            // poles per lane
      constexpr int HP = SP / 2;           // owner pairs per candidate
      const int h = q % HP;
      // the pole of element e: owner 2h's groups, owner 2h + 1's, then owner
      // 2h's leftovers, owner 2h + 1's
      auto pole = [&](int e) -> int {
        const int own = 2 * h + (e < 8 * NQ ? e / (4 * NQ) : (e - 8 * NQ) / (LO > 0 ? LO : 1));
        const int cI = e < 8 * NQ ? e % (4 * NQ) : 4 * NQ + (e - 8 * NQ) % (LO > 0 ? LO : 1);
        return pole_of(own, cI);
      };
      const LdsLayout<N> lay(L);
      double *st2 = lay.vb, *stz = lay.vw;
#pragma unroll
      for (int cI = 0; cI < NB; ++cI) {
        const int p = pole_of(q, cI);
        if (p < N) {   // (every frequency lane of the owner writes the same values)
          st2[p] = tau2s[cI];
          stz[p] = zc[cI] * ts[cI];
          if constexpr (MF) lay.vt[p] = ts[cI];
        }
      }
      wave_sync();
      double t2h[H], zh[H];
#pragma unroll
      for (int e = 0; e < H; ++e) {
        const int p = pole(e);
        t2h[e] = p < N ? st2[p] : 0.0;   // padded poles: no weight
        zh[e] = p < N ? stz[p] : 0.0;
      }
      double gh[H], gc[H];
#pragma unroll
      for (int e = 0; e < H; ++e) gh[e] = gc[e] = 0.0;
      // four points of the lane at a time (on the four-lane split the two
      // halves of a point subset take the same points, so their exchanges
      // pair up), compensated as below
      const int64_t s2 = 2 * (int64_t)SF;
      // w r at point kk, with the point's R / s in R
      auto pair_resid = [&](auto at, int64_t kk, double *R) {
        const double w = at(om, kk);
        basis_two_owners<NQ, LO>(w * w, t2h, sq, R);
        double part = 0.0;
#pragma unroll
        for (int e = 0; e < H; ++e) part = __builtin_fma(R[e], zh[e], part);
        if constexpr (HP == 2) part = part + dpp_quad<QP_SWAP1>(part);
        return w * __builtin_fma(-w, part, at(epi, kk));
      };
      auto blk = [&](auto at, int64_t k0, int np) {   // np >= 1 points
        double pb[H], R[H];
        {
          const double wr = pair_resid(at, k0, R);
#pragma unroll
          for (int e = 0; e < H; ++e) pb[e] = R[e] * wr;
        }
        for (int t = 1; t < np; ++t) {
          const double wr = pair_resid(at, k0 + t * s2, R);
#pragma unroll
          for (int e = 0; e < H; ++e) pb[e] = __builtin_fma(R[e], wr, pb[e]);
        }
#pragma unroll
        for (int e = 0; e < H; ++e) kahan_fma_acc(gh[e], gc[e], 1.0, pb[e]);
      };
      // (two blocks per trip, so that the compensated sums alternate between
      // two registers instead of being copied back every update)
      // (uniform tiles with a split: the trips that every lane has, the base
      // moved on by the scalar unit; then the lane's own)
      auto own = [](const double *p, int64_t kk) { return ld<WALK>(p, kk); };
      int64_t k = (q / HP) * SF + fl;
      if constexpr (WALK == 2) {
        const Reader rom(om, F, k), rei(epi, F, k);
        auto lane = [&](const double *p, int64_t ku) { return p == om ? rom((int32_t)ku) : rei((int32_t)ku); };
        int32_t u = 0;
        for (; u + 16 * SF <= (int32_t)F; u += 16 * SF) {
          blk(lane, u, 4);
          blk(lane, u + 8 * SF, 4);
        }
        k += u;
        for (; k + 3 * s2 < F; k += 4 * s2) blk(own, k, 4);
      } else {
        for (; k + 7 * s2 < F; k += 8 * s2) {
          blk(own, k, 4);
          blk(own, k + 4 * s2, 4);
        }
        if (k + 3 * s2 < F) {
          blk(own, k, 4);
          k += 4 * s2;
        }
      }
      if (k < F) blk(own, k, (int)((F - 1 - k) / s2) + 1);
      {
        double ngc[H];
#pragma unroll
        for (int e = 0; e < H; ++e) ngc[e] = -gc[e];
        freq_sum_dd_n<H, SP, HP>(gh, ngc, SL);   // the point subsets and the frequency lanes
      }
      wave_sync();
#pragma unroll
      for (int e = 0; e < H; ++e) {
        const int p = pole(e);
        if (p < N) stz[p] = gh[e];   // (both point subsets hold the same sums)
      }
      wave_sync();
#pragma unroll
      for (int cI = 0; cI < NB; ++cI) {
        const int p = pole_of(q, cI);
        if constexpr (MF) {
          // the owned poles' values come back from LDS: kept in registers
          // across the pass they would spill
          tau2s[cI] = p < N ? st2[p] : 0.0;
          ts[cI] = p < N ? lay.vt[p] : 0.0;
          zt[cI] = p < N ? lay.vz[p] : 0.0;
          invd_own[cI] = p < N ? lay.invd[p] : 0.0;
        }
        gv[cI] = (p < N ? stz[p] : 0.0) * ts[cI];
      }
    }
  } else if (GRAD || refine) {
    // I z = w sum_i (tau_i s_i z_i) (R_i / s_i), and I^T r = tau s ((R / s)^T (w r))
    double zs[NB];
#pragma unroll
    for (int cI = 0; cI < NB; ++cI) zs[cI] = zc[cI] * ts[cI];
    // R / s at point k (for the adjoint its column sums taken on the way) and w_k r_k
    // w_k r_k from the basis values Rv at point k (for the adjoint the column
    // sums of R taken on the way)
    auto resid_R = [&](double w, double ei, const double *Rv) {
      double part = 0.0;
#pragma unroll
      for (int cI = 0; cI < NB; ++cI) {
        if constexpr (GRAD) Sv[cI] += Rv[cI];
        part = __builtin_fma(Rv[cI], zs[cI], part);
      }
      return w * __builtin_fma(-w, group_sum<SP>(part), ei);
    };
    auto resid = [&](double w, double ei, double *Rv) {
      basis_Rs<NB>(w * w, tau2s, sq, Rv);
      return resid_R(w, ei, Rv);
    };
    // The compensated sum takes the terms of four points at a time, summed
    // plainly (at most four roundings of terms of the same four points, so
    // the error bound stays a small multiple of the roundoff of the terms'
    // magnitudes; a CPU emulation of the whole solve put the cost error
    // against the 80-bit oracle at the level of single-term compensation).
    auto block4 = [&](auto at, int64_t k0) {
      double pb[NB];
      if constexpr (odd_pole<NB>() && SP == 4) {
        // the points in pairs: the odd pole's values of two points share a
        // reciprocal (the terms and their order as below; on the four-lane
        // split only, where the extra registers are free: with one lane per
        // candidate they spill)
#pragma unroll
        for (int t = 0; t < 4; t += 2) {
          const int64_t ka = k0 + t * SF, kb = ka + SF;
          const double wa = at(om, ka), wb = at(om, kb);
          double Ra[NB], Rb[NB];
          basis_Rs2<NB>(wa * wa, wb * wb, tau2s, sq, Ra, Rb);
          const double wra = resid_R(wa, at(epi, ka), Ra);
#pragma unroll
          for (int cI = 0; cI < NB; ++cI) pb[cI] = t == 0 ? Ra[cI] * wra : __builtin_fma(Ra[cI], wra, pb[cI]);
          const double wrb = resid_R(wb, at(epi, kb), Rb);
#pragma unroll
          for (int cI = 0; cI < NB; ++cI) pb[cI] = __builtin_fma(Rb[cI], wrb, pb[cI]);
        }
      } else {
        double R[NB];
        {
          const double wr = resid(at(om, k0), at(epi, k0), R);
#pragma unroll
          for (int cI = 0; cI < NB; ++cI) pb[cI] = R[cI] * wr;
        }
#pragma unroll
        for (int t = 1; t < 4; ++t) {
          const int64_t kk = k0 + t * SF;
          const double wr = resid(at(om, kk), at(epi, kk), R);
#pragma unroll
          for (int cI = 0; cI < NB; ++cI) pb[cI] = __builtin_fma(R[cI], wr, pb[cI]);
        }
      }
#pragma unroll
      for (int cI = 0; cI < NB; ++cI) kahan_fma_acc(gv[cI], gl[cI], 1.0, pb[cI]);
    };
    // two blocks per trip: the compensated sums then alternate between two
    // registers instead of being copied back every update
    auto own = [](const double *p, int64_t kk) { return ld<WALK>(p, kk); };
    int64_t k = fl;
    if constexpr (WALK == 2) {   // the trips that every lane has; then the lane's own
      const Reader rom(om, F, fl), rei(epi, F, fl);
      auto lane = [&](const double *p, int64_t ku) { return p == om ? rom((int32_t)ku) : rei((int32_t)ku); };
      int32_t u = 0;
      for (; u + 8 * SF <= (int32_t)F; u += 8 * SF) {
        block4(lane, u);
        block4(lane, u + 4 * SF);
      }
      k += u;
      for (; k + 3 * SF < F; k += 4 * SF) block4(own, k);
    } else {
      for (; k + 7 * SF < F; k += 8 * SF) {
        block4(own, k);
        block4(own, k + 4 * SF);
      }
      if (k + 3 * SF < F) {
        block4(own, k);
        k += 4 * SF;
      }
    }
    if (k < F) {   // the last one to three points
      double pb[NB], R[NB];
#pragma unroll
      for (int cI = 0; cI < NB; ++cI) pb[cI] = 0.0;
      for (; k < F; k += SF) {
        const double wr = resid(ld<WALK>(om, k), ld<WALK>(epi, k), R);
#pragma unroll
        for (int cI = 0; cI < NB; ++cI) pb[cI] = __builtin_fma(R[cI], wr, pb[cI]);
      }
#pragma unroll
      for (int cI = 0; cI < NB; ++cI) kahan_fma_acc(gv[cI], gl[cI], 1.0, pb[cI]);
    }
    {
      double ngl[NB];
#pragma unroll
      for (int cI = 0; cI < NB; ++cI) ngl[cI] = -gl[cI];
      freq_sum_dd_n<NB, SP, SP>(gv, ngl, SL);
    }
    if constexpr (GRAD) freq_sum_n<NB, SP, SP>(Sv, SL);
#pragma unroll
    for (int cI = 0; cI < NB; ++cI) {
      gv[cI] = gv[cI] * ts[cI];
      if constexpr (GRAD) Sv[cI] = Sv[cI] * pole_scale<NB>(sq, cI);
    }
  }

  // correction: zt += A^-1 (D^-1 g - damping zt)
  if (refine) {
    if constexpr (SP == 1) {
      double dz[N];
#pragma unroll
      for (int i = 0; i < N; ++i) dz[i] = __builtin_fma(gv[i], invd_r[i], -damping * zt[i]);
      double Af[S::NT], uf[N];
      unpark<N>(lds_all, WAVE / SL, grp, Af, uf);
      chol_solve<N>(Af, uf, dz);
#pragma unroll
      for (int i = 0; i < N; ++i) zt[i] += dz[i];
    } else {
      const LdsLayout<N> lay(L);
      double *A = lay.A, *uinv = lay.uinv, *vw = lay.vw;
#pragma unroll
      for (int cI = 0; cI < NB; ++cI) {
        const int p = pole_of(q, cI);
        if (p < N) vw[p] = __builtin_fma(gv[cI], invd_own[cI], -damping * zt[cI]);
      }
      wave_sync();
      if constexpr (MF) {
        const Coop<N> coop((lds_ptr)A, (lds_ptr)uinv, sub & 15, first_lane);
        double x0, x1;
        coop.get((lds_cptr)vw, x0, x1);
        coop.forward(x0, x1);
        coop.backward(x0, x1);
        coop.put((lds_ptr)vw, x0, x1);
      } else {
        lds_chol_solve<N>((lds_cptr)A, (lds_cptr)uinv, (lds_ptr)vw);
      }
      wave_sync();
#pragma unroll
      for (int cI = 0; cI < NB; ++cI) {
        const int p = pole_of(q, cI);
        zt[cI] += p < N ? vw[p] : 0.0;
      }
    }
  }
  double wv_[NB];
  double ws_part = 0.0;
#pragma unroll
  for (int cI = 0; cI < NB; ++cI) {
    zc[cI] = zt[cI] * invd_own[cI];
    wv_[cI] = flip ? fabs(zc[cI]) : zc[cI];
    if constexpr (GRAD) ws_part = __builtin_fma(wv_[cI], Sv[cI], ws_part);
  }
  // eps_inf: the adjoint takes it from the column sums before its pass 3.
  // The forward kernels take it from the cost pass: with v_k = eps'_k -
  // (R w)_k, eps_inf is the mean of v and the real part of the cost is
  // sum (v - mean)^2 = sum (v - K)^2 - (sum (v - K))^2 / F for any shift K.
  // K = v_0 (the first point) differs from the mean by about one residual,
  // so the subtraction loses at most a few digits of the cost's last bits.
  double einf = 0.0, shift = 0.0;
  if constexpr (GRAD) {
    einf = (F > 0) ? (sum_er - group_sum<SP>(ws_part)) / (double)F : 0.0;
    shift = einf;
  } else if (F > 0) {
    const double w0 = ld<WALK>(om, 0);
    double Rv[NB];
    basis_Rs<NB>(w0 * w0, tau2s, sq, Rv);
    double pr = 0.0;
#pragma unroll
    for (int cI = 0; cI < NB; ++cI) pr = __builtin_fma(wv_[cI] * pole_scale<NB>(sq, cI), Rv[cI], pr);
    shift = ld<WALK>(epr, 0) - group_sum<SP>(pr);
  }

  // ---- pass 3: residuals and cost (+ g_w for the adjoint)
  double gw[GRAD ? NB : 1], gw2[GRAD ? NB : 1], wt[NB];
#pragma unroll
  for (int cI = 0; cI < (GRAD ? NB : 1); ++cI) gw[cI] = gw2[cI] = 0.0;
#pragma unroll
  for (int cI = 0; cI < NB; ++cI) wt[cI] = wv_[cI] * tau_of(cI);
  // from the basis values of every point (grouped form: the weights carry the
  // scales, and the adjoint's sums g_w get theirs afterwards); rr is
  // eps' - shift - R w, and sa collects its sum (the forward kernels' shifted
  // mean)
  auto pass3_basis = [&](double &sa) -> double {
    double acc = 0.0;
    double wvs[NB], wts[NB];
#pragma unroll
    for (int cI = 0; cI < NB; ++cI) {
      wvs[cI] = wv_[cI] * pole_scale<NB>(sq, cI);
      wts[cI] = wv_[cI] * ts[cI];
    }
    sa = 0.0;
    each_point<WALK, 1>(spec, fl, SF, [&](double w, double er, double ei) {
      double Rv[NB];
      basis_Rs<NB>(w * w, tau2s, sq, Rv);
      double pr = 0.0, pi = 0.0;
#pragma unroll
      for (int cI = 0; cI < NB; ++cI) {
        pr = __builtin_fma(wvs[cI], Rv[cI], pr);
        pi = __builtin_fma(wts[cI], Rv[cI], pi);
      }
      const double rr = (er - shift) - group_sum<SP>(pr);
      const double ri = __builtin_fma(-w, group_sum<SP>(pi), ei);
      if constexpr (!GRAD) sa += rr;
      acc = __builtin_fma(rr, rr, acc);
      acc = __builtin_fma(ri, ri, acc);
      if constexpr (GRAD) {
        // g_w = R^T r' + I^T r'' = s ((R/s)^T r' + tau ((R/s)^T (w r'')))
        const double wri = w * ri;
#pragma unroll
        for (int cI = 0; cI < NB; ++cI) {
          gw[cI] = __builtin_fma(Rv[cI], rr, gw[cI]);
          gw2[cI] = __builtin_fma(Rv[cI], wri, gw2[cI]);
        }
      }
    });
    return acc;
  };
  double cost, sa = 0.0;
  // lanes whose partial sums are added at the end: the frequency lanes of the
  // pole group (basis form: the pole group's sums are combined per point), or
  // all lanes of the candidate (rational form over the whole candidate)
  int red_from = SP;
  if constexpr (GRAD) {
    cost = pass3_basis(sa);
  } else {
    // (lanes whose cost is replaced by their status do not count)
    const bool matters = active && !bad && ok;
    bool use_basis = !flip;
    if (!use_basis) {
      if constexpr (SP == 1) {
        double tau2v[NB];
#pragma unroll
        for (int cI = 0; cI < NB; ++cI) tau2v[cI] = tau2_of(cI);
        use_basis = rational_cost_pass<NB, WALK>(tau2v, wv_, wt, matters, fl, SF, spec, shift, cost, sa);
      } else {
        // every lane of the candidate takes all N poles (gathered through the
        // candidate's LDS region, whose right-hand-side, first-solution and
        // scaling vectors are free after the solves) and every SL-th point:
        // one rational function of degree N per point instead of SP of degree
        // NB combined across lanes
        const LdsLayout<N> lay(L);
        double *t2s = lay.vb, *wsh = lay.vz, *wts = lay.invd;
        wave_sync();
#pragma unroll
        for (int cI = 0; cI < NB; ++cI) {
          const int p = pole_of(q, cI);
          if (p < N) {
            t2s[p] = tau2_of(cI);
            wsh[p] = wv_[cI];
            wts[p] = wt[cI];
          }
        }
        wave_sync();
        use_basis = rational_cost_pass<N, WALK>(t2s, wsh, wts, matters, sub, SL, spec, shift, cost, sa);
        red_from = 1;
      }
    }
    if (use_basis) {
      cost = pass3_basis(sa);
      red_from = SP;
    }
  }
  {
    double part[2] = {cost, sa};
    constexpr int K = GRAD ? 1 : 2;
    if (SP > 1 && red_from == 1) freq_sum_n<K, SP, 1>(part, SL);
    else freq_sum_n<K, SP, SP>(part, SL);
    cost = part[0];
    sa = part[1];
  }
  if constexpr (!GRAD) {
    if (F > 0) {
      cost -= sa * (sa / (double)F);
      einf = shift + sa / (double)F;
    }
  }

  const bool sing = !ok;
  const int st = bad ? ST_BADINPUT : (sing ? ST_SINGULAR : ST_OK);
  const bool writer = active && fl == 0;
  double gc = 1.0;
  if (writer && q == 0) {
    const double result = st == ST_OK ? cost : (st == ST_SINGULAR ? INFINITY : NAN);
    if constexpr (OWN) {
      ((lds_ptr)own.cost)[c] = result;
      if (a.status) a.status[c] = (int8_t)st;
      return;
    }
    a.cost[c] = result;
    if (a.eps_inf) a.eps_inf[c] = st == ST_OK ? einf : NAN;
    if (a.status) a.status[c] = (int8_t)st;
  }
  if (!OWN && writer && a.weights) {
#pragma unroll
    for (int cI = 0; cI < NB; ++cI) {
      const int p = pole_of(q, cI);
      if (p < N) a.weights[c * a.ld + p] = st == ST_OK ? wv_[cI] : NAN;
    }
  }
  if constexpr (!GRAD) {
    return;
  } else {
    // ---- adjoint: mu = M^-1 (s o g_w), M = D A D
    if (a.grad_cost) gc = active ? a.grad_cost[c] : 0.0;
    double mt[NB], mu[NB];
    freq_sum_n<NB, SP, SP>(gw2, SL);
    freq_sum_n<NB, SP, SP>(gw, SL);
#pragma unroll
    for (int cI = 0; cI < NB; ++cI) {
      gw[cI] = -2.0 * pole_scale<NB>(sq, cI) * __builtin_fma(tau_of(cI), gw2[cI], gw[cI]);
      const double s = (flip && zc[cI] < 0.0) ? -1.0 : 1.0;
      mt[cI] = s * gw[cI] * invd_own[cI];
    }
    if constexpr (SP == 1) {
      double Af[S::NT], uf[N];
      unpark<N>(lds_all, WAVE / SL, grp, Af, uf);
      chol_solve<N>(Af, uf, mt);
    } else {
      const LdsLayout<N> lay(L);
      double *A = lay.A, *uinv = lay.uinv, *vw = lay.vw;
#pragma unroll
      for (int cI = 0; cI < NB; ++cI) {
        const int p = pole_of(q, cI);
        if (p < N) vw[p] = mt[cI];
      }
      wave_sync();
      if constexpr (MF) {
        const Coop<N> coop((lds_ptr)A, (lds_ptr)uinv, sub & 15, first_lane);
        double x0, x1;
        coop.get((lds_cptr)vw, x0, x1);
        coop.forward(x0, x1);
        coop.backward(x0, x1);
        coop.put((lds_ptr)vw, x0, x1);
      } else {
        lds_chol_solve<N>((lds_cptr)A, (lds_cptr)uinv, (lds_ptr)vw);
      }
      wave_sync();
#pragma unroll
      for (int cI = 0; cI < NB; ++cI) {
        const int p = pole_of(q, cI);
        mt[cI] = p < N ? vw[p] : 0.0;
      }
    }
#pragma unroll
    for (int cI = 0; cI < NB; ++cI) mu[cI] = mt[cI] * invd_own[cI];

    // per-candidate record for the target gradient: [w | z | mu | tau | eps_inf, gc]
    if (writer && a.record) {
      double *rec = a.record + c * a.rec_ld;
#pragma unroll
      for (int cI = 0; cI < NB; ++cI) {
        const int p = pole_of(q, cI);
        if (p >= N) continue;
        rec[p] = wv_[cI];
        rec[N + p] = zc[cI];
        rec[2 * N + p] = mu[cI];
        rec[3 * N + p] = tau_of(cI);
        if (p == 0) {
          rec[4 * N] = einf;
          rec[4 * N + 1] = st == ST_OK ? gc : 0.0;
        }
      }
    }

    // ---- pass 4: basis derivatives against the residuals r', r'', q = eps'' -
    // I z and I mu.  With x^2 R = 1 - R, dR/dtheta = -2 ln10 I^2 and dI/dtheta =
    // ln10 I (2R - 1), so the gradient of pole i is, up to ln10, the sum of
    // I (2R - 1) (-2 w r'' + mu q - z (I mu) - 2 lambda mu z I) + 4 w I^2 r'.
    // tau and the group scales are applied after the sums: with R' = R / s and
    // h = 2 s R'^2 - R', I = tau s w R' and I (2R - 1) = tau s w h.  Three sums a
    // pole, what is known of the poles inside the first: two more would save an
    // operation and spill (56 registers at N = 16).  Against tau inside the sums,
    // reciprocals by pairs and four sums, adjoint of 128 candidates (N <= 11; 256
    // beyond) of 256 materials, F = 2,000: N = 8 953 -> 910 us, N = 11 1,444 ->
    // 1,288, N = 16 4,112 -> 3,961; N = 12, bound by the other passes, 3,040 ->
    // 3,054, at F = 200 736 -> 716.
    double T1[NB], T2[NB], T3[NB], wvs[NB], wts[NB], zts[NB], mts[NB];
#pragma unroll
    for (int cI = 0; cI < NB; ++cI) {
      T1[cI] = T2[cI] = T3[cI] = 0.0;
      wvs[cI] = wv_[cI] * pole_scale<NB>(sq, cI);
      wts[cI] = wv_[cI] * ts[cI];
      zts[cI] = zc[cI] * ts[cI];
      mts[cI] = mu[cI] * ts[cI];
    }
    each_point<WALK, 1>(spec, fl, SF, [&](double w, double er, double ei) {
        const double w2 = w * w;
        double Rv[NB];
        basis_Rs<NB>(w2, tau2s, sq, Rv);
        double pr = 0.0, pi = 0.0, pz = 0.0, pm = 0.0;
#pragma unroll
        for (int cI = 0; cI < NB; ++cI) {
          pr = __builtin_fma(wvs[cI], Rv[cI], pr);
          pi = __builtin_fma(wts[cI], Rv[cI], pi);
          pz = __builtin_fma(zts[cI], Rv[cI], pz);
          pm = __builtin_fma(mts[cI], Rv[cI], pm);
        }
        const double w2rr = w2 * ((er - einf) - group_sum<SP>(pr));
        const double w2ri = -2.0 * w * __builtin_fma(-w, group_sum<SP>(pi), ei);
        const double wqz = w * __builtin_fma(-w, group_sum<SP>(pz), ei);
        const double wqm = -w2 * group_sum<SP>(pm);
#pragma unroll
        for (int cI = 0; cI < NB; ++cI) {
          const double R = Rv[cI], R2 = R * R;
          const double h = __builtin_fma(2.0 * pole_scale<NB>(sq, cI), R2, -R);
          const double v = __builtin_fma(wts[cI], w2ri, __builtin_fma(mts[cI], wqz, zts[cI] * wqm));
          T1[cI] = __builtin_fma(v, h, T1[cI]);
          T2[cI] = __builtin_fma(w2rr, R2, T2[cI]);
          T3[cI] = __builtin_fma(w2 * R, h, T3[cI]);
        }
    });
#pragma unroll
    for (int cI = 0; cI < NB; ++cI) {
      T1[cI] = __builtin_fma(4.0 * wts[cI] * ts[cI], T2[cI], T1[cI]);
      T1[cI] = __builtin_fma(-2.0 * damping * mts[cI] * zts[cI], T3[cI], T1[cI]);
    }
    freq_sum_n<NB, SP, SP>(T1, SL);
    if (writer && a.grad_theta) {
      // padding entries of the row (poles beyond this material's count) are 0
      if (q == 0)
        for (int64_t p = N; p < a.ld; ++p) a.grad_theta[c * a.ld + p] = 0.0;
#pragma unroll
      for (int cI = 0; cI < NB; ++cI) {
        const int p = pole_of(q, cI);
        if (p < N) a.grad_theta[c * a.ld + p] = st == ST_OK ? gc * (LN10 * T1[cI]) : NAN;
      }
    }
  }
}

// The cost kernel: one tile per 64-lane block.  XCD-aware tile order:
// workgroups are dealt round-robin to the 8 XCDs, so block b runs on XCD
// b % 8 as its (b / 8)-th block.  The plan gives every XCD its own list of
// tiles (whole materials where possible, so that a material's spectra stay in
// one L2; the lists balanced by work, each longest first).  The grid covers
// the longest list; surplus blocks exit.
template <int N, int SP, bool GRAD, int UNI>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(waves_per_simd<N, SP, GRAD, UNI>())))
void fit_kernel(const FitArgs a) {
  const int xcd = blockIdx.x & 7;
  const int64_t j = blockIdx.x >> 3;
  if (j >= a.xcd_off[xcd + 1] - a.xcd_off[xcd]) return;
  fit_tile<N, SP, GRAD, UNI>(a, a.xcd_off[xcd] + j);
}

// The forward kernel with the refinement pass in double-double, general tiles.
template <int N, int SP>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(waves_per_simd<N, SP, false, 0>())))
void fit_dd_kernel(const FitArgs a) {
  const int xcd = blockIdx.x & 7;
  const int64_t j = blockIdx.x >> 3;
  if (j >= a.xcd_off[xcd + 1] - a.xcd_off[xcd]) return;
  fit_tile<N, SP, false, 0, true>(a, a.xcd_off[xcd] + j);
}

// Blocks of a cost-kernel grid: eight times the longest of the 8 XCD tile
// lists (block b runs tile b / 8 of XCD b % 8's list).
inline unsigned fit_grid_blocks(const FitArgs &a) {
  int64_t longest = 0;
  for (int x = 0; x < 8; ++x) longest = a.xcd_off[x + 1] - a.xcd_off[x] > longest ? a.xcd_off[x + 1] - a.xcd_off[x] : longest;
  return (unsigned)(longest * 8);
}

// Launch of the cost kernel for N poles: the adjoint (GRAD) or the forward
// kernel, in the uniform-tile form the plan found (split 1: scalar spectrum
// loads; wider splits: per-lane offsets) or the general one.  The grid covers
// the longest of the 8 XCD tile lists.
template <int N, int SP, bool GRAD> hipError_t launch_fit_split(const FitArgs &a, int64_t n_tiles, bool uni, hipStream_t s) {
  const size_t lds = (size_t)Shape<N, SP>::LDS_DOUBLES * 8 * a.cand_per_wave;
  FitArgs b = a;
  b.n_tiles = n_tiles;
  // (the plan's tiles are the forward kernel's: as many lanes a candidate)
  b.freq_split = a.freq_split * (pole_split_for(N) / SP);
  const unsigned blocks = fit_grid_blocks(a);
  if (blocks == 0) return hipSuccess;
  if (uni && b.freq_split == 1) {
    if constexpr (!Shape<N, SP>::MF)
      hipLaunchKernelGGL((fit_kernel<N, SP, GRAD, 1>), dim3(blocks), dim3(64), lds, s, b);
  } else if (uni)
    hipLaunchKernelGGL((fit_kernel<N, SP, GRAD, 2>), dim3(blocks), dim3(64), lds, s, b);
  else
    hipLaunchKernelGGL((fit_kernel<N, SP, GRAD, 0>), dim3(blocks), dim3(64), lds, s, b);
  return hipGetLastError();
}
template <int N, bool GRAD> hipError_t launch_fit_variant(const FitArgs &a, int64_t n_tiles, bool uni, hipStream_t s) {
  if (GRAD && !a.short_spectra) return launch_fit_split<N, pole_split_long_grad(N), GRAD>(a, n_tiles, uni, s);
  return launch_fit_split<N, pole_split_for(N), GRAD>(a, n_tiles, uni, s);
}

// The forward kernel with the extended-precision refinement: the general
// tile form only (it serves uniform tiles too).
template <int N> hipError_t launch_fit_dd_variant(const FitArgs &a, int64_t n_tiles, hipStream_t s) {
  constexpr int SP = pole_split_for(N);
  const size_t lds = (size_t)Shape<N, SP>::LDS_DOUBLES * 8 * a.cand_per_wave;
  FitArgs b = a;
  b.n_tiles = n_tiles;
  const unsigned blocks = fit_grid_blocks(a);
  if (blocks == 0) return hipSuccess;
  hipLaunchKernelGGL((fit_dd_kernel<N, SP>), dim3(blocks), dim3(64), lds, s, b);
  return hipGetLastError();
}

}  // namespace dfit
