// Target synthesis for the relaxation models of the paper (Sec. II-B):
// Debye (Eq. 3), Havriliak-Negami (Eq. 4) and its Cole-Cole / Cole-Davidson
// special cases, Jonscher (the constant-Q form eps_inf + chi (j w/w_p)^(n-1)),
// CRIM (Eq. 6 with a = 1/2, Debye water in a lossless matrix) and a tabulated
// sum of HN terms with multiplicative Gaussian noise.  eps = eps' - j eps''
// (Eq. 1).  One thread per frequency point; FP64; the complex powers are taken
// on the principal branch in polar form.

#include "common.hpp"
#include "elem.hpp"
#include "rng.hpp"
#include "fit_eval.hpp"

namespace dfit {

// The m in [0, M) with off[m] <= x < off[m + 1] (off ascending; x the same in
// every lane, all 64 lanes together): 64 probes a round, so two rounds reach
// 4,096 materials where a lane's own bisection waits for 12 loads in turn.
__device__ __forceinline__ int wave_owner(const int64_t *off, int32_t M, int64_t x) {
  const int lane = threadIdx.x & 63;
  int lo = 0, hi = M;
  while (hi - lo > 1) {
    const int step = (hi - lo + 63) >> 6;
    const int64_t at = (int64_t)lo + (int64_t)lane * step;
    const int n = __popcll(__builtin_amdgcn_ballot_w64(at < hi && off[at < hi ? at : lo] <= x));
    lo += (n > 0 ? n - 1 : 0) * step;
    hi = lo + step < hi ? lo + step : hi;
  }
  return lo;
}

struct Cx {
  double re, im;
};
__device__ __forceinline__ Cx cmul(Cx a, Cx b) { return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re}; }
__device__ __forceinline__ Cx cscale(Cx a, double s) { return {a.re * s, a.im * s}; }
__device__ __forceinline__ Cx cadd(Cx a, Cx b) { return {a.re + b.re, a.im + b.im}; }
__device__ __forceinline__ Cx cpolar(double mag, double ang) {
  double s, c;
  sincos(ang, &s, &c);
  return {mag * c, mag * s};
}
__device__ __forceinline__ Cx cinv(Cx a) {
  const double d = a.re * a.re + a.im * a.im;
  return {a.re / d, -a.im / d};
}
// principal square root
__device__ __forceinline__ Cx csqrt_p(Cx a) {
  const double r = hypot(a.re, a.im);
  double t = sqrt(0.5 * (r + fabs(a.re)));
  if (t == 0.0) return {0.0, 0.0};
  if (a.re >= 0.0) return {t, a.im / (2.0 * t)};
  return {fabs(a.im) / (2.0 * t), copysign(t, a.im)};
}

// One HN term with its parameter derivatives.  y = w tau0 > 0:
//   (j y)^alpha = y^alpha e^{j pi alpha / 2},  B = 1 + (j y)^alpha = |B| e^{j phi},
//   term = d_eps B^-beta = d_eps |B|^-beta e^{-j beta phi}
struct HnOut {
  Cx val;      // d_eps * B^-beta
  Cx d[5];     // d/d(eps_inf, d_eps, tau0, alpha, beta)
};
// the derivatives, from p = (j y)^alpha, ln y and B^-beta
__device__ __forceinline__ void hn_jac(HnOut &o, double d_eps, double tau0, double alpha, double beta, double ly, Cx p,
                                       Cx B, Cx Bmb, double lB, double phi) {
  const Cx Bmb1 = cmul(Bmb, cinv(B));                 // B^(-beta-1)
  const Cx k = cscale(Bmb1, -beta * d_eps);            // -beta d_eps B^(-beta-1)
  o.d[0] = {1.0, 0.0};
  o.d[1] = Bmb;
  o.d[2] = cmul(k, cscale(p, alpha / tau0));            // dB/dtau0 = alpha p / tau0
  o.d[3] = cmul(k, cmul(p, Cx{ly, 0.5 * M_PI}));        // dB/dalpha = p log(j y)
  o.d[4] = cscale(cmul(Bmb, Cx{lB, phi}), -d_eps);      // -d_eps B^-beta log B
}
// any parameters, by the library's functions
__device__ __noinline__ HnOut hn_term_any(double w, double d_eps, double tau0, double alpha, double beta,
                                          bool want_jac) {
  HnOut o;
  const double y = w * tau0;
  const double ly = log(y);
  const double pa = exp(alpha * ly);                   // y^alpha
  const Cx p = cpolar(pa, 0.5 * M_PI * alpha);         // (j y)^alpha
  const Cx B = {1.0 + p.re, p.im};
  const double lB = log(hypot(B.re, B.im));
  const double phi = atan2(B.im, B.re);
  const Cx Bmb = cpolar(exp(-beta * lB), -beta * phi);  // B^-beta
  o.val = cscale(Bmb, d_eps);
  if (want_jac) hn_jac(o, d_eps, tau0, alpha, beta, ly, p, B, Bmb, lB, phi);
  return o;
}
// 0 < alpha <= 1, so that B lies in the first quadrant with |B| >= 1, and y,
// y^alpha, |B|^2 and |B|^beta inside the double range
__device__ __forceinline__ HnOut hn_term(double w, double d_eps, double tau0, double alpha, double beta,
                                         bool want_jac) {
  const double y = w * tau0;
  if (!(y > 1e-140 && y < 1e140 && alpha > 0.0 && alpha <= 1.0 && fabs(beta) <= 2.0))
    return hn_term_any(w, d_eps, tau0, alpha, beta, want_jac);
  HnOut o;
  const elem::Pair ly = elem::log_pair(y);
  const double pa = elem::exp_prod(alpha, ly);
  Cx p;
  elem::sincos_mid(0.5 * M_PI * alpha, p.im, p.re);
  p = cscale(p, pa);
  const Cx B = {1.0 + p.re, p.im};
  const elem::Pair lB2 = elem::log_pair(__builtin_fma(B.re, B.re, B.im * B.im));   // 2 ln |B|
  const double phi = elem::atan_quot(B.im, B.re);
  Cx Bmb;
  elem::sincos_mid(-beta * phi, Bmb.im, Bmb.re);
  Bmb = cscale(Bmb, elem::exp_prod(-0.5 * beta, lB2));
  o.val = cscale(Bmb, d_eps);
  if (want_jac) hn_jac(o, d_eps, tau0, alpha, beta, ly.hi, p, B, Bmb, 0.5 * lB2.hi, phi);
  return o;
}

// One thread per frequency point; bound by the FP64 pipe (an HN term takes six
// elementary functions, the noise three and a Philox call).  With the library's
// functions 2,048 tables of 4,096 points (two terms and noise each on average)
// took 409 us, with those of elem.hpp 225-245 us (by the machine); 4,096 mixed materials of 1,000
// points 97 and 49 us.  The Jacobian's ten values a point go through LDS, so that
// the block writes its 20 KiB in order (a thread's own 80 bytes, store by store,
// touched 64 lines each; the mixed materials with it 180 us, now 115).
template <bool JAC> __global__ __launch_bounds__(256) void material_kernel(const MaterialArgs a) {
  const int64_t g = (int64_t)blockIdx.x * 256 + threadIdx.x;
  // material owning frequency g: the wave's first point's (its lanes search
  // together), and on from there
  const int64_t first = g - (threadIdx.x & 63);
  const bool live = g < a.n_freq;
  int m = wave_owner(a.f_off, a.M, first < a.n_freq ? first : a.n_freq - 1);
  Cx jac[5];
  bool have_jac = false;
  if (live) {
    while (m + 1 < a.M && a.f_off[m + 1] <= g) ++m;
    const int64_t k = g - a.f_off[m];
    const double *p = a.params + (int64_t)m * 16;
    const int kind = a.kind[m];
    const double w = a.omega[g];
    Cx eps = {0.0, 0.0};
    switch (kind) {
    case 0: case 1: case 2: case 3: {
      const double alpha = (kind == 0 || kind == 3) ? 1.0 : p[3];
      const double beta = (kind == 0 || kind == 2) ? 1.0 : p[4];
      HnOut t = hn_term(w, p[1], p[2], alpha, beta, JAC);
      eps = {p[0] + t.val.re, t.val.im};
      if (JAC) {
        for (int i = 0; i < 5; ++i) jac[i] = t.d[i];
        have_jac = true;
      }
      break;
    }
    case 4: {  // Jonscher: eps_inf + chi (j w / w_p)^(n-1)
      const double y = w / p[2];
      const double e = p[3] - 1.0;
      Cx t;
      if (y > 1e-140 && y < 1e140 && fabs(e) <= 2.0) {
        elem::sincos_mid(0.5 * M_PI * e, t.im, t.re);
        t = cscale(t, p[1] * elem::exp_prod(e, elem::log_pair(y)));
      } else {
        t = cpolar(p[1] * exp(e * log(y)), 0.5 * M_PI * e);
      }
      eps = {p[0] + t.re, t.im};
      break;
    }
    case 5: {  // CRIM, a = 1/2: sqrt(eps) = f sqrt(eps_w) + (1 - f) sqrt(eps_m)
      const double x = w * p[2];
      const double den = 1.0 + x * x;
      const Cx ew = {p[0] + p[1] / den, -p[1] * x / den};
      const Cx sw = csqrt_p(ew);
      const double sm = sqrt(p[4]);
      const Cx root = {p[3] * sw.re + (1.0 - p[3]) * sm, p[3] * sw.im};
      eps = cmul(root, root);
      break;
    }
    case 6: {  // eps_inf + sum of HN terms, times (1 + noise * gaussian)
      const int nt = (int)p[1];
      eps = {p[0], 0.0};
      for (int t = 0; t < nt && t < 3; ++t) {
        HnOut h = hn_term(w, p[2 + 4 * t], p[3 + 4 * t], p[4 + 4 * t], p[5 + 4 * t], false);
        eps = cadd(eps, h.val);
      }
      break;
    }
    default:
      eps = {NAN, NAN};
  }
    double er = eps.re, ei = -eps.im;
    if (kind == 6 && p[14] != 0.0) {
      // Box-Muller on two Philox uniforms (counter (k, 0, 0, noise stream), key (seed, m))
      const U64x4 r = philox4x64((uint64_t)k, 0, 0, STREAM_NOISE, a.noise_seed, (uint64_t)m);
      const double u1 = unit53(r.w[0]), u2 = unit53(r.w[1]);
      const double rad = sqrt(-2.0 * elem::log_pos(1.0 - u1));   // 1 - u1 in [2^-53, 1]
      double s, c;
      elem::sincos_mid(2.0 * M_PI * u2, s, c);
      er = er * (1.0 + p[14] * (rad * c));
      ei = ei * (1.0 + p[14] * (rad * s));
  }
    a.eps_re[g] = er;
    a.eps_im[g] = ei;
  }
  if constexpr (JAC) {
    __shared__ double J[256 * 10];
    if (live) {
#pragma unroll
      for (int i = 0; i < 5; ++i) {
        J[threadIdx.x * 10 + 2 * i] = have_jac ? jac[i].re : NAN;
        J[threadIdx.x * 10 + 2 * i + 1] = have_jac ? -jac[i].im : NAN;
      }
    }
    __syncthreads();
    const int64_t b0 = (int64_t)blockIdx.x * 256;
    const int n = (int)(a.n_freq - b0 < 256 ? a.n_freq - b0 : 256) * 10;
    for (int i = threadIdx.x; i < n; i += 256) a.jac[b0 * 10 + i] = J[i];
  }
}

hipError_t launch_material(const MaterialArgs &a, hipStream_t s) {
  const int64_t blocks = (a.n_freq + 255) / 256;
  if (a.jac) hipLaunchKernelGGL((material_kernel<true>), dim3((unsigned)blocks), dim3(256), 0, s, a);
  else hipLaunchKernelGGL((material_kernel<false>), dim3((unsigned)blocks), dim3(256), 0, s, a);
  return hipGetLastError();
}

// --------------------------------------------------------------------------
// Parameter gradient of HN-family targets: grad_params[m][q] =
//   sum_k J[k][q][0] g_re[k] + J[k][q][1] g_im[k]   (q = eps_inf, d_eps, tau0,
// alpha, beta), one block per material, fixed-order tree reduction.
// --------------------------------------------------------------------------
__global__ __launch_bounds__(256) void material_vjp_kernel(int32_t M, const int64_t *f_off, const double *jac,
                                                          const double *g_re, const double *g_im, double *gp) {
  __shared__ double red[5][256];
  const int tid = threadIdx.x;
  for (int64_t m = blockIdx.x; m < M; m += gridDim.x) {
    const int64_t a = f_off[m], b = f_off[m + 1];
    double acc[5] = {0, 0, 0, 0, 0};
    for (int64_t k = a + tid; k < b; k += blockDim.x) {
      const double *J = jac + k * 10;
      const double gr = g_re[k], gi = g_im[k];
#pragma unroll
      for (int q = 0; q < 5; ++q) acc[q] = __builtin_fma(J[2 * q], gr, __builtin_fma(J[2 * q + 1], gi, acc[q]));
    }
#pragma unroll
    for (int q = 0; q < 5; ++q) red[q][tid] = acc[q];
    __syncthreads();
    for (int w = blockDim.x / 2; w > 0; w >>= 1) {
      if (tid < w)
#pragma unroll
        for (int q = 0; q < 5; ++q) red[q][tid] += red[q][tid + w];
      __syncthreads();
    }
    if (tid < 16) gp[m * 16 + tid] = tid < 5 ? red[tid][0] : 0.0;
    __syncthreads();
  }
}

hipError_t launch_material_vjp(int32_t M, const int64_t *f_off, const double *jac, const double *g_re,
                               const double *g_im, double *gp, hipStream_t s) {
  const int blocks = M < 65536 ? M : 65536;
  hipLaunchKernelGGL(material_vjp_kernel, dim3((unsigned)blocks), dim3(256), 0, s, M, f_off, jac, g_re, g_im, gp);
  return hipGetLastError();
}

// --------------------------------------------------------------------------
// Debye basis materialised for inspection: re/im [n_cand][N][F] (coalesced
// along F).  Bound by the bytes written (16 a value).  A block takes 256 or 512
// points of one (candidate, pole) row, one or two a thread: two, so that 10^theta
// (44 instructions) is raised once for both; one for rows of a single block,
// where a second would only cost registers.  Threads past the row's end leave
// before the power.  With one point a thread, four and two: 1,024 candidates of
// 20 poles and 4,096 points (1.34 GB) 320, 228 and 197 us (6.8 TB/s); of 8 poles
// and 1,000 points (131 MB) 21.3, 21.1 and 20.7; 2,000 of 8 poles and 1,025
// points 42, 54 and 40; 1,024 of 20 poles and 1,000 points 54, 61 and 58.  (A block
// of four points a thread whose threads past the end raised the power too took
// 94 us for 20,000 candidates of 5 poles and 50 points, now 49.)
// --------------------------------------------------------------------------
constexpr int BASIS_POINTS = 2;   // of a thread where a row is longer than a block

template <int POINTS>
__global__ __launch_bounds__(256) void basis_kernel(const double *omega, int64_t F, const double *theta, int64_t ld,
                                                   uint32_t N, double *re, double *im) {
  const int64_t k0 = (int64_t)blockIdx.x * (256 * POINTS) + threadIdx.x;
  if (k0 >= F) return;
  const uint32_t row = blockIdx.y, c = row / N;   // row = c * N + i
  const double tau = exp10(theta[c * ld + (row - c * N)]);
  double *r = re + row * F, *m = im + row * F;
#pragma unroll
  for (int t = 0; t < POINTS; ++t) {
    const int64_t k = k0 + t * 256;
    if (k < F) {
      const double x = omega[k] * tau;
      const double R = rcp_nr(__builtin_fma(x, x, 1.0));
      r[k] = R;
      m[k] = x * R;
    }
  }
}

hipError_t launch_basis(const double *omega, int64_t F, const double *theta, int64_t ld, int64_t n_cand, int32_t N,
                        double *re, double *im, hipStream_t s) {
  const int points = F <= 256 ? 1 : BASIS_POINTS;
  const dim3 blocks((unsigned)((F + 256 * points - 1) / (256 * points)));
  const int64_t per_launch = 65535 / N;   // candidates whose rows fit the grid's second dimension
  for (int64_t c = 0; c < n_cand; c += per_launch) {
    const dim3 grid(blocks.x, (unsigned)((n_cand - c < per_launch ? n_cand - c : per_launch) * N));
    double *r = re + c * N * F, *m = im + c * N * F;
    if (points == 1)
      hipLaunchKernelGGL(basis_kernel<1>, grid, dim3(256), 0, s, omega, F, theta + c * ld, ld, (uint32_t)N, r, m);
    else
      hipLaunchKernelGGL(basis_kernel<BASIS_POINTS>, grid, dim3(256), 0, s, omega, F, theta + c * ld, ld, (uint32_t)N, r, m);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace dfit

namespace dfit {

// --------------------------------------------------------------------------
// Average fractional error of a fitted expansion (the paper's accuracy figure,
// Sec. IV): 100 (mean_k |eps'_k - model'_k| / |eps'_k| + mean_k |eps''_k -
// model''_k| / |eps''_k|), model = eps_inf + sum_i w_i / (1 + j w_k tau_i);
// points with eps'' = 0 are left out of the second mean.  One block of WAVES
// wavefronts per candidate, lanes strided over the frequencies, fixed-order
// reduction.
//
// Bound by the spectra's bytes and, near them, by the FP64 pipe: a pair of poles
// (read from LDS once for four points) shares a reciprocal, and lane i alone
// raises 10 to theta_i.  With each lane forming every tau into scratch memory
// (a run-time pole count) and an IEEE division per pole: 136 us for 4,096
// candidates of 12 poles and 1,000 points (98 MB of spectra), now 33 us.
// --------------------------------------------------------------------------
constexpr int64_t AFE_FEW = 2048;   // candidates that fill the chip with one wave each

struct AfeSums {
  double sr, si, ni;
};
__device__ __forceinline__ void afe_point(double er, double ei, double mr, double mi, AfeSums &s) {
  s.sr += fabs(er - mr) / fabs(er);
  if (ei != 0.0) {
    s.si += fabs(ei - mi) / fabs(ei);
    s.ni += 1.0;
  }
}

struct Pole {
  double tau, w;
};
constexpr int AFE_POINTS = 4;   // of a lane at a time: a pole pair read from LDS serves them all

// N poles in pairs (n2 even, the last padded with weight 0), |log10 tau| <=
// THETA_LIMIT and w < 1e45 rad/s: the product of two 1 + x^2 stays below 1e301
__device__ __forceinline__ void afe_sums(const double *om, const double *epr, const double *epi, int64_t F, int k0,
                                         int stride, const Pole *poles, int n2, double einf, AfeSums &s) {
  for (int64_t k = k0; k < F; k += AFE_POINTS * stride) {
    double o[AFE_POINTS], mr[AFE_POINTS], mi[AFE_POINTS];
#pragma unroll
    for (int t = 0; t < AFE_POINTS; ++t) {
      const int64_t kt = k + t * stride;
      o[t] = om[kt < F ? kt : k];
      mr[t] = einf;
      mi[t] = 0.0;
    }
    for (int i = 0; i < n2; i += 2) {
      const Pole a = poles[i], b = poles[i + 1];
#pragma unroll
      for (int t = 0; t < AFE_POINTS; ++t) {
        const double x0 = o[t] * a.tau, x1 = o[t] * b.tau;
        const double d0 = __builtin_fma(x0, x0, 1.0), d1 = __builtin_fma(x1, x1, 1.0);
        const double r = rcp_nr(d0 * d1);
        const double R0 = d1 * r, R1 = d0 * r;
        mr[t] = __builtin_fma(b.w, R1, __builtin_fma(a.w, R0, mr[t]));
        mi[t] = __builtin_fma(b.w, x1 * R1, __builtin_fma(a.w, x0 * R0, mi[t]));
      }
    }
#pragma unroll
    for (int t = 0; t < AFE_POINTS; ++t) {
      const int64_t kt = k + t * stride;
      if (kt < F) afe_point(epr[kt], epi[kt], mr[t], mi[t], s);
    }
  }
}

template <int WAVES>
__global__ __launch_bounds__(64 * WAVES) void afe_kernel(const AfeArgs a) {
  __shared__ Pole poles[DFIT_MAX_POLES];
  __shared__ AfeSums part[WAVES];
  __shared__ int plain_s;
  const int64_t c = blockIdx.x;
  const int tid = threadIdx.x;
  const int m = wave_owner(a.cand_off, a.M, c);
  const int64_t f0 = a.f_off[m], F = a.f_off[m + 1] - f0;
  const int N = a.n_poles[m];
  if (tid < 64) {
    double t = 0.0, w = 0.0;
    const bool own = tid < N;
    if (own) {
      t = a.theta[c * a.ld + tid];
      w = a.weights[c * a.ld + tid];
    }
    if (tid < DFIT_MAX_POLES) poles[tid] = {own ? exp10(t) : 0.0, w};
    const bool far = __builtin_amdgcn_ballot_w64(own && !(fabs(t) <= THETA_LIMIT)) != 0;
    if (tid == 0) plain_s = far ? 0 : 1;
  }
  __syncthreads();
  const double einf = a.eps_inf[c];
  const double *om = a.omega + f0, *epr = a.eps_re + f0, *epi = a.eps_im + f0;
  AfeSums s = {0.0, 0.0, 0.0};
  if (!plain_s) {   // relaxation times beyond the admissible range (or not numbers): one division a pole
    for (int64_t k = tid; k < F; k += 64 * WAVES) {
      double mr = einf, mi = 0.0;
      for (int i = 0; i < N; ++i) {
        const double x = om[k] * poles[i].tau;
        const double R = 1.0 / __builtin_fma(x, x, 1.0);
        mr = __builtin_fma(poles[i].w, R, mr);
        mi = __builtin_fma(poles[i].w, x * R, mi);
      }
      afe_point(epr[k], epi[k], mr, mi, s);
    }
  } else {
    afe_sums(om, epr, epi, F, tid, 64 * WAVES, poles, (N + 1) & ~1, einf, s);
  }
  for (int off = 32; off > 0; off >>= 1) {
    s.sr += __shfl_xor(s.sr, off, 64);
    s.si += __shfl_xor(s.si, off, 64);
    s.ni += __shfl_xor(s.ni, off, 64);
  }
  if constexpr (WAVES > 1) {
    if ((tid & 63) == 0) part[tid >> 6] = s;
    __syncthreads();
    s = part[0];
    for (int i = 1; i < WAVES; ++i) {
      s.sr += part[i].sr;
      s.si += part[i].si;
      s.ni += part[i].ni;
    }
  }
  if (tid == 0) a.afe[c] = 100.0 * (s.sr / (double)F + (s.ni > 0.0 ? s.si / s.ni : 0.0));
}

// Four wavefronts a candidate where one each would leave SIMDs idle (256 CUs
// of four): 4,096 candidates of 12 poles and 1,000 points 33 us with one, 2,047
// 20 us with four; one candidate of 4,096 points 11 us (94 before).
hipError_t launch_afe(const AfeArgs &a, int64_t n_cand, hipStream_t s) {
  if (n_cand == 0) return hipSuccess;
  if (n_cand > 0x7fffffff) return hipErrorInvalidValue;
  if (n_cand < AFE_FEW) hipLaunchKernelGGL((afe_kernel<4>), dim3((unsigned)n_cand), dim3(256), 0, s, a);
  else hipLaunchKernelGGL((afe_kernel<1>), dim3((unsigned)n_cand), dim3(64), 0, s, a);
  return hipGetLastError();
}

// dst entry e <- the first dst_off[e+1] - dst_off[e] points of the spectra of
// source material src_mat[e] (which has at least that many); one block per entry
__global__ __launch_bounds__(256) void gather_spectra_kernel(const int64_t *src_off, const int32_t *src_mat,
                                                             const int64_t *dst_off, const double *s0,
                                                             const double *s1, const double *s2, double *d0,
                                                             double *d1, double *d2) {
  const int64_t e = blockIdx.x;
  const int32_t m = src_mat[e];
  const int64_t a = src_off[m], b = dst_off[e], F = dst_off[e + 1] - b;
  for (int64_t k = threadIdx.x; k < F; k += blockDim.x) {
    d0[b + k] = s0[a + k];
    d1[b + k] = s1[a + k];
    d2[b + k] = s2[a + k];
  }
}

hipError_t launch_gather_spectra(int64_t n_entries, const int64_t *src_off, const int32_t *src_mat,
                                 const int64_t *dst_off, const double *s0, const double *s1, const double *s2,
                                 double *d0, double *d1, double *d2, hipStream_t s) {
  if (n_entries == 0) return hipSuccess;
  hipLaunchKernelGGL(gather_spectra_kernel, dim3((unsigned)n_entries), dim3(256), 0, s, src_off, src_mat, dst_off, s0,
                     s1, s2, d0, d1, d2);
  return hipGetLastError();
}

// rows: dst[dst_row[e] * dst_ld + i] = src[src_row[e] * src_ld + i], i < n[e]
__global__ __launch_bounds__(64) void scatter_rows_kernel(int64_t n_entries, const int64_t *src_row,
                                                          const int64_t *dst_row, const int32_t *n,
                                                          const double *src, int64_t src_ld, double *dst,
                                                          int64_t dst_ld) {
  const int64_t e = (int64_t)blockIdx.x * 64 + threadIdx.x;
  if (e >= n_entries) return;
  for (int i = 0; i < n[e]; ++i) dst[dst_row[e] * dst_ld + i] = src[src_row[e] * src_ld + i];
}

hipError_t launch_scatter_rows(int64_t n_entries, const int64_t *src_row, const int64_t *dst_row, const int32_t *n,
                               const double *src, int64_t src_ld, double *dst, int64_t dst_ld, hipStream_t s) {
  if (n_entries == 0) return hipSuccess;
  hipLaunchKernelGGL(scatter_rows_kernel, dim3((unsigned)((n_entries + 63) / 64)), dim3(64), 0, s, n_entries, src_row,
                     dst_row, n, src, src_ld, dst, dst_ld);
  return hipGetLastError();
}

}  // namespace dfit
