// C ABI of the Debye fitting library (declared in include/debyefit.h):
// argument validation on the host, launch planning and kernel dispatch.

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <map>
#include <numeric>
#include <string>
#include <vector>

#include "../../include/debyefit.h"
#include "common.hpp"
#include "fit_eval.hpp"

namespace {

thread_local std::string g_error;

int fail(int code, const char *fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_error = buf;
  return code;
}

int hip_fail(hipError_t e, const char *what) {
  return fail(DEBYE_EHIP, "%s: %s", what, hipGetErrorString(e));
}

#define CHECK_HIP(expr, what)                   \
  do {                                          \
    hipError_t e_ = (expr);                     \
    if (e_ != hipSuccess) return hip_fail(e_, what); \
  } while (0)

// Lanes per wave that the schedule tries to keep busy: the GPU has 256 CUs x 4
// SIMDs; at two waves per SIMD a batch needs about 2048 waves to fill it.
constexpr int64_t TARGET_WAVES = 2048;
// Waves of a bucket (one for each SIMD) up to which lanes go below 16 points:
// swarms of 32 particles and 100 points at split 4 and 8, forward (adjoint), us:
// 8 poles at 1,000 waves 22.1 and 16.9 (33.4 and 24.2), 1,280 22.1 and 23.8 (33.4
// and 35.8), 4,000 37 and 44 (56 and 68); 12 poles 36.7 and 33.5 (47.6 and 39.1) at
// 1,000, 37.7 and 41.4 (48.5 and 49.5) at 1,520, 51 and 80 (65 and 97) at 4,000.
constexpr int64_t SHORT_WAVES = 1024;
// LDS budget of one single-wave block: a CU has 160 KiB, and two waves per SIMD
// (eight per CU) need at most 20 KiB each
constexpr int LDS_PER_WAVE = 20 * 1024;
// concurrent streams over which the pole-count buckets of one evaluation are
// spread (one hardware queue each)
constexpr int MAX_STREAMS = 4;

}  // namespace

namespace dfit {
// error text for debye_last_error() from the library's other host files
int set_error(int code, const char *msg) { return fail(code, "%s", msg); }
}  // namespace dfit

struct Bucket {
  int32_t N = 0, SP = 1, SF = 1;
  int32_t lane_sf = 1, cpw = 64;   // frequency lanes per candidate in the kernel (>= SF), candidates per wave
  int64_t n_cands = 0, n_tiles = 0, max_f = 0, work = 0;
  int64_t xcd_off[9] = {};   // tiles of XCD x: xcd_off[x] .. xcd_off[x+1]-1
  bool uni = false;          // split 1 and every tile holds one material: wave-uniform spectra loads
  double flops = 0;          // algorithmic FP64 work of one evaluation of the bucket
  std::vector<int32_t> mats;
  std::vector<float> tile_est;  // estimated duration of each tile (for the persistent launch's order)
  int32_t *d_lane_cand = nullptr, *d_lane_mat = nullptr, *d_mats = nullptr;
};

struct debye_plan {
  int32_t M = 0, max_poles = 0;
  int32_t live = 1;   // one candidate in so many is evaluated
  int64_t n_freq = 0, n_cand = 0;
  std::vector<int64_t> f_off, cand_off;
  std::vector<int32_t> n_poles;
  std::vector<Bucket> buckets;
  std::map<int32_t, int32_t> sf_override;  // N (0 = all) -> frequency split
  std::map<int32_t, int32_t> sf_tuned;     // N -> split measured fastest by debye_plan_autotune
  double *d_record = nullptr;
  int64_t rec_ld = 0;
  // fork/join of the buckets over the caller's stream and side streams: bucket
  // i runs on the caller's (stream_of[i] == 0) or on side[stream_of[i] - 1]
  std::vector<hipStream_t> side;
  std::vector<hipEvent_t> ev_join;
  hipEvent_t ev_fork = nullptr;
  std::vector<int> stream_of;
  // several buckets: how an evaluation is launched (DEBYE_LAUNCH_*), whether
  // the caller fixed it or the autotuner chose it, and the persistent launch's
  // tables
  int32_t launch = DEBYE_LAUNCH_BUCKETS;
  bool launch_fixed = false, launch_tuned = false;
  dfit::RaggedBucket *d_rbuckets = nullptr;
  int64_t *d_items = nullptr;
  int32_t *d_counters = nullptr;
  int64_t item_off[9] = {};
  size_t ragged_lds = 0;
};

namespace {

void free_bucket(Bucket &b) {
  if (b.d_lane_cand) (void)hipFree(b.d_lane_cand);
  if (b.d_lane_mat) (void)hipFree(b.d_lane_mat);
  if (b.d_mats) (void)hipFree(b.d_mats);
  b.d_lane_cand = b.d_lane_mat = b.d_mats = nullptr;
}

// Fewest frequency lanes a candidate can have in the kernel: the four-lane
// pole split sums four points in one matrix instruction.  A narrower split
// set for such a bucket keeps its tiles, each run as several waves.
int min_split(int SP) { return SP == 4 ? 4 : 1; }

int pick_split(const debye_plan &p, const Bucket &b) {
  auto it = p.sf_override.find(b.N);
  if (it == p.sf_override.end()) it = p.sf_override.find(0);
  const int max_sf = 64 / b.SP;
  if (it != p.sf_override.end() && it->second > 0) return std::min(it->second, max_sf);
  auto tuned = p.sf_tuned.find(b.N);
  if (tuned != p.sf_tuned.end()) return std::min(tuned->second, max_sf);
  // smallest power of two that gives TARGET_WAVES waves, without splitting
  // short spectra below 16 points per lane, or 12 where the swarms then still
  // have a wave for each SIMD of one CU (a block runs such a swarm whole: 40
  // particles of 5 poles and 50 points 11.6 us an iteration at split 4, 15.1 at 2,
  // 12.8 at 8, whose fifth wave shares a SIMD) and the bucket at most SHORT_WAVES
  const int64_t avg_f = b.n_cands ? b.work / (b.n_cands * b.N) : 1;
  int64_t most = 0;   // candidates of the largest swarm
  for (int32_t m : b.mats) most = std::max(most, p.cand_off[m + 1] - p.cand_off[m]);
  int sf = min_split(b.SP);
  auto waves = [&](int split) { return (b.n_cands / p.live * b.SP * split + 63) / 64; };
  auto wider = [&]() {
    const int64_t points = avg_f / (2 * sf);
    return points >= 16 || (points >= 12 && most * b.SP * 2 * sf <= 256 && waves(2 * sf) <= SHORT_WAVES);
  };
  while (sf < max_sf && waves(sf) < TARGET_WAVES && wider()) sf *= 2;
  // the SP > 1 path keeps each candidate's normal matrix in LDS: fewer
  // candidates per wave until two waves per SIMD fit
  const int lds = dfit::lds_bytes_per_candidate(b.N);
  while (lds > 0 && sf < max_sf && (64 / (b.SP * sf)) * lds > LDS_PER_WAVE) sf *= 2;
  return sf;
}

// Work tiles of a bucket and their split over the 8 XCDs (host only).  Work
// items are runs of one material's candidates (a material with more than
// 1/32 of the bucket's tiles is cut into pieces, so that a few big swarms
// still spread over the chip); the items, longest tiles first, go one by one
// to the XCD with the least estimated work (LPT), which keeps a material's
// spectra in one L2 and finishes the XCDs together.  Each XCD's candidates
// are packed into tiles in that order (a tile may span two materials of the
// same XCD).  uni: every tile's candidates of one material (and spectra of
// fewer than 2^29 points).
struct Schedule {
  std::vector<int32_t> lane_cand, lane_mat;
  int64_t xcd_off[9] = {};
  bool uni = false;
};

Schedule make_schedule(const int64_t *f_off, const int64_t *cand_off, const std::vector<int32_t> &mats, int N, int SP,
                       int SF) {
  const int cpw = 64 / (SP * SF);
  struct Item {
    int32_t m;
    int64_t c0, c1;   // candidates [c0, c1)
    double tile_t;    // estimated duration of one tile: points per lane plus the solve
  };
  int64_t total_tiles = 0, n_cands = 0;
  for (int32_t m : mats) {
    total_tiles += (cand_off[m + 1] - cand_off[m] + cpw - 1) / cpw;
    n_cands += cand_off[m + 1] - cand_off[m];
  }
  const int64_t max_item = std::max<int64_t>(1, total_tiles / 32) * cpw;  // candidates
  std::vector<Item> items;
  for (int32_t m : mats) {
    const int64_t F = f_off[m + 1] - f_off[m];
    const double t = (double)((F + SF - 1) / SF) + 0.05 * N * N;
    for (int64_t c = cand_off[m]; c < cand_off[m + 1]; c += max_item)
      items.push_back({m, c, std::min(c + max_item, cand_off[m + 1]), t});
  }
  std::stable_sort(items.begin(), items.end(), [](const Item &x, const Item &y) { return x.tile_t > y.tile_t; });
  std::vector<std::vector<int32_t>> xc(8), xm(8);
  double load[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (const Item &it : items) {
    const int x = (int)(std::min_element(load, load + 8) - load);
    load[x] += it.tile_t * (double)(it.c1 - it.c0) / cpw;
    for (int64_t c = it.c0; c < it.c1; ++c) {
      xc[x].push_back((int32_t)c);
      xm[x].push_back(it.m);
    }
  }
  Schedule sc;
  std::vector<int32_t> &lc = sc.lane_cand, &lm = sc.lane_mat;
  lc.reserve(n_cands + 8 * cpw);
  lm.reserve(n_cands + 8 * cpw);
  for (int x = 0; x < 8; ++x) {
    lc.insert(lc.end(), xc[x].begin(), xc[x].end());
    lm.insert(lm.end(), xm[x].begin(), xm[x].end());
    while (lc.size() % cpw) {
      lc.push_back(-1);
      lm.push_back(0);
    }
    sc.xcd_off[x + 1] = (int64_t)lc.size() / cpw;
  }
  const int64_t n_tiles = (int64_t)lc.size() / cpw;
  sc.uni = true;
  for (int32_t m : mats)
    if (f_off[m + 1] - f_off[m] >= ((int64_t)1 << 29)) sc.uni = false;  // 32-bit byte offsets
  for (int64_t t = 0; sc.uni && t < n_tiles; ++t)
    for (int64_t l = t * cpw; l < (t + 1) * cpw; ++l)
      if (lc[l] >= 0 && lm[l] != lm[t * cpw]) {
        sc.uni = false;
        break;
      }
  return sc;
}

int build_tiles(debye_plan &p, Bucket &b) {
  free_bucket(b);
  b.SF = pick_split(p, b);
  b.lane_sf = std::max(b.SF, min_split(b.SP));
  b.cpw = 64 / (b.SP * b.lane_sf);
  const Schedule sc = make_schedule(p.f_off.data(), p.cand_off.data(), b.mats, b.N, b.SP, b.SF);
  for (int x = 0; x < 9; ++x) b.xcd_off[x] = sc.xcd_off[x] * (b.lane_sf / b.SF);
  b.uni = sc.uni;
  const std::vector<int32_t> &lc = sc.lane_cand, &lm = sc.lane_mat;
  b.n_tiles = (int64_t)lc.size() / b.cpw;
  if (b.n_tiles == 0) return DEBYE_OK;
  // estimated tile duration: the longest spectrum of its candidates, per
  // frequency lane, times a per-point cost that follows the kernel's
  // executed instructions (Gram accumulators, basis values, ring moves,
  // the other passes), plus the dense solve
  {
    const int SP = b.SP, NB = (b.N + SP - 1) / SP, D = SP == 2 ? NB : 0;
    // (a matrix instruction takes the pipe for four issue slots)
    const int NG = SP == 1 ? b.N * (b.N + 1) / 2 : SP == 2 ? NB * (D + 1) : 4 * (NB * (NB + 1) / 2);
    const double per_point = NG + 12.0 * NB + 60.0 + (SP > 1 ? 2.0 * D + 24.0 : 0.0);
    b.tile_est.assign(b.n_tiles, 0.0f);
    for (int64_t t = 0; t < b.n_tiles; ++t) {
      int64_t fmax = 0;
      for (int64_t l = t * b.cpw; l < (t + 1) * b.cpw; ++l)
        if (lc[l] >= 0) fmax = std::max(fmax, p.f_off[lm[l] + 1] - p.f_off[lm[l]]);
      b.tile_est[t] = (float)((double)((fmax + b.lane_sf - 1) / b.lane_sf) * per_point + 0.5 * (double)b.N * b.N * b.N);
    }
  }
  if (hipMalloc(&b.d_lane_cand, lc.size() * 4) != hipSuccess || hipMalloc(&b.d_lane_mat, lm.size() * 4) != hipSuccess ||
      hipMalloc(&b.d_mats, b.mats.size() * 4) != hipSuccess)
    return fail(DEBYE_ENOMEM, "plan: device allocation failed");
  CHECK_HIP(hipMemcpy(b.d_lane_cand, lc.data(), lc.size() * 4, hipMemcpyHostToDevice), "plan upload");
  CHECK_HIP(hipMemcpy(b.d_lane_mat, lm.data(), lm.size() * 4, hipMemcpyHostToDevice), "plan upload");
  CHECK_HIP(hipMemcpy(b.d_mats, b.mats.data(), b.mats.size() * 4, hipMemcpyHostToDevice), "plan upload");
  return DEBYE_OK;
}

// Tables of the persistent launch (plans with several pole-count buckets):
// one descriptor per bucket, and per XCD the union of the buckets' tiles of
// that XCD (each bucket's lists are already balanced over the XCDs by work),
// longest estimated duration first.  Rebuilt after every re-tiling.
int build_ragged(debye_plan &p) {
  if (p.d_rbuckets) (void)hipFree(p.d_rbuckets);
  if (p.d_items) (void)hipFree(p.d_items);
  p.d_rbuckets = nullptr;
  p.d_items = nullptr;
  for (int x = 0; x < 9; ++x) p.item_off[x] = 0;
  p.ragged_lds = 0;
  if (p.buckets.size() < 2) return DEBYE_OK;
  std::vector<dfit::RaggedBucket> rb(p.buckets.size());
  std::vector<std::vector<std::pair<float, int64_t>>> per_xcd(8);
  for (size_t i = 0; i < p.buckets.size(); ++i) {
    const Bucket &bk = p.buckets[i];
    rb[i] = dfit::RaggedBucket{bk.N, bk.lane_sf, bk.cpw, bk.uni ? 1 : 0, bk.d_lane_cand, bk.d_lane_mat};
    p.ragged_lds = std::max(p.ragged_lds, (size_t)dfit::lds_bytes_per_candidate(bk.N) * bk.cpw);
    for (int x = 0; x < 8; ++x)
      for (int64_t t = bk.xcd_off[x]; t < bk.xcd_off[x + 1]; ++t)
        per_xcd[x].push_back({bk.tile_est[t], ((int64_t)i << 40) | t});
  }
  std::vector<int64_t> items;
  for (int x = 0; x < 8; ++x) {
    std::stable_sort(per_xcd[x].begin(), per_xcd[x].end(),
                     [](const std::pair<float, int64_t> &u, const std::pair<float, int64_t> &v) { return u.first > v.first; });
    for (const auto &it : per_xcd[x]) items.push_back(it.second);
    p.item_off[x + 1] = (int64_t)items.size();
  }
  if (!p.d_counters && hipMalloc(&p.d_counters, 8 * sizeof(int32_t)) != hipSuccess) {
    p.d_counters = nullptr;
    return fail(DEBYE_ENOMEM, "plan: persistent-launch counters allocation failed");
  }
  if (hipMalloc(&p.d_rbuckets, rb.size() * sizeof(dfit::RaggedBucket)) != hipSuccess ||
      hipMalloc(&p.d_items, std::max<size_t>(items.size(), 1) * 8) != hipSuccess)
    return fail(DEBYE_ENOMEM, "plan: persistent-launch tables allocation failed");
  CHECK_HIP(hipMemcpy(p.d_rbuckets, rb.data(), rb.size() * sizeof(dfit::RaggedBucket), hipMemcpyHostToDevice),
            "plan upload");
  if (!items.empty())
    CHECK_HIP(hipMemcpy(p.d_items, items.data(), items.size() * 8, hipMemcpyHostToDevice), "plan upload");
  return DEBYE_OK;
}

// blocks of the persistent launch: eight one-wave blocks per CU (two waves
// per SIMD), each looping over its XCD's items
constexpr int32_t RAGGED_BLOCKS = 256 * 8;

int check_batch(const debye_batch *b) {
  if (!b) return fail(DEBYE_EINVAL, "batch is NULL");
  if (b->n_mat < 1) return fail(DEBYE_ERANGE, "n_mat must be >= 1 (got %d)", b->n_mat);
  if (b->max_poles < 1 || b->max_poles > DEBYE_MAX_POLES)
    return fail(DEBYE_ERANGE, "max_poles must be in 1..%d (got %d)", DEBYE_MAX_POLES, b->max_poles);
  if (b->n_freq < 1) return fail(DEBYE_ERANGE, "n_freq must be >= 1");
  if (b->n_cand < 0) return fail(DEBYE_ERANGE, "n_cand must be >= 0");
  if (!b->f_off || !b->cand_off || !b->n_poles || !b->omega || !b->eps_re || !b->eps_im)
    return fail(DEBYE_EINVAL, "batch has a NULL device pointer");
  return DEBYE_OK;
}

int check_plan_batch(const debye_plan *p, const debye_batch *b, int64_t ld) {
  if (!p) return fail(DEBYE_EINVAL, "plan is NULL");
  int rc = check_batch(b);
  if (rc) return rc;
  if (b->n_mat != p->M || b->n_cand != p->n_cand || b->n_freq != p->n_freq || b->max_poles != p->max_poles)
    return fail(DEBYE_EINVAL, "batch shape does not match the plan (M %d/%d, candidates %lld/%lld, points %lld/%lld)",
                b->n_mat, p->M, (long long)b->n_cand, (long long)p->n_cand, (long long)b->n_freq, (long long)p->n_freq);
  if (ld < p->max_poles) return fail(DEBYE_ERANGE, "ld (%lld) < max_poles (%d)", (long long)ld, p->max_poles);
  return DEBYE_OK;
}

static_assert((unsigned)DEBYE_FLAG_NO_SIGN_FLIP == (unsigned)dfit::FLAG_NO_SIGN_FLIP &&
                  (unsigned)DEBYE_FLAG_NO_REFINE == (unsigned)dfit::FLAG_NO_REFINE &&
                  (unsigned)DEBYE_FLAG_DD_REFINE == (unsigned)dfit::FLAG_DD_REFINE,
              "the kernels read the ABI's flag bits");

int check_damping(double damping, uint32_t flags) {
  if (!(damping >= 0.0) || !std::isfinite(damping)) return fail(DEBYE_ERANGE, "damping must be finite and >= 0");
  if (flags & ~(uint32_t)(DEBYE_FLAG_NO_SIGN_FLIP | DEBYE_FLAG_NO_REFINE | DEBYE_FLAG_DD_REFINE))
    return fail(DEBYE_EINVAL, "unknown flag bits 0x%x", flags);
  if ((flags & DEBYE_FLAG_NO_REFINE) && (flags & DEBYE_FLAG_DD_REFINE))
    return fail(DEBYE_EINVAL, "DEBYE_FLAG_NO_REFINE and DEBYE_FLAG_DD_REFINE exclude each other");
  return DEBYE_OK;
}

// the adjoint kernels and the polish have no double-double refinement
int check_grad_flags(uint32_t flags) {
  if (flags & DEBYE_FLAG_DD_REFINE)
    return fail(DEBYE_EINVAL, "DEBYE_FLAG_DD_REFINE is for forward evaluations only");
  return DEBYE_OK;
}

dfit::FitArgs fit_args(const debye_plan *p, const Bucket &bk, const debye_batch *b, const double *theta, int64_t ld,
                       double damping, uint32_t flags) {
  dfit::FitArgs a{};
  a.f_off = b->f_off;
  a.omega = b->omega;
  a.eps_re = b->eps_re;
  a.eps_im = b->eps_im;
  a.theta = theta;
  a.ld = ld;
  a.damping = damping;
  a.flags = flags;
  a.freq_split = bk.lane_sf;
  a.cand_per_wave = bk.cpw;
  a.short_spectra = bk.work <= dfit::SHORT_SPECTRA * bk.n_cands * bk.N;
  a.lane_cand = bk.d_lane_cand;
  a.lane_mat = bk.d_lane_mat;
  for (int x = 0; x < 9; ++x) a.xcd_off[x] = bk.xcd_off[x];
  (void)p;
  return a;
}

// ---- optimiser runs ----
// How a run's evaluations are launched.  A small iteration over several pole
// counts is bound by its launches, their fork and their join, so a run whose
// caller left that to the library (use_graph, no launch mode set or tuned)
// takes one persistent launch, with the same results, from four pole counts on
// up to RUN_TILES tiles a pole count on average.  A generation of differential
// evolution with a launch a bucket and with one for all: 3 pole counts 61 and 61
// us at 24 tiles, 61 and 65 at 768; 4 pole counts 77 and 65 at 32, 78 and 70 at
// 1,024, 78 and 94 at 2,048; 12 pole counts 132 and 101 at 104, 139 and 136 at
// 3,328, 224 and 232 at 6,656; 24 pole counts 274 and 158 at 456, 407 and 666 at
// 14,592.
constexpr int64_t RUN_TILES = 256;
int32_t run_launch(const debye_plan *p, int32_t use_graph) {
  const int64_t counts = (int64_t)p->buckets.size();
  if (!use_graph || p->launch_fixed || p->launch_tuned || counts < 4) return p->launch;
  int64_t tiles = 0;
  for (const Bucket &b : p->buckets) tiles += b.n_tiles;
  return tiles <= RUN_TILES * counts ? DEBYE_LAUNCH_PERSISTENT : p->launch;
}

// use_graph on a stream under capture is refused
int check_run_stream(int32_t use_graph, hipStream_t s) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (use_graph && hipStreamIsCapturing(s, &st) != hipSuccess) (void)hipGetLastError();
  return st == hipStreamCaptureStatusNone ? DEBYE_OK
                                          : fail(DEBYE_EHIP, "use_graph must be 0 on a stream under capture");
}

// Enqueue launch(bucket, stream) for every non-empty bucket.  With several
// buckets some fork from `stream` onto the plan's side streams and join back,
// so different pole counts overlap on the GPU; under stream capture the fork
// and join become parallel branches of the graph.  The caller's stream takes its
// share: each side stream costs the host a wait, a record and a wait more (with
// all buckets on side streams a generation over 2 pole counts took 57 us, now
// 42, over 9 123 and 103, over 24 391 and 226).
template <class LAUNCH> int for_buckets(const debye_plan *p, hipStream_t stream, LAUNCH &&launch) {
  const int n_side = (int)p->side.size();
  if (n_side) CHECK_HIP(hipEventRecord(p->ev_fork, stream), "fork event");
  for (int j = 0; j < n_side; ++j) CHECK_HIP(hipStreamWaitEvent(p->side[j], p->ev_fork, 0), "fork wait");
  int rc = DEBYE_OK;
  for (size_t i = 0; i < p->buckets.size() && rc == DEBYE_OK; ++i) {
    const int j = n_side ? p->stream_of[i] : 0;
    if (p->buckets[i].n_tiles) rc = launch(p->buckets[i], j ? p->side[j - 1] : stream);
  }
  // join every side stream, also after a failed launch, so no capture is left open
  for (int j = 0; j < n_side; ++j) {
    CHECK_HIP(hipEventRecord(p->ev_join[j], p->side[j]), "join event");
    CHECK_HIP(hipStreamWaitEvent(stream, p->ev_join[j], 0), "join wait");
  }
  return rc;
}

}  // namespace

namespace {
int fit_eval_impl(const debye_plan *p, const debye_batch *b, const double *log10_tau, int64_t ld, double damping,
                  uint32_t flags, double *cost, double *weights, double *eps_inf, int8_t *status,
                  const int32_t *skip_mat, int32_t launch, hipStream_t stream);
}  // namespace

extern "C" {

const char *debye_last_error(void) { return g_error.c_str(); }
const char *debye_version(void) { return "debyefit 0.1 (gfx950, FP64)"; }

// live: one candidate in so many is evaluated (the others' waves exit at once)
static int plan_create(const debye_batch *shape, const int64_t *f_off_host, const int64_t *cand_off_host,
                       const int32_t *n_poles_host, uint32_t flags, int32_t live, debye_plan **out) {
  if (!out) return fail(DEBYE_EINVAL, "out is NULL");
  *out = nullptr;
  int rc = check_batch(shape);
  if (rc) return rc;
  if (!f_off_host || !cand_off_host || !n_poles_host) return fail(DEBYE_EINVAL, "host shape arrays are NULL");
  if (flags & ~(uint32_t)DEBYE_PLAN_TARGET_GRAD) return fail(DEBYE_EINVAL, "unknown plan flag bits 0x%x", flags);
  const int32_t M = shape->n_mat;
  if (f_off_host[0] != 0 || cand_off_host[0] != 0) return fail(DEBYE_EINVAL, "offsets must start at 0");
  int32_t maxN = 0;
  for (int32_t m = 0; m < M; ++m) {
    if (f_off_host[m + 1] - f_off_host[m] < 1)
      return fail(DEBYE_ERANGE, "material %d has %lld frequency points (need >= 1)", m,
                  (long long)(f_off_host[m + 1] - f_off_host[m]));
    if (cand_off_host[m + 1] < cand_off_host[m]) return fail(DEBYE_EINVAL, "cand_off is decreasing at %d", m);
    if (n_poles_host[m] < 1 || n_poles_host[m] > DEBYE_MAX_POLES)
      return fail(DEBYE_ERANGE, "material %d: n_poles %d outside 1..%d", m, n_poles_host[m], DEBYE_MAX_POLES);
    maxN = std::max(maxN, n_poles_host[m]);
  }
  if (f_off_host[M] != shape->n_freq || cand_off_host[M] != shape->n_cand)
    return fail(DEBYE_EINVAL, "n_freq / n_cand do not match the offsets");
  if (maxN != shape->max_poles) return fail(DEBYE_EINVAL, "max_poles (%d) != max of n_poles (%d)", shape->max_poles, maxN);
  if (cand_off_host[M] > INT32_MAX) return fail(DEBYE_ERANGE, "more than 2^31-1 candidates");

  debye_plan *p = new debye_plan();
  p->M = M;
  p->live = live;
  p->max_poles = maxN;
  p->n_freq = shape->n_freq;
  p->n_cand = shape->n_cand;
  p->f_off.assign(f_off_host, f_off_host + M + 1);
  p->cand_off.assign(cand_off_host, cand_off_host + M + 1);
  p->n_poles.assign(n_poles_host, n_poles_host + M);
  std::map<int32_t, Bucket> by_n;
  for (int32_t m = 0; m < M; ++m) {
    const int64_t P = cand_off_host[m + 1] - cand_off_host[m];
    if (P == 0) continue;
    Bucket &b = by_n[n_poles_host[m]];
    b.N = n_poles_host[m];
    b.SP = dfit::pole_split(b.N);
    b.mats.push_back(m);
    b.n_cands += P;
    const int64_t F = f_off_host[m + 1] - f_off_host[m];
    b.max_f = std::max(b.max_f, F);
    b.work += P * F * b.N;
    b.flops += (double)P * ((double)F * (b.N * b.N + 13.0 * b.N + 5.0) + b.N * b.N * (b.N / 3.0 + 2.0));
  }
  for (auto &kv : by_n) p->buckets.push_back(std::move(kv.second));
  // per-candidate adjoint records for the target gradient (set-up, so that
  // debye_fit_eval_grad itself never allocates)
  if (flags & DEBYE_PLAN_TARGET_GRAD) {
    p->rec_ld = 4 * p->max_poles + 2;   // [w | z | mu | tau | eps_inf, gc]
    if (hipMalloc(&p->d_record, (size_t)std::max<int64_t>(p->n_cand, 1) * p->rec_ld * 8) != hipSuccess) {
      p->d_record = nullptr;
      debye_plan_destroy(p);
      return fail(DEBYE_ENOMEM, "plan: adjoint record allocation failed");
    }
  }
  // largest work first
  std::stable_sort(p->buckets.begin(), p->buckets.end(), [](const Bucket &x, const Bucket &y) { return x.flops > y.flops; });
  for (auto &b : p->buckets) {
    rc = build_tiles(*p, b);
    if (rc) {
      debye_plan_destroy(p);
      return rc;
    }
  }
  if ((rc = build_ragged(*p))) {
    debye_plan_destroy(p);
    return rc;
  }
  // several pole counts: the buckets run concurrently on the caller's stream
  // and side streams, each bucket (largest first) on the one with the least
  // work so far
  const int n_side = std::min<int>(MAX_STREAMS, (int)p->buckets.size()) - 1;
  if (n_side > 0) {
    p->side.assign(n_side, nullptr);
    p->ev_join.assign(n_side, nullptr);
    bool ok = hipEventCreateWithFlags(&p->ev_fork, hipEventDisableTiming) == hipSuccess;
    for (int j = 0; j < n_side && ok; ++j)
      ok = hipStreamCreateWithFlags(&p->side[j], hipStreamNonBlocking) == hipSuccess &&
           hipEventCreateWithFlags(&p->ev_join[j], hipEventDisableTiming) == hipSuccess;
    if (!ok) {
      debye_plan_destroy(p);
      return fail(DEBYE_EHIP, "plan: stream or event creation failed");
    }
    std::vector<double> load(n_side + 1, 0.0);
    for (const Bucket &b : p->buckets) {
      const int j = (int)(std::min_element(load.begin(), load.end()) - load.begin());
      p->stream_of.push_back(j);
      load[j] += b.flops;
    }
  }
  *out = p;
  return DEBYE_OK;
}

int debye_plan_create(const debye_batch *shape, const int64_t *f_off_host, const int64_t *cand_off_host,
                      const int32_t *n_poles_host, uint32_t flags, debye_plan **out) {
  return plan_create(shape, f_off_host, cand_off_host, n_poles_host, flags, 1, out);
}

int debye_plan_destroy(debye_plan *p) {
  if (!p) return DEBYE_OK;
  for (hipStream_t st : p->side)
    if (st) (void)hipStreamSynchronize(st);
  for (auto &b : p->buckets) free_bucket(b);
  if (p->d_record) (void)hipFree(p->d_record);
  if (p->d_rbuckets) (void)hipFree(p->d_rbuckets);
  if (p->d_items) (void)hipFree(p->d_items);
  if (p->d_counters) (void)hipFree(p->d_counters);
  for (hipStream_t st : p->side)
    if (st) (void)hipStreamDestroy(st);
  for (hipEvent_t ev : p->ev_join)
    if (ev) (void)hipEventDestroy(ev);
  if (p->ev_fork) (void)hipEventDestroy(p->ev_fork);
  delete p;
  return DEBYE_OK;
}

int debye_plan_set_freq_split(debye_plan *p, int32_t n_poles, int32_t split) {
  if (!p) return fail(DEBYE_EINVAL, "plan is NULL");
  if (split < 0 || split > 64 || (split & (split - 1))) return fail(DEBYE_ERANGE, "split must be 0 or a power of two <= 64");
  if (split == 0) p->sf_override.erase(n_poles);
  else p->sf_override[n_poles] = split;
  for (auto &b : p->buckets) {
    int rc = build_tiles(*p, b);
    if (rc) return rc;
  }
  return build_ragged(*p);
}

int debye_plan_set_launch(debye_plan *p, int32_t mode) {
  if (!p) return fail(DEBYE_EINVAL, "plan is NULL");
  if (mode != DEBYE_LAUNCH_AUTO && mode != DEBYE_LAUNCH_BUCKETS && mode != DEBYE_LAUNCH_PERSISTENT)
    return fail(DEBYE_EINVAL, "unknown launch mode %d", mode);
  p->launch_fixed = mode != DEBYE_LAUNCH_AUTO;
  p->launch_tuned = false;
  const int32_t m = mode == DEBYE_LAUNCH_AUTO ? DEBYE_LAUNCH_BUCKETS : mode;
  p->launch = m;
  return DEBYE_OK;
}

int debye_plan_get_launch(const debye_plan *p) {
  if (!p) return fail(DEBYE_EINVAL, "plan is NULL");
  return p->buckets.size() > 1 ? p->launch : DEBYE_LAUNCH_BUCKETS;
}

int debye_plan_autotune(debye_plan *p, const debye_batch *b, const double *log10_tau, int64_t ld, double damping,
                        uint32_t flags, int32_t reps, hipStream_t stream) {
  int rc = check_plan_batch(p, b, ld);
  if (rc) return rc;
  if ((rc = check_damping(damping, flags))) return rc;
  if (!log10_tau) return fail(DEBYE_EINVAL, "log10_tau is NULL");
  if (reps < 1 || reps > 100) return fail(DEBYE_ERANGE, "reps must be in 1..100");
  double *cost = nullptr;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  auto cleanup = [&](int r) {
    (void)hipStreamSynchronize(stream);
    if (cost) (void)hipFree(cost);
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    return r;
  };
  if (hipMalloc(&cost, (size_t)std::max<int64_t>(p->n_cand, 1) * 8) != hipSuccess)
    return cleanup(fail(DEBYE_ENOMEM, "autotune: cost buffer allocation failed"));
  if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess)
    return cleanup(fail(DEBYE_EHIP, "autotune: event creation failed"));
  // time `reps` launches of a bucket at its current schedule
  auto time_bucket = [&](Bucket &bk, int n, float *ms) -> int {
    dfit::FitArgs a = fit_args(p, bk, b, log10_tau, ld, damping, flags);
    a.cost = cost;
    hipError_t e = hipEventRecord(e0, stream);
    for (int r = 0; r < n && e == hipSuccess; ++r) e = dfit::launch_fit(bk.N, a, bk.n_tiles, false, bk.uni, stream);
    if (e == hipSuccess) e = hipEventRecord(e1, stream);
    if (e == hipSuccess) e = hipEventSynchronize(e1);
    if (e == hipSuccess) e = hipEventElapsedTime(ms, e0, e1);
    return e == hipSuccess ? DEBYE_OK : hip_fail(e, "autotune launch");
  };
  for (Bucket &bk : p->buckets) {
    if (!bk.n_cands || p->sf_override.count(bk.N) || p->sf_override.count(0)) continue;
    const int64_t avg_f = bk.work / (bk.n_cands * bk.N);
    std::vector<int> splits;
    for (int sf = min_split(bk.SP); sf <= 64 / bk.SP; sf *= 2) {
      if (sf > min_split(bk.SP) && avg_f / sf < 8) break;
      splits.push_back(sf);
    }
    // bring the clocks up first (about 30 ms of this bucket's work), so that
    // the first split timed is not penalised
    float ms = 0;
    p->sf_tuned[bk.N] = splits[0];
    if ((rc = build_tiles(*p, bk)) || (rc = time_bucket(bk, 1, &ms))) return cleanup(rc);
    const int warm = std::min(200, std::max(1, (int)(30.0f / std::max(ms, 0.01f))));
    if ((rc = time_bucket(bk, warm, &ms))) return cleanup(rc);
    // three rounds over the splits, the best time of each (box-to-box and
    // run-to-run spread is a few percent, about the margin between splits)
    std::vector<float> best(splits.size(), INFINITY);
    for (int round = 0; round < 3; ++round)
      for (size_t i = 0; i < splits.size(); ++i) {
        p->sf_tuned[bk.N] = splits[i];
        if ((rc = build_tiles(*p, bk)) || (rc = time_bucket(bk, reps, &ms))) return cleanup(rc);
        best[i] = std::min(best[i], ms);
      }
    // a wider split must win clearly (3 %): it costs reductions, and timing
    // noise should not flip the schedule between runs
    size_t pick = 0;
    for (size_t i = 1; i < splits.size(); ++i)
      if (best[i] < 0.97f * best[pick]) pick = i;
    p->sf_tuned[bk.N] = splits[pick];
    if ((rc = build_tiles(*p, bk))) return cleanup(rc);
  }
  if ((rc = build_ragged(*p))) return cleanup(rc);
  // several buckets: the forked per-bucket launches against the one
  // persistent launch, whole evaluations on the tuned tiles (three rounds,
  // the best of each; the persistent launch must win by 3 %)
  if (p->buckets.size() > 1 && !p->launch_fixed) {
    auto time_eval = [&](int32_t mode, int n, float *ms) -> int {
      p->launch = mode;
      hipError_t e = hipEventRecord(e0, stream);
      int r = DEBYE_OK;
      for (int k = 0; k < n && r == DEBYE_OK && e == hipSuccess; ++k)
        r = debye_fit_eval(p, b, log10_tau, ld, damping, flags, cost, nullptr, nullptr, nullptr, stream);
      if (r) return r;
      if (e == hipSuccess) e = hipEventRecord(e1, stream);
      if (e == hipSuccess) e = hipEventSynchronize(e1);
      if (e == hipSuccess) e = hipEventElapsedTime(ms, e0, e1);
      return e == hipSuccess ? DEBYE_OK : hip_fail(e, "autotune launch");
    };
    float best[2] = {INFINITY, INFINITY}, ms = 0;
    const int32_t modes[2] = {DEBYE_LAUNCH_BUCKETS, DEBYE_LAUNCH_PERSISTENT};
    for (int m = 0; m < 2; ++m)
      if ((rc = time_eval(modes[m], 1, &ms))) return cleanup(rc);
    for (int round = 0; round < 3; ++round)
      for (int m = 0; m < 2; ++m) {
        if ((rc = time_eval(modes[m], reps, &ms))) return cleanup(rc);
        best[m] = std::min(best[m], ms);
      }
    p->launch = best[1] < 0.97f * best[0] ? DEBYE_LAUNCH_PERSISTENT : DEBYE_LAUNCH_BUCKETS;
    p->launch_tuned = true;
  }
  return cleanup(DEBYE_OK);
}

int debye_schedule_preview(const int64_t *f_off, const int64_t *cand_off, const int32_t *mats, int32_t n_mats,
                           int32_t n_poles, int32_t pole_split, int32_t freq_split, int32_t *lane_cand,
                           int32_t *lane_mat, int64_t capacity, int64_t *xcd_off, int32_t *uniform) {
  if (!f_off || !cand_off || (n_mats > 0 && !mats) || !xcd_off || !uniform)
    return fail(DEBYE_EINVAL, "NULL pointer");
  if (n_mats < 0 || n_poles < 1 || n_poles > DEBYE_MAX_POLES || (pole_split != 1 && pole_split != 2 && pole_split != 4) ||
      freq_split < 1 || freq_split * pole_split > 64 || (freq_split & (freq_split - 1)))
    return fail(DEBYE_ERANGE, "schedule preview: bad sizes");
  const std::vector<int32_t> ms(mats, mats + n_mats);
  const Schedule sc = make_schedule(f_off, cand_off, ms, n_poles, pole_split, freq_split);
  for (int x = 0; x < 9; ++x) xcd_off[x] = sc.xcd_off[x];
  *uniform = sc.uni ? 1 : 0;
  const int64_t n = (int64_t)sc.lane_cand.size();
  if (lane_cand && lane_mat) {
    if (capacity < n) return fail(DEBYE_ERANGE, "schedule preview: capacity %lld < %lld slots", (long long)capacity,
                                  (long long)n);
    std::copy(sc.lane_cand.begin(), sc.lane_cand.end(), lane_cand);
    std::copy(sc.lane_mat.begin(), sc.lane_mat.end(), lane_mat);
  }
  return (int)std::min<int64_t>(n, INT32_MAX);
}

int debye_plan_info(const debye_plan *p, int32_t i, int32_t *n_poles, int32_t *pole_split, int32_t *freq_split,
                    int64_t *n_tiles, int32_t *uniform) {
  if (!p) return fail(DEBYE_EINVAL, "plan is NULL");
  if (i < 0) return (int)p->buckets.size();
  if (i >= (int)p->buckets.size()) return fail(DEBYE_ERANGE, "bucket index out of range");
  const Bucket &b = p->buckets[i];
  if (n_poles) *n_poles = b.N;
  if (pole_split) *pole_split = b.SP;
  if (freq_split) *freq_split = b.SF;
  if (n_tiles) *n_tiles = b.n_tiles;
  if (uniform) *uniform = b.uni ? 1 : 0;
  return DEBYE_OK;
}

int debye_afe(const debye_batch *b, const double *log10_tau, int64_t ld, const double *weights, const double *eps_inf,
              double *afe, hipStream_t stream) {
  int rc = check_batch(b);
  if (rc) return rc;
  if (ld < b->max_poles) return fail(DEBYE_ERANGE, "ld < max_poles");
  if (!log10_tau || !weights || !eps_inf || !afe) return fail(DEBYE_EINVAL, "NULL pointer");
  if (b->n_cand > INT32_MAX) return fail(DEBYE_ERANGE, "more than 2^31-1 candidates");
  dfit::AfeArgs a{b->n_mat, b->f_off, b->cand_off, b->n_poles, b->omega, b->eps_re, b->eps_im,
                  log10_tau, weights, eps_inf, ld, afe};
  CHECK_HIP(dfit::launch_afe(a, b->n_cand, stream), "debye_afe launch");
  return DEBYE_OK;
}

int debye_basis(const double *omega, int64_t F, const double *log10_tau, int64_t ld, int64_t n_cand, int32_t N,
                double *re, double *im, hipStream_t stream) {
  if (!omega || !log10_tau || !re || !im) return fail(DEBYE_EINVAL, "NULL pointer");
  if (F < 1 || N < 1 || N > DEBYE_MAX_POLES || n_cand < 0) return fail(DEBYE_ERANGE, "bad size (F %lld, N %d)", (long long)F, N);
  if (ld < N) return fail(DEBYE_ERANGE, "ld < N");
  if (n_cand == 0) return DEBYE_OK;
  CHECK_HIP(dfit::launch_basis(omega, F, log10_tau, ld, n_cand, N, re, im, stream), "debye_basis launch");
  return DEBYE_OK;
}

int debye_fit_eval(const debye_plan *p, const debye_batch *b, const double *log10_tau, int64_t ld, double damping,
                   uint32_t flags, double *cost, double *weights, double *eps_inf, int8_t *status, hipStream_t stream) {
  return fit_eval_impl(p, b, log10_tau, ld, damping, flags, cost, weights, eps_inf, status, nullptr,
                       p ? p->launch : DEBYE_LAUNCH_BUCKETS, stream);
}

}  // extern "C"

namespace {
// debye_fit_eval with an optional mask of materials to leave out ([M],
// nonzero = skip: waves holding only such candidates exit at once and their
// outputs are left as they were), in the given launch mode
int fit_eval_impl(const debye_plan *p, const debye_batch *b, const double *log10_tau, int64_t ld, double damping,
                  uint32_t flags, double *cost, double *weights, double *eps_inf, int8_t *status,
                  const int32_t *skip_mat, int32_t launch, hipStream_t stream) {
  int rc = check_plan_batch(p, b, ld);
  if (rc) return rc;
  if ((rc = check_damping(damping, flags))) return rc;
  if (!log10_tau || !cost) return fail(DEBYE_EINVAL, "log10_tau and cost must not be NULL");
  if (launch == DEBYE_LAUNCH_PERSISTENT && p->buckets.size() > 1 && !(flags & DEBYE_FLAG_DD_REFINE)) {
    // one launch over every bucket, on the caller's stream
    dfit::RaggedArgs r{};
    r.common = fit_args(p, p->buckets[0], b, log10_tau, ld, damping, flags);
    r.common.cost = cost;
    r.common.weights = weights;
    r.common.eps_inf = eps_inf;
    r.common.status = status;
    r.common.skip_mat = skip_mat;
    r.buckets = p->d_rbuckets;
    r.items = p->d_items;
    for (int x = 0; x < 9; ++x) r.item_off[x] = p->item_off[x];
    r.counters = p->d_counters;
    CHECK_HIP(dfit::launch_fit_ragged(r, RAGGED_BLOCKS, p->ragged_lds, stream), "debye_fit_eval persistent launch");
    return DEBYE_OK;
  }
  return for_buckets(p, stream, [&](const Bucket &bk, hipStream_t s) -> int {
    dfit::FitArgs a = fit_args(p, bk, b, log10_tau, ld, damping, flags);
    a.cost = cost;
    a.weights = weights;
    a.eps_inf = eps_inf;
    a.status = status;
    a.skip_mat = skip_mat;
    CHECK_HIP(dfit::launch_fit(bk.N, a, bk.n_tiles, false, bk.uni, s), "debye_fit_eval launch");
    return DEBYE_OK;
  });
}
}  // namespace

namespace {
// cost + adjoint launches of every bucket; `record` ([n_cand][rec_ld]
// doubles) holds the per-candidate adjoint records the target-gradient
// kernel reads back (NULL without target gradients)
int fit_eval_grad_launch(const debye_plan *p, const debye_batch *b, const double *log10_tau, int64_t ld,
                         double damping, uint32_t flags, const double *grad_cost, double *cost,
                         double *grad_log10_tau, double *grad_eps_re, double *grad_eps_im, int8_t *status,
                         double *record, int64_t rec_ld, hipStream_t stream, const int32_t *skip_mat = nullptr) {
  const bool targets = grad_eps_re != nullptr;
  if (targets) {
    // materials without candidates get zero target gradients (a fill kernel,
    // not a memset, so that the call can be captured into a graph)
    CHECK_HIP(dfit::launch_fill(grad_eps_re, p->n_freq, 0.0, stream), "fill");
    CHECK_HIP(dfit::launch_fill(grad_eps_im, p->n_freq, 0.0, stream), "fill");
  }
  return for_buckets(p, stream, [&](const Bucket &bk, hipStream_t s) -> int {
    dfit::FitArgs a = fit_args(p, bk, b, log10_tau, ld, damping, flags);
    a.cost = cost;
    a.status = status;
    a.grad_cost = grad_cost;
    a.grad_theta = grad_log10_tau;
    a.record = targets ? record : nullptr;
    a.rec_ld = rec_ld;
    a.skip_mat = targets ? nullptr : skip_mat;
    CHECK_HIP(dfit::launch_fit(bk.N, a, bk.n_tiles, true, bk.uni, s), "debye_fit_eval_grad launch");
    if (!targets) return DEBYE_OK;
    dfit::TargetGradArgs t{};
    t.f_off = b->f_off;
    t.cand_off = b->cand_off;
    t.omega = b->omega;
    t.eps_re = b->eps_re;
    t.eps_im = b->eps_im;
    t.theta = log10_tau;
    t.ld = ld;
    t.record = record;
    t.rec_ld = rec_ld;
    t.mat_list = bk.d_mats;
    t.grad_re = grad_eps_re;
    t.grad_im = grad_eps_im;
    // the bucket's materials only: disjoint from the other buckets' points
    CHECK_HIP(dfit::launch_target_grad(bk.N, t, bk.max_f, (int32_t)bk.mats.size(), s), "target gradient launch");
    return DEBYE_OK;
  });
}

int fit_eval_grad_check(const debye_plan *p, const debye_batch *b, const double *log10_tau, int64_t ld,
                        double damping, uint32_t flags, const double *cost, const double *grad_eps_re,
                        const double *grad_eps_im) {
  int rc = check_plan_batch(p, b, ld);
  if (rc) return rc;
  if ((rc = check_damping(damping, flags))) return rc;
  if ((rc = check_grad_flags(flags))) return rc;
  if (!log10_tau || !cost) return fail(DEBYE_EINVAL, "log10_tau and cost must not be NULL");
  if ((grad_eps_re == nullptr) != (grad_eps_im == nullptr))
    return fail(DEBYE_EINVAL, "grad_eps_re and grad_eps_im must both be set or both be NULL");
  return DEBYE_OK;
}

}  // namespace

namespace dfit {
// debye_fit_eval_grad with the target-gradient records in a buffer the caller
// provides: after the argument checks, and only when target gradients are
// requested, `record_buffer` is asked for a device buffer of at least the
// bytes the batch needs ([n_cand][4 max_poles + 2] doubles); it returns
// DEBYE_OK and the address, or an error code (e.g. DEBYE_ERANGE when it is
// too small).  Nothing is allocated here.
int fit_eval_grad_external(const debye_plan *p, const debye_batch *b, const double *log10_tau, int64_t ld,
                           double damping, uint32_t flags, const double *grad_cost, double *cost,
                           double *grad_log10_tau, double *grad_eps_re, double *grad_eps_im, int8_t *status,
                           int (*record_buffer)(size_t bytes, double **out), hipStream_t stream) {
  int rc = fit_eval_grad_check(p, b, log10_tau, ld, damping, flags, cost, grad_eps_re, grad_eps_im);
  if (rc) return rc;
  if (!grad_eps_re)
    return fit_eval_grad_launch(p, b, log10_tau, ld, damping, flags, grad_cost, cost, grad_log10_tau, nullptr,
                                nullptr, status, nullptr, 0, stream);
  const int64_t rec_ld = 4 * (int64_t)p->max_poles + 2;
  double *rec = nullptr;
  if ((rc = record_buffer((size_t)std::max<int64_t>(p->n_cand, 1) * (size_t)rec_ld * 8, &rec))) return rc;
  return fit_eval_grad_launch(p, b, log10_tau, ld, damping, flags, grad_cost, cost, grad_log10_tau, grad_eps_re,
                              grad_eps_im, status, rec, rec_ld, stream);
}
}  // namespace dfit

namespace {
// A swarm fit whose batch cannot fill the chip is bound by its launches: where
// every material's block is resident at once it runs as one launch, a block a
// material (swarm.hip), whose wavefronts, up to one a SIMD, take all of the
// material's tiles at once.  One-lane candidates only (N <= 11): the tiles of
// several lanes keep too much in LDS for a swarm's state to join them.
//
// Resident blocks of a CU, by what they measured against the steps (us an
// iteration, one launch and step by step): from 6 poles on a wavefront a SIMD
// (the kernel's registers allow no second), 1,024 materials of 3 particles, N = 8,
// F = 50 16 and 23, 1,400 31 and 25; 256 of 64 particles, F = 100 23 and 30, 300
// 45 and 42; of 3 particles, F = 2,000 (three wavefronts) 30 and 38, 60 and 38.
// Up to 5 poles two a SIMD: N = 5, 512 materials of 64 particles, F = 100 26 and
// 32, 700 38 and 40, 1,400 72 and 64; blocks of one wavefront, which do not wait
// for each other's rounds, up to three a SIMD: 3,000 materials of 3 particles, F =
// 50 25 and 30, 4,096 32 and 33, 10,000 94 and 56.
int64_t swarm_blocks(int N, int waves, int64_t lds) {
  const int64_t by_waves = N > 5 ? 4 / waves : waves == 1 ? 12 : 8 / waves;
  return std::min<int64_t>(by_waves, 160 * 1024 / (lds + 1024));   // (beside its static arrays)
}

// wavefronts of a block for the materials of bucket bk (0: step by step), the
// LDS of the largest one's state and of the block
int swarm_waves(const debye_plan &p, const Bucket &bk, int64_t *state, int64_t *lds) {
  int64_t most = 0;
  *state = 0;
  if (bk.N > dfit::SWARM_POLES) return 0;
  for (int32_t m : bk.mats) {
    const int64_t P = p.cand_off[m + 1] - p.cand_off[m], F = p.f_off[m + 1] - p.f_off[m];
    if (P > INT16_MAX || F > INT16_MAX) return 0;   // (their state is far beyond the LDS)
    most = std::max(most, (P + bk.cpw - 1) / bk.cpw);
    *state = std::max(*state, dfit::swarm_state_bytes(P, bk.N, F));
  }
  const int64_t per_wave = std::max<int64_t>(1, (int64_t)dfit::lds_bytes_per_candidate(bk.N) * bk.cpw);
  *lds = most * per_wave + *state;
  return most <= dfit::SWARM_WAVES && *lds <= dfit::SWARM_LDS ? (int)most : 0;
}

bool swarm_in_one_launch(const debye_plan &p, uint32_t flags) {
  if (p.launch != DEBYE_LAUNCH_BUCKETS || (flags & DEBYE_FLAG_DD_REFINE)) return false;
  for (int32_t m = 0; m < p.M; ++m)
    if (p.cand_off[m + 1] == p.cand_off[m]) return false;   // a swarm without particles
  double share = 0.0;   // of the chip's 256 CUs that the blocks of all buckets take
  for (const Bucket &bk : p.buckets) {
    int64_t state, lds;
    const int waves = swarm_waves(p, bk, &state, &lds);
    if (waves == 0) return false;
    share += (double)bk.mats.size() / (256.0 * (double)swarm_blocks(bk.N, waves, lds));
  }
  return share > 0.0 && share <= 1.0;
}
}  // namespace

extern "C" {

int debye_fit_eval_grad(const debye_plan *p, const debye_batch *b, const double *log10_tau, int64_t ld,
                        double damping, uint32_t flags, const double *grad_cost, double *cost,
                        double *grad_log10_tau, double *grad_eps_re, double *grad_eps_im, int8_t *status,
                        hipStream_t stream) {
  int rc = fit_eval_grad_check(p, b, log10_tau, ld, damping, flags, cost, grad_eps_re, grad_eps_im);
  if (rc) return rc;
  if (grad_eps_re && !p->d_record)
    return fail(DEBYE_EINVAL, "target gradients need a plan created with DEBYE_PLAN_TARGET_GRAD");
  return fit_eval_grad_launch(p, b, log10_tau, ld, damping, flags, grad_cost, cost, grad_log10_tau, grad_eps_re,
                              grad_eps_im, status, p->d_record, p->rec_ld, stream);
}

int debye_material_eval(int32_t M, const int8_t *kind, const double *params, const int64_t *f_off, int64_t n_freq,
                        const double *omega, uint64_t noise_seed, double *eps_re, double *eps_im, double *jac,
                        hipStream_t stream) {
  if (M < 1) return fail(DEBYE_ERANGE, "M must be >= 1");
  if (n_freq < 1) return fail(DEBYE_ERANGE, "n_freq must be >= 1");
  if (!kind || !params || !f_off || !omega || !eps_re || !eps_im) return fail(DEBYE_EINVAL, "NULL pointer");
  dfit::MaterialArgs a{M, kind, params, f_off, n_freq, omega, noise_seed, eps_re, eps_im, jac};
  CHECK_HIP(dfit::launch_material(a, stream), "debye_material_eval launch");
  return DEBYE_OK;
}

int debye_material_vjp(int32_t M, const int64_t *f_off, int64_t n_freq, const double *jac, const double *grad_re,
                       const double *grad_im, double *grad_params, hipStream_t stream) {
  if (M < 1) return fail(DEBYE_ERANGE, "M must be >= 1");
  if (n_freq < 1) return fail(DEBYE_ERANGE, "n_freq must be >= 1");
  if (!f_off || !jac || !grad_re || !grad_im || !grad_params) return fail(DEBYE_EINVAL, "NULL pointer");
  CHECK_HIP(dfit::launch_material_vjp(M, f_off, jac, grad_re, grad_im, grad_params, stream), "debye_material_vjp launch");
  return DEBYE_OK;
}

static int pso_check(const debye_batch *b, int64_t ld, const double *lb, const double *ub, debye_pso_params p) {
  int rc = check_batch(b);
  if (rc) return rc;
  if (ld < b->max_poles) return fail(DEBYE_ERANGE, "ld < max_poles");
  if (!lb || !ub) return fail(DEBYE_EINVAL, "lb/ub are NULL");
  if (!std::isfinite(p.inertia) || !std::isfinite(p.c1) || !std::isfinite(p.c2))
    return fail(DEBYE_ERANGE, "PSO coefficients must be finite");
  return DEBYE_OK;
}

int debye_pso_init(const debye_batch *b, int64_t ld, const double *lb, const double *ub, debye_pso_params p, double *x,
                   double *v, double *pbest_x, double *pbest_cost, double *gbest_cost, int64_t *gbest_idx,
                   hipStream_t stream) {
  int rc = pso_check(b, ld, lb, ub, p);
  if (rc) return rc;
  if (!x || !v || !pbest_x || !pbest_cost || !gbest_cost || !gbest_idx) return fail(DEBYE_EINVAL, "NULL state pointer");
  dfit::PsoArgs a{};
  a.M = b->n_mat;
  a.cand_off = b->cand_off;
  a.n_poles = b->n_poles;
  a.ld = ld;
  a.lb = lb;
  a.ub = ub;
  a.seed = p.seed;
  a.x = x;
  a.v = v;
  a.pbest_x = pbest_x;
  a.pbest_cost = pbest_cost;
  a.gbest_cost = gbest_cost;
  a.gbest_idx = gbest_idx;
  CHECK_HIP(dfit::launch_pso_init(a, b->n_cand, stream), "debye_pso_init launch");
  return DEBYE_OK;
}

int debye_pso_step(const debye_batch *b, int64_t ld, const double *lb, const double *ub, debye_pso_params p, int32_t t,
                   int32_t move, const double *cost, double *x, double *v, double *pbest_x, double *pbest_cost,
                   double *gbest_x, double *gbest_cost, int64_t *gbest_idx, double *history, int64_t hist_ld,
                   hipStream_t stream) {
  int rc = pso_check(b, ld, lb, ub, p);
  if (rc) return rc;
  if (t < 1) return fail(DEBYE_ERANGE, "iteration t must be >= 1");
  if (history && hist_ld < t) return fail(DEBYE_ERANGE, "hist_ld (%lld) < t (%d)", (long long)hist_ld, t);
  if (!cost || !x || !v || !pbest_x || !pbest_cost || !gbest_x || !gbest_cost || !gbest_idx)
    return fail(DEBYE_EINVAL, "NULL state pointer");
  dfit::PsoArgs a{};
  a.M = b->n_mat;
  a.cand_off = b->cand_off;
  a.n_poles = b->n_poles;
  a.ld = ld;
  a.lb = lb;
  a.ub = ub;
  a.inertia = p.inertia;
  a.c1 = p.c1;
  a.c2 = p.c2;
  a.seed = p.seed;
  a.t = t;
  a.move = move ? 1 : 0;
  a.cost = cost;
  a.x = x;
  a.v = v;
  a.pbest_x = pbest_x;
  a.pbest_cost = pbest_cost;
  a.gbest_x = gbest_x;
  a.gbest_cost = gbest_cost;
  a.gbest_idx = gbest_idx;
  a.history = history;
  a.hist_ld = hist_ld;
  CHECK_HIP(dfit::launch_pso_step(a, stream), "debye_pso_step launch");
  return DEBYE_OK;
}

static dfit::PsoArgs pso_args(const debye_batch *b, int64_t ld, const double *lb, const double *ub, debye_pso_params p,
                               int32_t t, int32_t move, const debye_swarm *sw) {
  dfit::PsoArgs a{};
  a.M = b->n_mat;
  a.cand_off = b->cand_off;
  a.n_poles = b->n_poles;
  a.ld = ld;
  a.lb = lb;
  a.ub = ub;
  a.inertia = p.inertia;
  a.c1 = p.c1;
  a.c2 = p.c2;
  a.seed = p.seed;
  a.t = t;
  a.move = move;
  a.cost = sw->cost;
  a.x = sw->x;
  a.v = sw->v;
  a.pbest_x = sw->pbest_x;
  a.pbest_cost = sw->pbest_cost;
  a.gbest_x = sw->gbest_x;
  a.gbest_cost = sw->gbest_cost;
  a.gbest_idx = sw->gbest_idx;
  a.history = sw->history;
  a.hist_ld = sw->hist_ld;
  return a;
}

int debye_pso_run(const debye_plan *plan, const debye_batch *b, int64_t ld, const double *lb, const double *ub,
                  debye_pso_params p, int32_t iters, double damping, uint32_t flags, const debye_swarm *sw,
                  int32_t use_graph, hipStream_t stream) {
  int rc = check_plan_batch(plan, b, ld);
  if (rc) return rc;
  if ((rc = check_damping(damping, flags))) return rc;
  if ((rc = pso_check(b, ld, lb, ub, p))) return rc;
  if (!sw || !sw->x || !sw->v || !sw->pbest_x || !sw->pbest_cost || !sw->gbest_x || !sw->gbest_cost ||
      !sw->gbest_idx || !sw->cost)
    return fail(DEBYE_EINVAL, "NULL swarm pointer");
  if (iters < 0) return fail(DEBYE_ERANGE, "iters must be >= 0");
  if (sw->history && sw->hist_ld < (int64_t)iters + 1) return fail(DEBYE_ERANGE, "hist_ld must be >= iters + 1");
  if ((rc = check_run_stream(use_graph, stream))) return rc;
  if (swarm_in_one_launch(*plan, flags))
    return for_buckets(plan, stream, [&](const Bucket &bk, hipStream_t bs) -> int {
      dfit::FitArgs fa = fit_args(plan, bk, b, sw->x, ld, damping, flags);
      fa.cost = sw->cost;
      fa.status = sw->status;
      int64_t state, lds;
      const int waves = swarm_waves(*plan, bk, &state, &lds);
      CHECK_HIP(dfit::launch_swarm(bk.N, fa, pso_args(b, ld, lb, ub, p, 0, 1, sw), bk.d_mats, (int32_t)bk.mats.size(),
                                   waves, (int32_t)state, iters, bs),
                "swarm launch");
      return DEBYE_OK;
    });
  const int32_t launch = run_launch(plan, use_graph);
  auto eval = [&]() {
    return fit_eval_impl(plan, b, sw->x, ld, damping, flags, sw->cost, nullptr, nullptr, sw->status, nullptr, launch,
                         stream);
  };
  CHECK_HIP(dfit::launch_pso_init(pso_args(b, ld, lb, ub, p, 0, 0, sw), b->n_cand, stream), "swarm init");
  if ((rc = eval())) return rc;
  for (int32_t t = 1; t <= iters; ++t) {
    CHECK_HIP(dfit::launch_pso_step(pso_args(b, ld, lb, ub, p, t, 1, sw), stream), "swarm step");
    if ((rc = eval())) return rc;
  }
  CHECK_HIP(dfit::launch_pso_step(pso_args(b, ld, lb, ub, p, iters + 1, 0, sw), stream), "final bests");
  return DEBYE_OK;
}

// ---- differential evolution ----
static int de_check(const debye_batch *b, int64_t ld, const double *lb, const double *ub, debye_de_params p) {
  int rc = check_batch(b);
  if (rc) return rc;
  if (ld < b->max_poles) return fail(DEBYE_ERANGE, "ld < max_poles");
  if (!lb || !ub) return fail(DEBYE_EINVAL, "lb/ub are NULL");
  if (!(p.f_lo >= 0.0 && p.f_lo <= p.f_hi && p.f_hi <= 2.0) || !(p.cr >= 0.0 && p.cr <= 1.0))
    return fail(DEBYE_ERANGE, "DE parameters out of range (0 <= f_lo <= f_hi <= 2, 0 <= cr <= 1)");
  return DEBYE_OK;
}

static dfit::DeArgs de_args(const debye_batch *b, int64_t ld, const double *lb, const double *ub, debye_de_params p,
                            int32_t t) {
  dfit::DeArgs a{};
  a.M = b->n_mat;
  a.cand_off = b->cand_off;
  a.n_poles = b->n_poles;
  a.ld = ld;
  a.lb = lb;
  a.ub = ub;
  a.f_lo = p.f_lo;
  a.f_hi = p.f_hi;
  a.cr = p.cr;
  a.seed = p.seed;
  a.t = t;
  return a;
}

int debye_de_init(const debye_batch *b, int64_t ld, const double *lb, const double *ub, debye_de_params p, double *x,
                  double *fit, double *best_cost, int64_t *best_idx, hipStream_t stream) {
  int rc = de_check(b, ld, lb, ub, p);
  if (rc) return rc;
  if (!x || !fit || !best_cost || !best_idx) return fail(DEBYE_EINVAL, "NULL population pointer");
  dfit::DeArgs a = de_args(b, ld, lb, ub, p, 0);
  a.x = x;
  a.fit = fit;
  a.best_cost = best_cost;
  a.best_idx = best_idx;
  CHECK_HIP(dfit::launch_de_init(a, b->n_cand, stream), "DE init");
  return DEBYE_OK;
}

int debye_de_trial(const debye_batch *b, int64_t ld, const double *lb, const double *ub, debye_de_params p, int32_t t,
                   const double *x, double *u, hipStream_t stream) {
  int rc = de_check(b, ld, lb, ub, p);
  if (rc) return rc;
  if (!x || !u) return fail(DEBYE_EINVAL, "NULL population pointer");
  if (t < 1) return fail(DEBYE_ERANGE, "generation must be >= 1");
  dfit::DeArgs a = de_args(b, ld, lb, ub, p, t);
  a.x = const_cast<double *>(x);
  a.u = u;
  CHECK_HIP(dfit::launch_de_trial(a, b->n_cand, stream), "DE trial");
  return DEBYE_OK;
}

int debye_de_select(const debye_batch *b, int64_t ld, int32_t t, const double *u, const double *cost_u, double *x,
                    double *fit, double *best_x, double *best_cost, int64_t *best_idx, double *history,
                    int64_t hist_ld, hipStream_t stream) {
  int rc = check_batch(b);
  if (rc) return rc;
  if (ld < b->max_poles) return fail(DEBYE_ERANGE, "ld < max_poles");
  if (!u || !cost_u || !x || !fit || !best_x || !best_cost || !best_idx) return fail(DEBYE_EINVAL, "NULL pointer");
  if (t < 0 || (history && hist_ld <= t)) return fail(DEBYE_ERANGE, "generation must be >= 0 and < hist_ld");
  dfit::DeArgs a = de_args(b, ld, nullptr, nullptr, debye_de_params{0, 0, 0, 0}, t);
  a.u = const_cast<double *>(u);
  a.cost_u = cost_u;
  a.x = x;
  a.fit = fit;
  a.best_x = best_x;
  a.best_cost = best_cost;
  a.best_idx = best_idx;
  a.history = history;
  a.hist_ld = hist_ld;
  CHECK_HIP(dfit::launch_de_select(a, stream), "DE select");
  return DEBYE_OK;
}

int debye_de_run(const debye_plan *plan, const debye_batch *b, int64_t ld, const double *lb, const double *ub,
                 debye_de_params p, int32_t iters, double damping, uint32_t flags, const debye_population *pop,
                 int32_t use_graph, hipStream_t stream) {
  int rc = check_plan_batch(plan, b, ld);
  if (rc) return rc;
  if ((rc = check_damping(damping, flags))) return rc;
  if ((rc = de_check(b, ld, lb, ub, p))) return rc;
  if (!pop || !pop->x || !pop->u || !pop->fit || !pop->cost || !pop->best_x || !pop->best_cost || !pop->best_idx)
    return fail(DEBYE_EINVAL, "NULL population pointer");
  if (iters < 0) return fail(DEBYE_ERANGE, "iters must be >= 0");
  if (pop->history && pop->hist_ld < (int64_t)iters + 1) return fail(DEBYE_ERANGE, "hist_ld must be >= iters + 1");
  if ((rc = check_run_stream(use_graph, stream))) return rc;
  const int32_t launch = run_launch(plan, use_graph);
  auto eval = [&](const double *x) {
    return fit_eval_impl(plan, b, x, ld, damping, flags, pop->cost, nullptr, nullptr, pop->status, nullptr, launch,
                         stream);
  };
  auto sel = [&](int32_t t) {
    dfit::DeArgs a = de_args(b, ld, lb, ub, p, t);
    a.u = pop->u;
    a.cost_u = pop->cost;
    a.x = pop->x;
    a.fit = pop->fit;
    a.best_x = pop->best_x;
    a.best_cost = pop->best_cost;
    a.best_idx = pop->best_idx;
    a.history = pop->history;
    a.hist_ld = pop->hist_ld;
    return a;
  };
  dfit::DeArgs a0 = sel(0);
  CHECK_HIP(dfit::launch_de_init(a0, b->n_cand, stream), "DE init");
  // generation 0: the initial population is its own trial set
  if ((rc = eval(pop->x))) return rc;
  CHECK_HIP(hipMemcpyAsync(pop->u, pop->x, (size_t)b->n_cand * ld * 8, hipMemcpyDeviceToDevice, stream), "copy");
  CHECK_HIP(dfit::launch_de_select(a0, stream), "DE select");
  for (int32_t t = 1; t <= iters; ++t) {
    const dfit::DeArgs a = sel(t);
    CHECK_HIP(dfit::launch_de_trial(a, b->n_cand, stream), "DE trial");
    if ((rc = eval(pop->u))) return rc;
    CHECK_HIP(dfit::launch_de_select(a, stream), "DE select");
  }
  return DEBYE_OK;
}

// ---- annealing ----
static int da_check(const debye_batch *b, int64_t ld, debye_da_params p) {
  int rc = check_batch(b);
  if (rc) return rc;
  if (ld < b->max_poles) return fail(DEBYE_ERANGE, "ld < max_poles");
  if (!(p.qv > 1.0 && p.qv < 3.0) || !(p.qa < 1.0) || !(p.t0 > 0.0) || !std::isfinite(p.t0) || !std::isfinite(p.qa))
    return fail(DEBYE_ERANGE, "annealing parameters out of range (1 < qv < 3, qa < 1, t0 > 0)");
  return DEBYE_OK;
}

static dfit::DaArgs da_args(const debye_batch *b, int64_t ld, const double *lb, const double *ub, debye_da_params p,
                            int32_t t) {
  dfit::DaArgs a{};
  a.M = b->n_mat;
  a.cand_off = b->cand_off;
  a.n_poles = b->n_poles;
  a.ld = ld;
  a.lb = lb;
  a.ub = ub;
  a.qv = p.qv;
  a.qa = p.qa;
  a.t0 = p.t0;
  a.seed = p.seed;
  a.t = t;
  return a;
}

int debye_da_init(const debye_batch *b, int64_t ld, const double *lb, const double *ub, debye_da_params p, double *x,
                  double *fit, double *best_cost, int64_t *best_idx, hipStream_t stream) {
  int rc = da_check(b, ld, p);
  if (rc) return rc;
  if (!lb || !ub || !x || !fit || !best_cost || !best_idx) return fail(DEBYE_EINVAL, "NULL pointer");
  dfit::DaArgs a = da_args(b, ld, lb, ub, p, 0);
  a.x = x;
  a.fit = fit;
  a.best_cost = best_cost;
  a.best_idx = best_idx;
  CHECK_HIP(dfit::launch_da_init(a, b->n_cand, stream), "annealing init");
  return DEBYE_OK;
}

int debye_da_visit(const debye_batch *b, int64_t ld, const double *lb, const double *ub, debye_da_params p, int32_t t,
                   const double *x, double *y, hipStream_t stream) {
  int rc = da_check(b, ld, p);
  if (rc) return rc;
  if (!lb || !ub || !x || !y) return fail(DEBYE_EINVAL, "NULL pointer");
  if (t < 1) return fail(DEBYE_ERANGE, "generation must be >= 1");
  dfit::DaArgs a = da_args(b, ld, lb, ub, p, t);
  a.x = const_cast<double *>(x);
  a.u = y;
  CHECK_HIP(dfit::launch_da_visit(a, b->n_cand, stream), "annealing visit");
  return DEBYE_OK;
}

int debye_da_accept(const debye_batch *b, int64_t ld, debye_da_params p, int32_t t, const double *y,
                    const double *cost_y, double *x, double *fit, double *best_x, double *best_cost, int64_t *best_idx,
                    double *history, int64_t hist_ld, hipStream_t stream) {
  int rc = da_check(b, ld, p);
  if (rc) return rc;
  if (!y || !cost_y || !x || !fit || !best_x || !best_cost || !best_idx) return fail(DEBYE_EINVAL, "NULL pointer");
  if (t < 0 || (history && hist_ld <= t)) return fail(DEBYE_ERANGE, "generation must be >= 0 and < hist_ld");
  dfit::DaArgs a = da_args(b, ld, nullptr, nullptr, p, t);
  a.u = const_cast<double *>(y);
  a.cost_u = cost_y;
  a.x = x;
  a.fit = fit;
  a.best_x = best_x;
  a.best_cost = best_cost;
  a.best_idx = best_idx;
  a.history = history;
  a.hist_ld = hist_ld;
  CHECK_HIP(dfit::launch_da_accept(a, stream), "annealing accept");
  return DEBYE_OK;
}

int debye_da_run(const debye_plan *plan, const debye_batch *b, int64_t ld, const double *lb, const double *ub,
                 debye_da_params p, int32_t iters, double damping, uint32_t flags, const debye_population *pop,
                 int32_t use_graph, hipStream_t stream) {
  int rc = check_plan_batch(plan, b, ld);
  if (rc) return rc;
  if ((rc = check_damping(damping, flags))) return rc;
  if ((rc = da_check(b, ld, p))) return rc;
  if (!lb || !ub) return fail(DEBYE_EINVAL, "lb/ub are NULL");
  if (!pop || !pop->x || !pop->u || !pop->fit || !pop->cost || !pop->best_x || !pop->best_cost || !pop->best_idx)
    return fail(DEBYE_EINVAL, "NULL population pointer");
  if (iters < 0) return fail(DEBYE_ERANGE, "iters must be >= 0");
  if (pop->history && pop->hist_ld < (int64_t)iters + 1) return fail(DEBYE_ERANGE, "hist_ld must be >= iters + 1");
  if ((rc = check_run_stream(use_graph, stream))) return rc;
  const int32_t launch = run_launch(plan, use_graph);
  auto eval = [&](const double *x) {
    return fit_eval_impl(plan, b, x, ld, damping, flags, pop->cost, nullptr, nullptr, pop->status, nullptr, launch,
                         stream);
  };
  auto args = [&](int32_t t) {
    dfit::DaArgs a = da_args(b, ld, lb, ub, p, t);
    a.u = pop->u;
    a.cost_u = pop->cost;
    a.x = pop->x;
    a.fit = pop->fit;
    a.best_x = pop->best_x;
    a.best_cost = pop->best_cost;
    a.best_idx = pop->best_idx;
    a.history = pop->history;
    a.hist_ld = pop->hist_ld;
    return a;
  };
  dfit::DaArgs a0 = args(0);
  CHECK_HIP(dfit::launch_da_init(a0, b->n_cand, stream), "annealing init");
  if ((rc = eval(pop->x))) return rc;
  CHECK_HIP(hipMemcpyAsync(pop->u, pop->x, (size_t)b->n_cand * ld * 8, hipMemcpyDeviceToDevice, stream), "copy");
  CHECK_HIP(dfit::launch_da_accept(a0, stream), "annealing accept");
  for (int32_t t = 1; t <= iters; ++t) {
    const dfit::DaArgs a = args(t);
    CHECK_HIP(dfit::launch_da_visit(a, b->n_cand, stream), "annealing visit");
    if ((rc = eval(pop->u))) return rc;
    CHECK_HIP(dfit::launch_da_accept(a, stream), "annealing accept");
  }
  return DEBYE_OK;
}

// ---- L-BFGS polish: a context that owns the workspace and the plans (one
// candidate per material for the gradient, and those of the line search's
// stages), so that the calls below only enqueue work

// Trials a material of the line search's stages.  A stage costs a launch that
// is bound by latency up to a few thousand candidates, so few materials try
// many halvings at once; 30 trials are tried 2, 4, 8 and 16 at a time from 911
// to 1,024 materials and 1, 5, 8 and 16 beyond, each stage for the materials still
// undecided.  (2, 4, 8 and 16 beyond as well is no clear gain: per step, 2 steps,
// 1,100 materials of 8 poles and 500 points 176 and 171 us, 4,096 317 and 304,
// 65,536 of 200 points 1,953 and 2,007, 1,100 of 12 poles and 2,000 points 574 and
// 590; 20 steps 146 and 146, 254 and 254, 1,652 and 1,681, 498 and 542.)  Per
// step, 20 steps from a swarm's best (POLISH_FILL 512, 1,024, 2,048, 4,096): 256
// materials of 8 poles and 500 points 149, 136, 114, 112 us, 64 of 10 poles and
// 1,000 points 136, 130, 98, 98; 512 of 20 poles and 3,000 points 841, 835, 732,
// 844.
constexpr int32_t POLISH_FILL = 2048;
void polish_stages(int32_t M, int32_t T, int32_t *end) {
  constexpr int LAST = dfit::LBFGS_STAGES - 1;
  int32_t n[LAST + 1] = {}, left = T;
  for (int s = 0; s <= LAST; ++s) {
    n[s] = std::min(left, std::max(s == 0 ? 1 : 2 << s, (POLISH_FILL << s) / M));
    left -= n[s];
    if (s == LAST || left < n[s] / 2) {   // no short stage for the rest
      n[left >= n[s] / 2 ? LAST : n[1] > 0] += left;
      break;
    }
  }
  for (int s = 0; s < dfit::LBFGS_STAGES; ++s) end[s] = (s ? end[s - 1] : 0) + n[s];
}
// About one candidate in so many is still evaluated in a stage: its frequencies
// are split as widely as for so many fewer, else a few wavefronts each run long.
// Per step, 20 steps from a swarm's best, with all of them counted and so: 1,024
// materials of 12 poles and 2,000 points 929 and 505 us, 8,192 of 6 poles and 500
// points 921 and 367.
constexpr int32_t POLISH_LIVE[dfit::LBFGS_STAGES] = {1, 4, 8, 16};

struct debye_polish {
  int32_t M = 0, max_poles = 0, mem = 0, max_trials = 0, steps = 0;
  int32_t stage_end[dfit::LBFGS_STAGES] = {};
  int64_t ld = 0, n_freq = 0;
  double c1 = 0;
  debye_plan *p1 = nullptr, *trials[dfit::LBFGS_STAGES] = {};   // (NULL: no trials in the stage)
  void *ws = nullptr;         // one allocation for every buffer below
  int64_t *offs = nullptr;    // [M+1] candidate offsets of each stage
  double *grad, *S, *Y, *rho, *dir, *gd, *trial_theta, *trial_cost, *new_theta, *new_cost, *new_grad, *cost, *acc_cost;
  int32_t *hist_n, *hist_head, *accepted, *done, *stalled;
  int8_t *trial_status, *new_status;
};

namespace {
int polish_check(const debye_polish *pp, const debye_batch *b, double damping, uint32_t flags) {
  if (!pp) return fail(DEBYE_EINVAL, "polish context is NULL");
  int rc = check_batch(b);
  if (rc) return rc;
  if (b->n_mat != pp->M || b->n_cand != pp->M || b->n_freq != pp->n_freq || b->max_poles != pp->max_poles)
    return fail(DEBYE_EINVAL, "batch does not match the polish context (one candidate per material)");
  if ((rc = check_damping(damping, flags))) return rc;
  return check_grad_flags(flags);
}

dfit::LbfgsArgs polish_args(const debye_polish *pp, const debye_batch *b, double *theta, const double *lb,
                            const double *ub, double *cost_hist) {
  dfit::LbfgsArgs la{};
  la.M = pp->M;
  la.n_poles = b->n_poles;
  la.ld = pp->ld;
  la.mem = pp->mem;
  la.max_trials = pp->max_trials;
  std::copy(pp->stage_end, pp->stage_end + dfit::LBFGS_STAGES, la.stage_end);
  la.c1 = pp->c1;
  la.lb = lb;
  la.ub = ub;
  la.theta = theta;
  la.cost = pp->cost;
  la.acc_cost = pp->acc_cost;
  la.grad = pp->grad;
  la.S = pp->S;
  la.Y = pp->Y;
  la.rho = pp->rho;
  la.hist_n = pp->hist_n;
  la.hist_head = pp->hist_head;
  la.dir = pp->dir;
  la.gd = pp->gd;
  la.trial_theta = pp->trial_theta;
  la.trial_cost = pp->trial_cost;
  la.trial_status = pp->trial_status;
  la.done = pp->done;
  la.stalled = pp->stalled;
  la.new_theta = pp->new_theta;
  la.accepted = pp->accepted;
  la.new_cost = pp->new_cost;
  la.new_grad = pp->new_grad;
  la.new_status = pp->new_status;
  la.cost_hist = cost_hist;
  la.steps = pp->steps;
  return la;
}
}  // namespace

int debye_polish_create(const debye_batch *shape, const int64_t *f_off_host, const int32_t *n_poles_host, int64_t ld,
                        debye_lbfgs_params lp, debye_polish **out) {
  if (!out) return fail(DEBYE_EINVAL, "out is NULL");
  *out = nullptr;
  int rc = check_batch(shape);
  if (rc) return rc;
  if (!f_off_host || !n_poles_host) return fail(DEBYE_EINVAL, "host shape arrays are NULL");
  if (ld < shape->max_poles) return fail(DEBYE_ERANGE, "ld < max_poles");
  if (shape->n_cand != shape->n_mat) return fail(DEBYE_EINVAL, "polish needs exactly one candidate per material");
  if (lp.steps < 0 || lp.mem < 1 || lp.mem > DFIT_MAX_MEM || lp.max_trials < 1 || lp.max_trials > 64 ||
      !(lp.c1 > 0.0 && lp.c1 < 1.0))
    return fail(DEBYE_ERANGE, "L-BFGS parameters out of range (steps >= 0, mem 1..%d, trials 1..64, 0 < c1 < 1)",
                DFIT_MAX_MEM);
  const int32_t M = shape->n_mat;
  const int T = lp.max_trials;
  constexpr int STAGES = dfit::LBFGS_STAGES;
  debye_polish *pp = new debye_polish();
  polish_stages(M, T, pp->stage_end);
  std::vector<int64_t> one(M + 1), offs((size_t)STAGES * (M + 1));
  for (int32_t m = 0; m <= M; ++m) {
    one[m] = m;
    for (int s = 0; s < STAGES; ++s)
      offs[(size_t)s * (M + 1) + m] = (int64_t)m * (pp->stage_end[s] - (s ? pp->stage_end[s - 1] : 0));
  }
  pp->M = M;
  pp->max_poles = shape->max_poles;
  pp->mem = lp.mem;
  pp->max_trials = T;
  pp->steps = lp.steps;
  pp->c1 = lp.c1;
  pp->ld = ld;
  pp->n_freq = shape->n_freq;
  auto bail = [&](int r) {
    debye_polish_destroy(pp);
    return r;
  };
  const int64_t n1 = (int64_t)M * ld, nT = (int64_t)M * T;
  const size_t doubles = (size_t)(n1 /*grad*/ + 2 * (int64_t)M * lp.mem * ld /*S,Y*/ + (int64_t)M * lp.mem /*rho*/ +
                                  n1 /*dir*/ + M /*gd*/ + nT * ld /*trial theta*/ + nT /*trial cost*/ + n1 /*new theta*/ +
                                  M /*new cost*/ + n1 /*new grad*/ + M /*cost*/ + M /*accepted cost*/);
  const size_t bytes = offs.size() * 8 + doubles * 8 + (size_t)5 * M * 4 + (size_t)nT + (size_t)M + 64;
  if (hipMalloc(&pp->ws, bytes) != hipSuccess) {
    pp->ws = nullptr;
    return bail(fail(DEBYE_ENOMEM, "polish workspace allocation failed"));
  }
  pp->offs = (int64_t *)pp->ws;
  double *dp = (double *)(pp->offs + offs.size());
  auto take = [&](int64_t n) {
    double *r = dp;
    dp += n;
    return r;
  };
  pp->grad = take(n1);
  pp->S = take((int64_t)M * lp.mem * ld);
  pp->Y = take((int64_t)M * lp.mem * ld);
  pp->rho = take((int64_t)M * lp.mem);
  pp->dir = take(n1);
  pp->gd = take(M);
  pp->trial_theta = take(nT * ld);
  pp->trial_cost = take(nT);
  pp->new_theta = take(n1);
  pp->new_cost = take(M);
  pp->new_grad = take(n1);
  pp->cost = take(M);
  pp->acc_cost = take(M);
  int32_t *ip = (int32_t *)dp;
  pp->hist_n = ip;
  pp->hist_head = ip + M;
  pp->accepted = ip + 2 * M;
  pp->done = ip + 3 * M;
  pp->stalled = ip + 4 * M;
  pp->trial_status = (int8_t *)(ip + 5 * M);
  pp->new_status = pp->trial_status + nT;
  if (hipMemcpy(pp->offs, offs.data(), offs.size() * 8, hipMemcpyHostToDevice) != hipSuccess)
    return bail(fail(DEBYE_EHIP, "polish: upload of the trial offsets failed"));
  std::vector<int64_t> f_h(f_off_host, f_off_host + M + 1);
  if ((rc = debye_plan_create(shape, f_h.data(), one.data(), n_poles_host, 0, &pp->p1))) return bail(rc);
  debye_batch bt = *shape;
  for (int s = 0; s < STAGES; ++s) {
    const int64_t *host = offs.data() + (size_t)s * (M + 1);
    if (host[M] == 0) continue;
    bt.cand_off = pp->offs + (size_t)s * (M + 1);
    bt.n_cand = host[M];
    if ((rc = plan_create(&bt, f_h.data(), host, n_poles_host, 0, POLISH_LIVE[s], &pp->trials[s]))) return bail(rc);
  }
  *out = pp;
  return DEBYE_OK;
}

int debye_polish_destroy(debye_polish *pp) {
  if (!pp) return DEBYE_OK;
  debye_plan_destroy(pp->p1);
  for (debye_plan *p : pp->trials) debye_plan_destroy(p);
  if (pp->ws) {
    (void)hipDeviceSynchronize();   // no work of the context may still read the workspace
    (void)hipFree(pp->ws);
  }
  delete pp;
  return DEBYE_OK;
}

int debye_polish_begin(debye_polish *pp, const debye_batch *b, const double *theta, double damping, uint32_t flags,
                       hipStream_t stream) {
  int rc = polish_check(pp, b, damping, flags);
  if (rc) return rc;
  if (!theta) return fail(DEBYE_EINVAL, "theta is NULL");
  // empty history (a fill kernel, not a memset, so that the call can be captured)
  CHECK_HIP(dfit::launch_fill_i32(pp->hist_n, 2 * (int64_t)pp->M, 0, stream), "fill");
  CHECK_HIP(dfit::launch_fill_i32(pp->stalled, (int64_t)pp->M, 0, stream), "fill");
  return debye_fit_eval_grad(pp->p1, b, theta, pp->ld, damping, flags, nullptr, pp->cost, pp->grad, nullptr, nullptr,
                             pp->new_status, stream);
}

namespace {
// the step whose direction and trial points are there already; with `next` the
// next step's are formed as well
int polish_rest_of_step(debye_polish *pp, const debye_batch *b, dfit::LbfgsArgs la, double damping, uint32_t flags,
                        bool next, hipStream_t stream) {
  int rc;
  debye_batch bt = *b;
  int64_t row = 0;
  int32_t t_lo = 0;
  for (int s = 0; s < dfit::LBFGS_STAGES; ++s) {
    const int32_t t_hi = pp->stage_end[s] - 1;
    if (t_hi < t_lo) continue;
    bt.cand_off = pp->offs + (size_t)s * (pp->M + 1);
    bt.n_cand = (int64_t)pp->M * (t_hi + 1 - t_lo);
    // The first stage leaves out the materials that no longer move.  One whose
    // step found no acceptable trial is stalled for good: its point, gradient
    // and history stay as they were, so every later step would rebuild the
    // same trials and reject them again.
    if ((rc = fit_eval_impl(pp->trials[s], &bt, pp->trial_theta + row * pp->ld, pp->ld, damping, flags,
                            pp->trial_cost + row, nullptr, nullptr, pp->trial_status + row,
                            s == 0 ? pp->stalled : pp->done, pp->trials[s]->launch, stream)))
      return rc;
    CHECK_HIP(dfit::launch_lbfgs_select(la, t_lo, t_hi, stream), "lbfgs select");
    row += bt.n_cand;
    t_lo = t_hi + 1;
  }
  // cost and gradient at the accepted points (the stalled materials, which
  // accepted none, are left out)
  if ((rc = fit_eval_grad_launch(pp->p1, b, pp->new_theta, pp->ld, damping, flags, nullptr, pp->new_cost, pp->new_grad,
                                 nullptr, nullptr, pp->new_status, nullptr, 0, stream, pp->stalled)))
    return rc;
  CHECK_HIP(dfit::launch_lbfgs_update(la, next, stream), "lbfgs update");
  return DEBYE_OK;
}
}  // namespace

int debye_polish_step(debye_polish *pp, const debye_batch *b, double *theta, const double *lb, const double *ub,
                      double damping, uint32_t flags, int32_t step, double *cost_hist, hipStream_t stream) {
  int rc = polish_check(pp, b, damping, flags);
  if (rc) return rc;
  if (!theta || !lb || !ub) return fail(DEBYE_EINVAL, "NULL pointer");
  if (step < 0 || (cost_hist && step >= pp->steps))
    return fail(DEBYE_ERANGE, "step %d outside 0..%d", step, pp->steps - 1);
  dfit::LbfgsArgs la = polish_args(pp, b, theta, lb, ub, cost_hist);
  la.step = step;
  CHECK_HIP(dfit::launch_lbfgs_direction(la, stream), "lbfgs direction");
  return polish_rest_of_step(pp, b, la, damping, flags, false, stream);
}

int debye_lbfgs_polish(debye_polish *pp, const debye_batch *b, double *theta, const double *lb, const double *ub,
                       double damping, uint32_t flags, double *cost_hist, hipStream_t stream) {
  int rc = polish_check(pp, b, damping, flags);
  if (rc) return rc;
  if (!theta || !lb || !ub) return fail(DEBYE_EINVAL, "NULL pointer");
  if (pp->steps == 0) return DEBYE_OK;
  if ((rc = debye_polish_begin(pp, b, theta, damping, flags, stream))) return rc;
  dfit::LbfgsArgs la = polish_args(pp, b, theta, lb, ub, cost_hist);
  CHECK_HIP(dfit::launch_lbfgs_direction(la, stream), "lbfgs direction");
  for (la.step = 0; la.step < pp->steps; ++la.step)
    if ((rc = polish_rest_of_step(pp, b, la, damping, flags, la.step + 1 < pp->steps, stream))) return rc;
  return DEBYE_OK;
}

}  // extern "C"
