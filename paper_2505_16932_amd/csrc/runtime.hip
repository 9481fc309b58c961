// Host runtime of the C ABI in pe.h: argument checks, workspace layout, tile
// tables, launch sequence of the online stage, plans and hipGraph capture.
//
// Launch sequence for T steps (Section 3.5 / the Appendix A.1 listing, with
// the scale folded into step 1):
//   prep [+ finalize] [+ planes]           ||G||_F, max|G|, X_0 copies
//   for t: gram [+ reduce], a2 [+ reduce], update [+ its last tiles]
// Each launch covers every matrix of the call of one (precision, tile) class
// (grouped, persistent blocks); matrices of at most 64 rows run all of their
// steps in one launch (resident.hip).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "pe.h"
#include "pe_device.h"

namespace pe {
hipError_t launch_put(const PutChunk& c, hipStream_t st);
hipError_t launch_finalize(const KArgs& a, hipStream_t st);
hipError_t launch_select(const KArgs& a, hipStream_t st);
hipError_t launch_combine(int prec, const KArgs& a, hipStream_t st);
hipError_t launch_quant(int kind, const KArgs& a, int grid_cap, hipStream_t st);
hipError_t launch_fast(int prec, int bt, int kind, const KArgs& a, hipStream_t st);
hipError_t launch_planes(const KArgs& a, hipStream_t st);
hipError_t launch_power(int phase, const KArgs& a, hipStream_t st);
hipError_t launch_init_b(const KArgs& a, hipStream_t st);
hipError_t launch_est(const KArgs& a, int iters, hipStream_t st, const int32_t* offs_a, int total_a,
                      const int32_t* offs_b, int total_b);
hipError_t launch_mlp_forward(const float* params, const float* feats, int B, float* logits,
                              hipStream_t st);
hipError_t launch_mlp_grad(const float* params, const float* feats, const int32_t* labels, int B,
                           float* part, float* part_loss, float* grad_out, float* loss_out,
                           float* upd_params, float* m, float* v, int step, float lr, hipStream_t st);
hipError_t launch_quantize(const void* x, int x_bf16, uint8_t* q, int64_t n, float scale,
                           hipStream_t st);
hipError_t launch_prep(int prec, const KArgs& a, int grid_cap, hipStream_t st);
void warm_launch_grids();
hipError_t launch_gemm(int prec, int bt, int kind, const KArgs& a, int grid_cap, hipStream_t st);
hipError_t launch_reduce(int prec, int bt, int kind, const KArgs& a, int grid_cap, hipStream_t st);
hipError_t launch_small_gemm(int prec, int bt, int kind, const KArgs& a, hipStream_t st);
hipError_t launch_resident(int bucket, const KArgs& a, const ResSchedule& s, hipStream_t st);
hipError_t launch_f32_gemm(int kind, const KArgs& a, hipStream_t st);
hipError_t launch_f32_reduce(int kind, const KArgs& a, hipStream_t st);
hipError_t launch_f32_fast(int kind, const KArgs& a, hipStream_t st);
hipError_t launch_small_reduce(int prec, int bt, int kind, const KArgs& a, hipStream_t st);
}  // namespace pe

using namespace pe;

namespace {

thread_local std::string g_last_error;

enum Phase { PH_PREP = 0, PH_GRAM, PH_A2, PH_UPD, PH_RGRAM, PH_RA2, PH_COMBINE, PH_EST_A, PH_EST_B,
             PH_QX, PH_QA, PH_FSYRK, PH_PW, PH_PLANES, PH_RES, PH_N };

// Schedule classes of the learned path: (l, T'), T' = 0 meaning the call's T;
// class 4 is the caller's schedule for all T steps.  Steps past a class's T'
// leave the matrix as it is (its kernels skip it; the last step copies X).
struct ClassDef { double ell; int steps; };
constexpr ClassDef kClassTable[kClasses] = {{1e-1, 2}, {1e-1, 3}, {3e-2, 3}, {1e-2, 4},
                                            {1e-3, 0}, {3e-3, 4}, {3e-4, 0}, {1e-4, 0}};
constexpr int kFixedClass = 4;
int class_steps(int c, int T) { return kClassTable[c].steps > 0 ? std::min(T, kClassTable[c].steps) : T; }
constexpr int kEstIters = 8;

bool learned_mode(const pe_opts* o) { return o->predictor != nullptr || o->force_class >= 0; }

constexpr int kGemmGridCap = 512;       // 128-tile kernel: 2 resident blocks per CU x 256 CUs
constexpr int kGemmGridCapLarge = 256;  // 256-tile kernel: 1 resident block per CU
constexpr int kPrepGridCap = 2048;
constexpr int kReduceGridCap = 1024;
constexpr int kQuantGridCap = 2048;
// Gram-side items wanted per launch before split-K kicks in.  Split-K buys
// parallelism with FP32 partial tiles written and summed by a second launch;
// measured on a single 4096 x 1024 bf16 matrix (36 Gram tiles of 128), splits
// of 15 / 8 / 4 / 2 / 1 gave 0.83 / 0.68 / 0.58 / 0.55 / 0.58 ms per call, so
// the target stays low: a couple of splits for calls with tens of tiles.
constexpr int kFillTarget = 64;

size_t align_up(size_t x, size_t a = 256) { return (x + a - 1) / a * a; }
int64_t round_up(int64_t x, int64_t a) { return (x + a - 1) / a * a; }

pe_status hip_fail(hipError_t e, const char* where) {
  char buf[256];
  snprintf(buf, sizeof buf, "%s: %s", where, hipGetErrorString(e));
  g_last_error = buf;
  return PE_EHIP;
}

// Launch classes: (precision, block tile).  Every phase launches once per class
// present in a call, over the items of that class's matrices only, so one
// grouped call can mix tiles (per-shape-class choices of the autotuned table)
// and precisions (matrices too small for bf16 rounding to average out run
// FP32 operands inside a bf16 call).
constexpr int kNCls = 8;  // fp32 and bf16 on each of the three tiles; kTiny on the 64, kF32M on the 128 tile
inline int cls_of(int prec, int bt) {
  return prec == kTiny ? 6 : prec == kF32M ? 7 : (prec == kF32 ? 0 : 3) + (bt == kTileLarge ? 2 : bt == kTileSmall ? 1 : 0);
}
inline int cls_prec(int c) { return c < 3 ? kF32 : c < 6 ? kBF16 : c == 6 ? kTiny : kF32M; }
inline int cls_bt(int c) { return kTileTiny << (c % 3); }
inline bool is_f32(int prec) { return prec == kF32 || prec == kTiny || prec == kF32M; }

struct Layout {
  std::vector<MatDesc> descs;           // device pointers filled when ws != nullptr
  std::vector<int32_t> prec, bt;        // per matrix
  // item tables: offs[ph][cls] holds count + 1 prefix offsets in which the
  // matrices of other classes contribute no items (phases that do not depend
  // on the class -- the estimate's matrix-vector products -- keep every
  // matrix in class 0's table)
  std::vector<int32_t> offs[PH_N][kNCls];
  int32_t totals[PH_N][kNCls] = {};
  // Gram items per class ordered by matrix, longest k (Lp) first: per-tile
  // work is proportional to Lp, and persistent blocks take items round-robin,
  // so long tiles first and short ones last balance the CUs
  std::vector<int32_t> ord_gram[kNCls];
  size_t bytes = 0;
  size_t descs_off = 0, offs_off = 0, coef_off = 0;
  size_t sel_off = 0;  // learned plans: kSelWords words per matrix (class, flag, features, estimate)
  int prep_group = kPrepGroup;
  bool fold_norm = false; // KArgs::fold_norm
  bool alike = false;     // KArgs::alike
  // item tables in use, packed behind the descriptors: word offset of each
  // phase and class, and of each class's Gram order (-1: none)
  int32_t tab[PH_N][kNCls], tab_ord[kNCls];
  bool resident = false;  // some matrices run the resident kernel
  bool x0b = false;    // every bf16-path matrix has MatDesc::x0b
};

// per-matrix selection record of a learned plan, contiguous over the matrices
// so pe_plan_selection reads all of them with one copy: words 0-15 class and
// fallback flag, 16-31 the 16 features, 32-47 the estimate
constexpr int kSelWords = 48;

bool valid_matrix(const pe_matrix& m) {
  if (m.m < 0 || m.n < 0) return false;
  if (m.m == 0 || m.n == 0) return true;
  if (!m.G || (!m.X && !m.W)) return false;
  if (m.ldg < m.n || (m.X && m.ldx < m.n)) return false;
  if (m.g_dtype != PE_F32 && m.g_dtype != PE_BF16) return false;
  if (m.X && m.x_dtype != PE_F32 && m.x_dtype != PE_BF16) return false;
  if (m.M && m.ldm < m.n) return false;
  if (m.W && (m.ldw < m.n || (m.w_dtype != PE_F32 && m.w_dtype != PE_BF16))) return false;
  if (m.m > (1 << 20) || m.n > (1 << 20)) return false;
  return true;
}

pe_status check_opts(const pe_opts* o) {
  if (!o) return PE_EINVAL;
  if (o->T < 1 || o->T > kMaxSteps || !o->abc) return PE_EINVAL;
  if (o->compute < PE_COMPUTE_F32 || o->compute > PE_COMPUTE_FP8) return PE_EINVAL;
  if (o->norm_mode != 0 && o->norm_mode != 1) return PE_EINVAL;
  if (o->tile < 0 || o->tile > 2) return PE_EINVAL;
  if (o->compute == PE_COMPUTE_FP8) {
    if (o->fp8_steps < 0 || o->fp8_steps > o->T - 1) return PE_EINVAL;
  }
  for (int i = 0; i < 3 * o->T; ++i)
    if (!std::isfinite(o->abc[i])) return PE_EINVAL;
  if (o->force_class < -1 || o->force_class >= kClasses) return PE_EINVAL;
  if (!std::isfinite(o->fallback_tau)) return PE_EINVAL;
  if (o->split_k < 0 || o->split_k > 64) return PE_EINVAL;
  if (o->fast_restart < 0 || !std::isfinite(o->fast_eps) || o->fast_eps < 0.0f) return PE_EINVAL;
  if (o->fast_restart > 0 &&
      (o->compute != PE_COMPUTE_F32 || learned_mode(o) || o->tile == 2)) return PE_EUNSUPPORTED;
  if (!(o->muon_beta >= 0.0f && o->muon_beta < 1.0f) || !std::isfinite(o->muon_lr) ||
      !std::isfinite(o->muon_wd)) return PE_EINVAL;
  if (o->spectral_init < 0 || o->spectral_init > 1000) return PE_EINVAL;
  if (o->spectral_init > 0 &&
      ((o->compute == PE_COMPUTE_FP8 && o->fp8_steps > 0) || learned_mode(o) || o->fast_restart > 0))
    return PE_EUNSUPPORTED;
  return PE_OK;
}

// Block tile per matrix: 256 x 256 (8 waves, 32x32 MFMA fragments, wave tile
// 128 x 64) halves the LDS and L2 traffic per flop of the 128 x 128 tile, but
// pads s and L to multiples of 256 and yields 4x fewer tiles.  The choice comes
// from the autotuned table, keyed by shape class (precision, s bucket, aspect
// bucket; see shape_class()) and call regime (_x1 / _xN, see tile_for());
// without an entry the 256 tile is taken for s >= 512 when the call's update
// has at least one 256 tile per CU.  FP32 matrices always take the small tiles
// (small_tiles picks 64 or 128), kF32M the 128 tile.
std::mutex g_tab_mu;
std::map<std::string, int> g_tile_table;

std::string shape_class(int prec, int64_t s, int64_t L) {
  static const int64_t sb[] = {256, 512, 1024, 2048, 4096};
  int i = 0;
  while (i < 5 && s > sb[i]) ++i;
  const double a = (double)L / (double)s;
  const int ab = a <= 1.5 ? 1 : (a <= 4.0 ? 4 : 16);
  char buf[64];
  snprintf(buf, sizeof buf, "%s_s%lld_a%d", prec == kF32 ? "f32" : "bf16",
           (long long)(i < 5 ? sb[i] : 8192), ab);
  return buf;
}

// Largest bounds with which operands stay in planes (planes_fit)
constexpr double kFitX = 8.0, kFitB = 128.0, kFitD = 2048.0;

// Largest power of two q with q * bound <= 2^14 (a quarter of the fp16 range).
float plane_scale(double bound) {
  if (!(bound > 1e-30)) bound = 1e-30;
  if (!(bound < 1e30)) bound = 1e30;
  return (float)std::ldexp(1.0, 14 - (int)std::ceil(std::log2(bound)));
}

// Bounds on the singular values of the fp32 path's operands per kernel step.
// X_0 = G / (1.01 ||G||_F + ..) has none above 1; a step with p(x) = a x + b x^3
// + c x^5 takes a bound u to max |p| on [0, u] (the quarter of the range that
// plane_scale leaves covers the rounding of the iterate), A has norm u^2 and
// B - beta I twice max |b y + c y^2| at most.  The learned path takes the
// largest bound over the classes.  The spectrum-aware step's cubic is chosen on
// the device, which also chooses the scale of its B (kScInitQ); it maps the
// spectrum to [0, 1] where its power method has converged.
struct PlaneBounds {
  std::vector<double> x, a, b;
};
PlaneBounds plane_bounds(const std::vector<std::vector<double>>& tables, int T, int t0) {
  const int n = T + t0;
  PlaneBounds r;
  r.x.assign(n + 1, 0.0);
  r.a.assign(n, 0.0);
  r.b.assign(n, 0.0);
  for (const auto& abc : tables) {
    double u = 1.0;
    for (int t = 0; t < n; ++t) {
      r.x[t] = std::max(r.x[t], u);
      r.a[t] = std::max(r.a[t], u * u);
      if (t >= t0) {
        const double* k = &abc[3 * (t - t0)];
        double un = 0.0, bn = 0.0;
        auto at = [&](double y) {  // y = x^2 in [0, u^2]
          if (!(y > 0.0) || y > u * u) return;
          const double h = y * (k[1] + k[2] * y);
          un = std::max(un, std::sqrt(y) * std::fabs(k[0] + h));
          bn = std::max(bn, std::fabs(h));
        };
        // the ends and the extrema of p (a + 3 b y + 5 c y^2 = 0) and of b y + c y^2
        at(u * u);
        at(-k[1] / (2.0 * k[2]));
        const double disc = 9.0 * k[1] * k[1] - 20.0 * k[0] * k[2];
        if (disc >= 0.0) {
          at((-3.0 * k[1] + std::sqrt(disc)) / (10.0 * k[2]));
          at((-3.0 * k[1] - std::sqrt(disc)) / (10.0 * k[2]));
        }
        if (k[2] == 0.0) at(-k[0] / (3.0 * k[1]));
        r.b[t] = std::max(r.b[t], 2.0 * bn);
        u = std::min(std::max(un, 1e-20), 1e20);
      }
    }
    r.x[n] = std::max(r.x[n], u);
  }
  return r;
}

// The products of the fast rectangular iteration in order (see
// small_fast_kernel), in segments of `restart` steps:
//   product(seg, kind, fp, fq, e1, c1, e2, c2, cacc, out, cdiag)
//   update(seg, last, q, D)
template <typename P, typename U>
pe_status fast_walk(const float* abc, int T, int restart, float eps, P&& product, U&& update) {
  pe_status s;
  int seg = 0;
  for (int t0 = 0; t0 < T; t0 += restart, ++seg) {
    const int k = std::min(restart, T - t0);
    int dcur = kFbD0;
    // Y = X X^T (of the normalised X_0 in the first segment, plus eps I)
    if ((s = product(seg, 0, -1, -1, kFbNone, 0.f, kFbNone, 0.f, 1.f, kFbR, seg == 0 ? eps : 0.f)) != PE_OK) return s;
    float q = 1.0f;
    for (int j = 0; j < k; ++j) {
      const float a = abc[3 * (t0 + j)], b = abc[3 * (t0 + j) + 1], cc = abc[3 * (t0 + j) + 2];
      // B_t = b R + c R^2 (into D directly on the segment's first step, D_1 = B_1)
      const int bdst = j == 0 ? dcur : kFbB;
      if ((s = product(seg, 1, kFbR, kFbR, kFbR, b, kFbNone, 0.f, cc, bdst, 0.f)) != PE_OK) return s;
      if (j > 0) {
        const int dn = dcur == kFbD0 ? kFbD1 : kFbD0;
        if ((s = product(seg, 1, dcur, kFbB, dcur, a, kFbB, q, 1.f, dn, 0.f)) != PE_OK) return s;
        dcur = dn;
      }
      if (j + 1 < k) {
        if ((s = product(seg, 1, kFbR, bdst, kFbNone, 0.f, kFbNone, 0.f, 1.f, kFbP, 0.f)) != PE_OK) return s;
        if ((s = product(seg, 1, kFbP, bdst, kFbR, a * a, kFbP, 2.f * a, 1.f, kFbR, 0.f)) != PE_OK) return s;
      }
      q *= a;
    }
    if ((s = update(seg, t0 + k >= T, q, dcur)) != PE_OK) return s;
  }
  return PE_OK;
}

// Bounds on its operands in the same order, one per product and update (the
// next X), from the recursions on scalars sampled over each segment's spectrum
// [0, u^2], evenly and, below the first even sample, by half powers of two (a
// schedule that has brought the upper part to 1 still moves the lower one); grew: whether one is past the planes' reach (see planes_fit).
std::vector<double> fast_bounds(const float* abc, int T, int restart, float eps, bool* grew) {
  constexpr int kEven = 256, kSamples = kEven + 64;
  typedef std::vector<double> Vec;
  Vec y(kSamples), val[5], out;
  for (auto& v : val) v.assign(kSamples, 0.0);
  double u = 1.0;
  *grew = false;
  auto product = [&](int, int kind, int fp_, int fq_, int fe1, float c1, int fe2, float c2, float cacc, int fout,
                     float cdiag) {
    if (kind == 0)
      for (int i = 0; i < kSamples; ++i) y[i] = u * u / kEven * (i < kEven ? i + 1 : std::exp2(-0.5 * (i - kEven + 1)));
    Vec v(kSamples);
    double m = 0.0;
    for (int i = 0; i < kSamples; ++i) {
      v[i] = cacc * (kind == 0 ? y[i] : val[fp_][i] * val[fq_][i]) + cdiag;
      if (fe1 >= 0) v[i] += c1 * val[fe1][i];
      if (fe2 >= 0) v[i] += c2 * val[fe2][i];
      m = std::max(m, std::fabs(v[i]));
    }
    val[fout] = v;
    out.push_back(m);
    *grew = *grew || !(m <= (fout == kFbD0 || fout == kFbD1 ? kFitD : kFitB));
    return PE_OK;
  };
  auto update = [&](int, bool last, float q, int dcur) {
    double un = 1e-20;
    for (int i = 0; i < kSamples; ++i) un = std::max(un, std::sqrt(y[i]) * std::fabs(q + val[dcur][i]));
    u = std::min(un, 1e20);
    out.push_back(u);
    *grew = *grew || (!last && !(u <= kFitX));
    return PE_OK;
  };
  (void)fast_walk(abc, T, restart, eps, product, update);
  return out;
}

// Whether the schedule keeps within the operand planes' reach.  An operand is
// held to 2^-39 of its bound, so what matters is how far the bound can lie above
// the values: measured with a first step (k, 0, 0) and Newton-Schulz steps on
// Gaussian inputs, planes against FP32 MFMA: X bounded by 4, B by 152: 4.6e-8 and
// 4.5e-8 (s = 4096); X 2, B 737: 6.0e-8 and 4.7e-8; X 8, B 2.9e3: 1.6e-7 and
// 5.0e-8; the fast iteration with D bounded by 2.6e3 and R, B, P by 441 3.8e-8
// and 3.9e-8, by 1.2e4 and 1.5e3 8.2e-8 and 4.6e-8.  Schedules for [l, 1] have
// X 2, B 16, and in segments of three steps D 130.
bool planes_fit(const pe_opts* o) {
  std::vector<float> abc(o->abc, o->abc + 3 * o->T);
  if (o->fast_restart > 0) {
    bool grew = false;
    fast_bounds(abc.data(), o->T, o->fast_restart, o->fast_eps, &grew);
    return !grew;
  }
  const PlaneBounds r = plane_bounds({std::vector<double>(abc.begin(), abc.end())}, o->T, 0);
  for (int t = 0; t < o->T; ++t)
    if (!(r.x[t] <= kFitX) || !(r.b[t] <= kFitB)) return false;
  return true;
}

// Precision of one matrix: FP32 on the FP32 path; on the bf16/FP8 paths FP32
// as well when the smaller side is below kTinyS, where a handful of singular
// values leave bf16 rounding errors nothing to average over (relative errors
// up to ~1e-1 at s = 2-8 on Gaussian inputs) and the products cost nothing.
constexpr int64_t kTinyS = 16;
int prec_for(const pe_opts* o, const pe_matrix& m, bool fit) {
  const int64_t s = std::min(m.m, m.n);
  if (s < kTinyS) return kTiny;
  if (o->compute != PE_COMPUTE_F32) return kBF16;
  if (!fit) return kF32M;
  // FP32 results of long schedules stay with FP32 MFMA's summation order (see
  // f32.hip for where the lines lie); a bf16 result or a weight step hides the
  // difference, and the fast, learned and spectrum-aware forms have their own
  // error bars
  const bool plain = o->fast_restart == 0 && !learned_mode(o) && o->spectral_init == 0;
  if (plain && m.X && m.x_dtype == PE_F32 && !m.W && ((o->T == 6 && s > 1024) || (o->T > 6 && s > 384))) return kF32M;
  return kF32;
}

// Call regimes of the autotuned table: "xN" for calls with at least
// kBatchFlops algorithmic FLOP per step (3 s^2 L + s^3 summed over the
// matrices; the autotuner's batches carry ~3e12 per step) or with more than
// kBatchTiles update tiles of 256 (four rounds on the 256-CU part), where padding
// to 256 costs at most 1.35 times the work of padding to 128, or with two rounds,
// kBatchTilesMin, where it costs at most 1.1 times (unless a weight step goes with
// a bf16 output, which the 256 tile takes it from, the small ones from the FP32
// X_T); "x1" below and otherwise.
// e4m3 calls, whose small tiles convert while staging, count tiles and FLOP only.
// Measured per call, 256 against 128: 1536 x 1536 x 16 (576 tiles) 1.61 and 2.07
// ms, 1024 x 4096 x 8 (512) 0.94 and 1.04, 2048 x 2048 x 8 (512) 1.79 and 1.90,
// 768 x 3072 x 16 (576) 0.94 and 0.94, 2048 x 32768 (1024) 2.92 and 3.29; below
// two rounds 1024 x 1024 x 8 (128) 0.62 and 0.46, 512 x 2048 x 8 (128) 0.35 and
// 0.24; with padding, two rounds: 520 x 2080 x 20 (1.6 times) 0.82 and 0.70, 1100
// x 4400 x 6 (1.27) 1.14 and 1.09; four: 384 x 1536 x 96 (1.8) 1.45 and 1.14,
// 640 x 2560 x 48 (1.44) 2.03 and 1.92, 896 x 3584 x 24 (1.31) 2.06 and 2.15,
// 1100 x 4400 x 14 (1.27) 2.21 and 2.43.
constexpr double kBatchFlops = 3e12;
constexpr int64_t kBatchTiles = 1024, kBatchTilesMin = 512;

// Block tile of one matrix.  Forced by opts.tile; else the autotuned table's
// entry for the matrix's shape class in the call's regime; else 256 for bf16
// matrices with s >= 512 in calls whose update has at least one 256-tile per
// CU, 128 otherwise.
int tile_for(const pe_opts* o, int prec, int64_t s, int64_t L, bool batch_regime, int64_t upd_tiles256) {
  if (is_f32(prec) || o->tile == 1) return kTileSmall;
  if (o->tile == 2) return kTileLarge;
  {
    std::lock_guard<std::mutex> lk(g_tab_mu);
    if (!g_tile_table.empty()) {
      auto it = g_tile_table.find(shape_class(prec, s, L) + (batch_regime ? "_xN" : "_x1"));
      if (it != g_tile_table.end()) return it->second == 2 ? kTileLarge : kTileSmall;
    }
  }
  return (s >= 512 && upd_tiles256 >= 256) ? kTileLarge : kTileSmall;
}

// Tiles of a matrix on the small-tile family (tile id 1): ubt for the update,
// which also sets the padding, sbt <= ubt for the symmetric products; tiles128:
// update tiles of 128 of all the call's matrices of the family.
//  * s <= 64: everything on the 64 tile (a 128 tile would be three quarters
//    padding; 432 matrices of 768 x 64 that the resident kernel runs in 81 us
//    took 416 us per call on the 64 tile and 906 on the 128 tile).
//  * Symmetric products: the 64 tile up to s = 1536, where a single matrix has
//    at most 78 upper tiles of 128 for 256 CUs (1024 x 4096: 253 us per call
//    against 370 with 128 tiles and split-K; 1536 x 1536: 270 against 337; at
//    2048 x 2048 the 128 tile wins, 410 against 438); in calls that fill the
//    chip anyway they stay ahead or near (256 x 1024 x 48: 269 against 300, 1024
//    x 1024 x 16: 753 against 717) except for s <= 128 (4096 x 128 x 256: 1.78
//    against 1.70 ms).  On the fp32 path, where the 64 tile multiplies four
//    plane pairs and the 128 tile three, calls of more than 1024 update tiles
//    take the 128 tile (768 x 3072 x 12: 1.61 against 1.83 ms; x 8: 1.15 against
//    1.23; x 4: 0.85 against 0.75).
//  * Update: the 64 tile where both the matrix (64 tiles of 128) and the call
//    (256) have few: one 1024 x 1024 takes 170 us per call against 199, sixteen
//    of them 867 against 753.
void small_tiles(int prec, int64_t s, int64_t L, int64_t tiles128, int* ubt, int* sbt) {
  const int64_t own = (s + 127) / 128 * ((L + 127) / 128);
  *ubt = s <= 64 || (own <= 64 && tiles128 <= 256) ? kTileTiny : kTileSmall;
  const bool full = prec == kF32 ? tiles128 > 1024 : s <= 128 && tiles128 > 512;
  *sbt = *ubt == kTileTiny || (s <= 1536 && !full) ? kTileTiny : kTileSmall;
}

// With split_k = 1 a matrix has the same bits in every call that gives it the same
// tile id: whatever orders its sums (64 or 128 tiles, the resident kernel, the
// norm's items, the ring's k groups, smaller tiles in a short last round) then
// depends on the matrix alone.
bool alike(const pe_opts* o) { return o->split_k == 1; }

// A matrix that the resident kernel can run: bf16 products in the plain
// iteration (no e4m3 step, learned choice or spectrum-aware step), at most 64
// rows and 1024 columns after orientation.
bool fits_resident(const pe_opts* o, int prec, int64_t s, int64_t L) {
  return prec == kBF16 && o->tile != 2 && s <= 64 && L <= 1024 && !learned_mode(o) && o->spectral_init == 0 &&
         !(o->compute == PE_COMPUTE_FP8 && o->fp8_steps > 0);
}
// It runs them when the whole call fits (one 64 x 64 takes 77 us in grouped
// launches, 432 of 768 x 64 446 us) or when there are many (a launch of its own
// takes 20-30 us, more than a few small matrices add to the other matrices'
// launches).
constexpr int kResidentMany = 64;

// Build the per-matrix descriptors and the item tables.  With ws == nullptr
// only sizes are computed.
pe_status build_layout(int count, const pe_matrix* mats, const pe_opts* o, char* ws, Layout* L) {
  L->descs.clear();
  L->resident = false;
  L->prec.assign(count, kBF16);
  L->bt.assign(count, kTileSmall);
  for (int p = 0; p < PH_N; ++p)
    for (int c = 0; c < kNCls; ++c) L->offs[p][c].assign(1, 0);
  // update tiles of the whole call at the 256 tile (the built-in tile rule)
  int64_t upd256 = 0;
  double call_flops = 0.0, work256 = 0.0, work128 = 0.0;
  bool step_bf16 = false;
  for (int i = 0; i < count; ++i) {
    const pe_matrix& m = mats[i];
    if (m.m <= 0 || m.n <= 0) continue;
    const int64_t s = std::min(m.m, m.n), Lx = std::max(m.m, m.n);
    upd256 += round_up(s, kTileLarge) / kTileLarge * (round_up(Lx, kTileLarge) / kTileLarge);
    call_flops += 3.0 * (double)s * s * Lx + (double)s * s * s;
    auto work = [&](int t) { return (double)round_up(s, t) * round_up(s, t) * round_up(Lx, t); };
    step_bf16 = step_bf16 || (m.W && m.X && m.x_dtype == PE_BF16);
    if (s > 256) {  // (smaller ones take the small tiles in either regime)
      work256 += work(kTileLarge);
      work128 += work(kTileSmall);
    }
  }
  const bool fp8 = o->compute == PE_COMPUTE_FP8 && o->fp8_steps > 0;
  const bool large = call_flops >= kBatchFlops || upd256 > kBatchTiles;
  const bool batch_regime = fp8 ? large : (large && work256 <= 1.35 * work128) ||
                                          (upd256 >= kBatchTilesMin && work256 <= 1.1 * work128 && !step_bf16);
  // first pass: precision and tile; the second needs the call's totals
  struct Shape { int64_t s, L, sp, Lp; int nb, nbL, nbs, syrk, upd, prep, prec, bt, sbt, cls, scls; bool family, res; };
  std::vector<Shape> sh;
  int64_t syrk_total[kNCls] = {}, tiles128 = 0;
  int fits = 0, present = 0;
  const bool fit = o->compute != PE_COMPUTE_F32 || planes_fit(o);
  int64_t prep_tiles = 0, most_prep = 0;
  bool f32m = false, small_only = true;
  for (int i = 0; i < count; ++i) {
    const pe_matrix& m = mats[i];
    Shape q{};
    q.prec = kBF16;
    q.bt = q.sbt = kTileSmall;
    if (m.m > 0 && m.n > 0) {
      q.s = std::min(m.m, m.n);
      q.L = std::max(m.m, m.n);
      q.prec = prec_for(o, m, fit);
      q.bt = q.sbt = tile_for(o, q.prec, q.s, q.L, batch_regime, upd256);
      // (e4m3 steps convert their operands on the 128 tile while staging them)
      q.family = q.prec == kF32 || q.prec == kTiny || (q.prec == kBF16 && q.bt == kTileSmall && !fp8);
      q.res = fits_resident(o, q.prec, q.s, q.L);
      ++present;
      fits += q.res;
    }
    sh.push_back(q);
  }
  const bool resident = fits == present || fits >= kResidentMany || alike(o);
  for (auto& q : sh) {
    q.res = q.res && resident;
    if (q.res) L->resident = true;
    else if (q.s > 0 && q.family) tiles128 += (q.s + 127) / 128 * ((q.L + 127) / 128);
  }
  // 256-wide updates go with 128-wide symmetric products where those take fewer
  // rounds: a 256 tile per CU, or two 128 tiles, which do a fourth of its work
  // each and take 1.15 times as long for it.  (Per call, 256 against 128: one
  // 3584 x 3584, 105 and 406 tiles: 1361 and 1132 us; 1024 x 4096 x 12, 120 and
  // 432: 1442 and 1257; one 4096 x 4096, 136 and 528: 1656 and 1779; 3072 x 3072 x
  // 6, 468 and 1800: 3787 and 4158.)  Always up to three tiles of 256 per side,
  // where half of every diagonal tile is work done twice (48 GPT-small matrices:
  // 2.51 against 2.77 ms per call).  A tile forced by the caller stays as it is.
  auto mixed = [&](const Shape& q) { return q.prec == kBF16 && q.bt == kTileLarge && !fp8; };
  int64_t n128 = 0, n256 = 0;
  auto fewer_rounds = [&]() { return o->tile == 0 && 1.15 * (2 * ((n128 + 511) / 512)) < 4.0 * ((n256 + 255) / 256); };
  auto count_tiles = [&](const Shape& q) {
    const int64_t b = (q.s + 255) / 256;
    n256 += b * (b + 1) / 2;
    n128 += b * (2 * b + 1);
  };
  for (const auto& q : sh)
    if (mixed(q) && q.s > 768) count_tiles(q);
  bool syrk128 = fewer_rounds();
  // second pass: the small family's tiles, padded shapes and tile counts
  for (int i = 0; i < count; ++i) {
    Shape& q = sh[i];
    if (q.s > 0 && !q.res) {
      if (alike(o)) {  // as in a call of its own
        tiles128 = (q.s + 127) / 128 * ((q.L + 127) / 128);
        n128 = n256 = 0;
        count_tiles(q);
        syrk128 = fewer_rounds();
      }
      if (q.family) small_tiles(q.prec, q.s, q.L, tiles128, &q.bt, &q.sbt);
      if (mixed(q) && (q.s <= 768 || syrk128)) q.sbt = kTileSmall;
      const int bt = q.bt;
      q.sp = round_up(q.s, bt);
      q.Lp = round_up(q.L, bt);
      q.nb = (int)(q.sp / bt);
      q.nbL = (int)(q.Lp / bt);
      q.nbs = (int)(q.sp / q.sbt);
      q.syrk = q.nbs * (q.nbs + 1) / 2;
      q.upd = q.nb * q.nbL;
      q.prep = (int)((q.sp / kPrepTile) * (q.Lp / kPrepTile));  // tiles; items below
      prep_tiles += q.prep;
      f32m = f32m || q.prec == kF32M;
      small_only = small_only && q.bt != kTileLarge && q.prec != kF32M && !(q.prec == kBF16 && !q.family);
    }
    q.cls = cls_of(q.prec, q.bt);
    q.scls = cls_of(q.prec, q.sbt);
    syrk_total[q.scls] += q.syrk;
    L->prec[i] = q.prec;
    L->bt[i] = q.bt;
  }
  // Norm-pass items: one tile each in small calls, where a four-tile item would
  // run its loads one after another on an idle chip (768 x 768: 12 -> 8 us), four
  // otherwise; FP32 MFMA keeps its four, and with them the bits of its norm.
  // Without the finalize launch (4.8 us) when every matrix runs the small tiles
  // and has few partial sums.
  L->prep_group = prep_tiles <= 1024 && !f32m && !alike(o) ? 1 : kPrepGroup;
  for (auto& q : sh) {
    q.prep = (q.prep + L->prep_group - 1) / L->prep_group;
    most_prep = std::max<int64_t>(most_prep, q.prep);
  }
  L->fold_norm = small_only && most_prep <= kFoldPartials && !learned_mode(o) && !alike(o);
  L->alike = alike(o);
  int want[kNCls];
  for (int c = 0; c < kNCls; ++c)
    want[c] = syrk_total[c] > 0 ? (int)std::min<int64_t>(64, (kFillTarget + syrk_total[c] - 1) / syrk_total[c]) : 1;
  size_t off = 0;
  L->descs_off = off;
  off += sizeof(MatDesc) * (size_t)std::max(count, 1);
  L->offs_off = off;  // right behind the descriptors: one upload carries both
  off = align_up(off + sizeof(int32_t) * ((size_t)PH_N * kNCls * (count + 1) + (size_t)kNCls * count));
  const bool learned = learned_mode(o);
  L->coef_off = off;
  if (learned) off = align_up(off + sizeof(float) * kClasses * 3 * (size_t)o->T + sizeof(int32_t) * kClasses);
  L->sel_off = off;
  if (learned) off = align_up(off + sizeof(int32_t) * kSelWords * (size_t)std::max(count, 1));
  for (int i = 0; i < count; ++i) {
    const pe_matrix& m = mats[i];
    const Shape& q = sh[i];
    const int prec = q.prec, bt = q.bt;
    // operand bytes per element (kTiny: its fp32 arrays are the operands)
    const size_t esz = prec == kTiny ? 0 : prec == kBF16 ? 2 : 4;
    const bool q8 = prec == kBF16 && o->compute == PE_COMPUTE_FP8 && o->fp8_steps > 0 && bt == kTileLarge;
    MatDesc d;
    memset(&d, 0, sizeof d);
    d.G = m.G;
    d.Out = m.X;
    d.ldg = m.ldg;
    d.ldo = m.ldx;
    d.M = m.M;
    d.ldm = m.ldm;
    d.W = m.W;
    d.ldw = m.ldw;
    d.w_bf16 = m.W && m.w_dtype == PE_BF16;
    d.m = (int32_t)m.m;
    d.n = (int32_t)m.n;
    d.s = (int32_t)q.s;
    d.L = (int32_t)q.L;
    d.sp = (int32_t)q.sp;
    d.Lp = (int32_t)q.Lp;
    d.trans = m.m > m.n;
    d.g_bf16 = m.g_dtype == PE_BF16;
    // 16-byte loads of G rows need an aligned base and a leading dimension
    // that keeps every row 16-byte aligned
    {
      const int64_t per16 = d.g_bf16 ? 8 : 4;
      d.g_vec = ((uintptr_t)m.G % 16 == 0) && (m.ldg % per16 == 0);
    }
    // the first update reads X_0 from its bf16 copy when that copy is exact;
    // a first update that is also the last (one step) reads both halves
    d.x0b = prec == kBF16 && d.g_bf16 && !m.M && o->T + (o->spectral_init > 0 ? 1 : 0) >= 2;
    d.out_bf16 = m.X && m.x_dtype == PE_BF16;
    d.o_vec = d.out_bf16 && ((uintptr_t)m.X % 16 == 0) && (m.ldx % 8 == 0);
    d.nb = q.nb;
    d.nbL = q.nbL;
    d.nbs = q.nbs;
    d.n_prep = q.prep;
    d.syrk_nt = q.syrk;
    d.upd_nt = q.upd;
    // split-K: enough Gram-side items to fill the GPU, at least 4 k-stages per
    // split of the Gram; A^2 (k = s, short) splits only with 16 k-stages per
    // split, since its reduce also runs the combine epilogue (on one 4096 x
    // 1024 bf16 matrix a two-way A^2 split took 12 us plus 22 us of reduce)
    const int bk = prec == kF32M ? 32 : 64;
    // (the 64 tile already shares k out among its four waves: 1024 k per part)
    const int max_gram = std::max<int64_t>(1, q.Lp / (q.sbt == kTileTiny ? 1024 : 4 * bk));
    const int max_a2 = std::max<int64_t>(1, q.sp / (16 * bk));
    const int cap = o->split_k > 0 ? o->split_k : 64;
    d.gram_split = q.syrk ? std::min(std::min(want[q.scls], max_gram), cap) : 1;
    d.a2_split = q.syrk ? std::min(std::min(want[q.scls], max_a2), cap) : 1;
    const size_t begin = off;
    if (q.syrk) {
      auto take = [&](size_t bytes) {
        char* p = ws ? ws + off : nullptr;
        off = align_up(off + bytes);
        return (void*)p;
      };
      const size_t X = (size_t)q.sp * q.Lp, A = (size_t)q.sp * q.sp;
      if (prec == kBF16) d.Xl = (uint16_t*)take(X * 2);
      else d.Xf = (float*)take(X * 4);
      d.Xb = take(X * esz);
      d.Xb1 = take(X * esz);
      // A in FP32 on the fp32 path; the bf16 paths keep only its bf16 copy,
      // which both A^2 and the bA term of the combine read
      // (bf16 paths: an FP32 A only for the spectrum-aware init's power method)
      // (the fp32 path's planes of A lie in the idle copy of X)
      if (o->fast_restart == 0) {
        d.Af = (is_f32(prec) || o->spectral_init > 0) ? (float*)take(A * 4) : nullptr;
        d.As = prec == kBF16 ? take(A * 2) : nullptr;
        d.Bs = take(A * (prec == kBF16 ? 2 : 4));
      }
      const int split = std::max(d.gram_split, d.a2_split);
      d.part = split > 1 ? (float*)take((size_t)q.syrk * split * q.sbt * q.sbt * 4) : nullptr;
      d.red = (double*)take((size_t)q.prep * 12 + 16);
      d.scal = (float*)take(kScN * 4);
      d.cnt = (uint32_t*)take(64);  // reserved
      d.trp = (float*)take((size_t)q.syrk * 2 * 4);
      // e4m3 operand copies of the FP8 steps (256 tile)
      if (q8) {
        d.Xq = (uint8_t*)take(X);
        d.Aq = (uint8_t*)take(A);
      }
      if (o->fast_restart > 0) {
        // both D share their fp32 values, which a product replaces in place; a
        // kTiny or kF32M product reads them as operands, and has no planes (kF32M
        // still takes their room, one of them for the second D: which of the two
        // a matrix runs depends on the schedule, its workspace does not)
        for (int k = 0; k < 5; ++k) {
          d.fb[k] = k == kFbD1 && prec != kTiny ? d.fb[kFbD0] : (float*)take(A * 4);
          d.fbp[k] = prec != kTiny && k != kFbP ? (uint16_t*)take(A * 4) : nullptr;
        }
        if (prec == kF32M) d.fb[kFbD1] = (float*)d.fbp[kFbD1];
        // pe_plan_launch_phase runs the ordinary iteration's phases on any plan
        d.Af = d.fb[kFbR];
        d.Bs = d.fb[kFbB];
      }
      if (o->spectral_init > 0 && !learned) d.vec = (float*)take(((size_t)2 * q.sp + q.Lp) * 4);
      if (learned) {
        int32_t* rec = ws ? (int32_t*)(ws + L->sel_off) + (size_t)i * kSelWords : nullptr;
        d.selp = rec;
        d.flagp = rec ? rec + 1 : nullptr;
        d.feat = rec ? (float*)(rec + 16) : nullptr;
        d.est = rec ? (float*)(rec + 32) : nullptr;
        d.A2f = (float*)take(A * 4);
        d.mom = (float*)take((size_t)q.syrk * 4 * 4);
        d.vec = (float*)take(((size_t)2 * q.sp + q.Lp) * 4);
      }
    }
    // Callers size and share workspaces by shape and compute type alone, and the
    // static scratch admits matrices by this size: whatever tile or kernel a
    // matrix gets, it is at least an FP32 iterate with two operand copies and A
    // and B (fast iteration: eight s x s matrices), padded to the 128 (or its 256) tile.
    if (q.s > 0) {
      const int pad = std::max(bt, (int)kTileSmall);
      const size_t S = round_up(q.s, pad), XX = S * round_up(q.L, pad), per = o->compute == PE_COMPUTE_F32 ? 4 : 2;
      off = std::max(off, begin + align_up(XX * (4 + 2 * per) + S * S * (o->fast_restart > 0 ? 32 : 2 * per)));
    }
    L->descs.push_back(d);
    // this matrix's items in its class's tables, none in the others
    auto push_to = [&](int ph, int cls, int n) {
      for (int c = 0; c < kNCls; ++c) L->offs[ph][c].push_back(L->offs[ph][c].back() + (c == cls ? n : 0));
    };
    auto push = [&](int ph, int n) { push_to(ph, q.cls, n); };
    auto push_s = [&](int ph, int n) { push_to(ph, q.scls, n); };  // symmetric products
    auto push_all = [&](int ph, int n) {
      for (int c = 0; c < kNCls; ++c) L->offs[ph][c].push_back(L->offs[ph][c].back() + (c == 0 ? n : 0));
    };
    push(PH_PREP, q.syrk ? q.prep : 0);
    push_to(PH_RES, (int)((q.L + 255) / 256) - 1, q.res ? 1 : 0);  // class slot: bucket of L
    push_s(PH_GRAM, q.syrk ? q.syrk * d.gram_split : 0);
    push_s(PH_A2, q.syrk ? q.syrk * d.a2_split : 0);
    push(PH_UPD, q.syrk ? q.upd : 0);
    // spectrum-aware init: power-method rows, four per item
    push(PH_PW, (q.syrk && o->spectral_init > 0) ? (int)((q.sp + 3) / 4) : 0);
    // fast rectangular iteration: unsplit upper-triangle tiles
    push_s(PH_FSYRK, (q.syrk && o->fast_restart > 0) ? q.syrk : 0);
    push(PH_PLANES, (q.syrk && prec == kF32) ? (int)(((size_t)q.sp * q.Lp + 16383) / 16384) : 0);
    push_s(PH_RGRAM, (q.syrk && d.gram_split > 1) ? q.syrk : 0);
    push_s(PH_RA2, (q.syrk && d.a2_split > 1) ? q.syrk : 0);
    // rows of B formed from a kept A^2 (learned path) or A (init step)
    push(PH_COMBINE, (q.syrk && (learned || (o->spectral_init > 0 && prec == kBF16))) ? (int)q.sp : 0);
    // quantisation passes: 16384 elements per item (sizes are multiples of 65536)
    push(PH_QX, (q.syrk && q8) ? (int)((size_t)q.sp * q.Lp / 16384) : 0);
    push(PH_QA, (q.syrk && q8) ? (int)((size_t)q.sp * q.sp / 16384) : 0);
    // power iteration: w = X^T v (length L), then y = X w (length s); a product
    // along the rows of the caller's m x n output takes one wave per row (4 per
    // block), one across its columns 64 columns per block
    {
      const bool t = m.m > m.n;
      const int rows4 = (int)((m.m + 3) / 4), cols64 = (int)((m.n + 63) / 64);
      push_all(PH_EST_A, (q.syrk && learned) ? (t ? rows4 : cols64) : 0);
      push_all(PH_EST_B, (q.syrk && learned) ? (t ? cols64 : rows4) : 0);
    }
  }
  // the first update reads X_0 from its bf16 copy only when every bf16-path
  // matrix of the call can (one kernel per launch, no per-matrix branch)
  {
    bool all = true;
    for (size_t i = 0; i < L->descs.size(); ++i)
      if (L->prec[i] == kBF16 && L->descs[i].syrk_nt > 0) all = all && L->descs[i].x0b;
    for (auto& d : L->descs) d.x0b = all ? d.x0b : 0;
    L->x0b = all;
  }
  for (int c = 0; c < kNCls; ++c) {
    // Gram phase in longest-k-first matrix order (stable)
    std::vector<int32_t> ord(count);
    for (int i = 0; i < count; ++i) ord[i] = i;
    std::stable_sort(ord.begin(), ord.end(), [&](int x, int y) { return sh[x].Lp > sh[y].Lp; });
    std::vector<int32_t> o2(1, 0);
    for (int k = 0; k < count; ++k) {
      const int i = ord[k];
      o2.push_back(o2.back() + (L->offs[PH_GRAM][c][i + 1] - L->offs[PH_GRAM][c][i]));
    }
    L->offs[PH_GRAM][c].swap(o2);
    L->ord_gram[c].swap(ord);
  }
  int32_t words = 0;
  for (int c = 0; c < kNCls; ++c) {
    bool sorted = true;
    for (int k = 0; k < count; ++k) sorted = sorted && L->ord_gram[c][k] == k;
    L->tab_ord[c] = !sorted && L->offs[PH_GRAM][c].back() ? words : -1;
    if (L->tab_ord[c] >= 0) words += count;
  }
  for (int p = 0; p < PH_N; ++p)
    for (int c = 0; c < kNCls; ++c) {
      L->totals[p][c] = L->offs[p][c].back();
      L->tab[p][c] = L->totals[p][c] ? words : -1;
      if (L->totals[p][c]) words += count + 1;
    }
  L->bytes = off;
  return PE_OK;
}

// Items of a phase over all classes (zero: nothing to launch).
int32_t phase_total(const Layout& L, int ph) {
  int32_t t = 0;
  for (int c = 0; c < kNCls; ++c) t += L.totals[ph][c];
  return t;
}

pe_status validate(int count, const pe_matrix* mats, const pe_opts* o) {
  if (count < 0 || (count > 0 && !mats)) return PE_EINVAL;
  if (count > 100000) return PE_EINVAL;
  pe_status st = check_opts(o);
  if (st != PE_OK) return st;
  bool muon = false;
  for (int i = 0; i < count; ++i) {
    if (!valid_matrix(mats[i])) return PE_EINVAL;
    muon = muon || mats[i].M || mats[i].W;
  }
  // the fallback re-run would apply the momentum and the weight step twice,
  // and its estimate reads X
  if (muon && learned_mode(o) && o->fallback_tau > 0.0f) return PE_EUNSUPPORTED;
  return PE_OK;
}

// Copy host words to device memory through kernel arguments (stream-ordered).
pe_status put_words(void* dst, const void* src, size_t bytes, hipStream_t st) {
  const uint32_t* w = (const uint32_t*)src;
  size_t nw = (bytes + 3) / 4;
  uint32_t* d = (uint32_t*)dst;
  while (nw > 0) {
    PutChunk c;
    memset(&c, 0, sizeof c);
    const int n = (int)std::min<size_t>(nw, kPutWords);
    c.dst = d;
    c.nwords = n;
    memcpy(c.w, w, (size_t)n * 4);
    hipError_t e = launch_put(c, st);
    if (e != hipSuccess) return hip_fail(e, "upload");
    d += n;
    w += n;
    nw -= n;
  }
  return PE_OK;
}

}  // namespace

struct pe_plan {
  int count = 0;
  int fp8_steps = 0;   // leading steps whose Gram-side products take e4m3 operands
  int T = 0;
  int norm_mode = 0;
  float muon_beta = 0.0f, muon_lr = 0.0f, muon_wd = 0.0f;
  int spectral_init = 0;    // > 0: power steps of the spectrum-aware init step
  int t0 = 0;               // kernel steps before the schedule (1 with the init step)
  int fast_restart = 0;     // > 0: Algorithm 4 in segments of this many steps
  float fast_eps = 0.0f;
  std::vector<float> abc;
  // fp32 path: scales of the operand planes of X_t, A_t and B_t per kernel step
  std::vector<float> sx, sa, sb;
  std::vector<float> sfast; // fast iteration: of each product's result, and of the next X after a segment
  bool learned = false;
  const float* mlp = nullptr;
  int force_class = -1;
  float tau = 0.0f;
  float* d_coef = nullptr;     // [classes][T][3]
  int32_t* d_steps = nullptr;  // [classes]: T' of each class
  Layout L;
  MatDesc* d_descs = nullptr;
  int32_t* d_offs = nullptr;
  hipStream_t cap_stream = nullptr;
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
};

namespace {

// The schedule of every class of a learned plan (class 4 is the caller's), rows
// past a class's T' the identity step (1, 0, 0); otherwise the one schedule.
pe_status class_tables(const pe_plan* p, std::vector<std::vector<double>>* out) {
  out->clear();
  const std::vector<double> own(p->abc.begin(), p->abc.end());
  if (!p->learned) {
    out->push_back(own);
    return PE_OK;
  }
  for (int c = 0; c < kClasses; ++c) {
    std::vector<double> abc = own;
    if (c != kFixedClass) {
      // the first T' steps of the greedy T-step schedule are its T'-step schedule
      const pe_status s = pe_coeffs(kClassTable[c].ell, p->T, nullptr, abc.data(), nullptr, nullptr, nullptr);
      if (s != PE_OK) return s;
    }
    for (int t = class_steps(c, p->T); t < p->T; ++t) {
      abc[3 * t] = 1.0;
      abc[3 * t + 1] = abc[3 * t + 2] = 0.0;
    }
    out->push_back(abc);
  }
  return PE_OK;
}

pe_status upload(pe_plan* p, char* ws, const std::vector<std::vector<double>>& tables, hipStream_t st) {
  p->d_descs = (MatDesc*)(ws + p->L.descs_off);
  p->d_offs = (int32_t*)(ws + p->L.offs_off);
  std::vector<uint32_t> words(sizeof(MatDesc) / 4 * p->L.descs.size());
  memcpy(words.data(), p->L.descs.data(), sizeof(MatDesc) * p->L.descs.size());
  auto put = [&](const std::vector<int32_t>& t) { words.insert(words.end(), t.begin(), t.end()); };
  for (int c = 0; c < kNCls; ++c)
    if (p->L.tab_ord[c] >= 0) put(p->L.ord_gram[c]);
  for (int ph = 0; ph < PH_N; ++ph)
    for (int c = 0; c < kNCls; ++c)
      if (p->L.tab[ph][c] >= 0) put(p->L.offs[ph][c]);
  pe_status s = put_words(p->d_descs, words.data(), words.size() * 4, st);
  if (s != PE_OK || !p->learned) return s;
  // the classes' schedules, then their T'
  const size_t nt = (size_t)kClasses * p->T * 3;
  std::vector<uint32_t> tab(nt + kClasses);
  float* ft = (float*)tab.data();
  for (int c = 0; c < kClasses; ++c) {
    for (int k = 0; k < 3 * p->T; ++k) ft[(size_t)c * p->T * 3 + k] = (float)tables[c][k];
    ((int32_t*)tab.data())[nt + c] = class_steps(c, p->T);
  }
  p->d_coef = (float*)(ws + p->L.coef_off);
  p->d_steps = (int32_t*)(p->d_coef + nt);
  return put_words(p->d_coef, tab.data(), tab.size() * 4, st);
}

KArgs base_args(const pe_plan* p) {
  KArgs a;
  memset(&a, 0, sizeof a);
  a.descs = p->d_descs;
  a.count = p->count;
  a.norm_mode = p->norm_mode;
  a.prep_group = p->L.prep_group;
  a.fold_norm = p->L.fold_norm;
  a.alike = p->L.alike;
  a.tail = -1;
  a.tmax = p->T;
  a.mbeta = p->muon_beta;
  a.mlr = p->muon_lr;
  a.mwd = p->muon_wd;
  if (p->learned) {
    a.sel_coef = p->d_coef;
    a.sel_steps = p->d_steps;
    a.mlp = p->mlp;
    a.force_class = p->force_class;
    a.fixed_class = kFixedClass;
    a.tau = p->tau;
  }
  return a;
}

const int32_t* offs_ptr(const pe_plan* p, int ph, int c) {
  return p->L.tab[ph][c] >= 0 ? p->d_offs + p->L.tab[ph][c] : nullptr;
}

void set_phase(const pe_plan* p, KArgs* a, int ph, int c) {
  a->offs = offs_ptr(p, ph, c);
  a->ord = ph == PH_GRAM && p->L.tab_ord[c] >= 0 ? p->d_offs + p->L.tab_ord[c] : nullptr;
  a->total = p->L.totals[ph][c];
}

// kernel step t: the init step (t < t0) or schedule step t - t0
void set_step(const pe_plan* p, KArgs* a, int t) {
  a->t = t;
  a->last = t == p->T + p->t0 - 1;
  if (t < p->t0) {
    a->init_step = 1;
    a->a = a->b = a->c = 0.0f;  // (a, b) per matrix from the power bound; c = 0
    return;
  }
  a->a = p->abc[3 * (t - p->t0) + 0];
  a->b = p->abc[3 * (t - p->t0) + 1];
  a->c = p->abc[3 * (t - p->t0) + 2];
}

pe_status enqueue_norm(const pe_plan* p, hipStream_t st, int fallback = 0) {
  KArgs a = base_args(p);
  a.fallback = fallback;
  hipError_t e;
  for (int c = 0; c < kNCls; ++c) {
    if (!p->L.totals[PH_PREP][c]) continue;
    set_phase(p, &a, PH_PREP, c);
    if ((e = launch_prep(cls_prec(c), a, kPrepGridCap, st)) != hipSuccess) return hip_fail(e, "prep launch");
  }
  if (!p->L.fold_norm && (e = launch_finalize(a, st)) != hipSuccess) return hip_fail(e, "finalize launch");
  // fp32 path: operand planes of X_0, now that the norm is known
  a.oscale = p->sx[0];
  for (int c = 0; c < kNCls; ++c) {
    if (!p->L.totals[PH_PLANES][c]) continue;
    set_phase(p, &a, PH_PLANES, c);
    if ((e = launch_planes(a, st)) != hipSuccess) return hip_fail(e, "planes launch");
  }
  return PE_OK;
}

// kind: 0 Gram, 1 A^2 + combine, 2 update; one launch (plus its split-K
// reduction) per class present
pe_status enqueue_gemm(const pe_plan* p, int t, int kind, hipStream_t st, int fallback = 0) {
  static const int ph_main[3] = {PH_GRAM, PH_A2, PH_UPD};
  static const int ph_red[3] = {PH_RGRAM, PH_RA2, -1};
  static const char* names[3] = {"gram launch", "a2 launch", "update launch"};
  for (int c = 0; c < kNCls; ++c) {
    if (t < p->t0 && kind == 1 && cls_prec(c) == kBF16) {
      if (!p->L.totals[PH_COMBINE][c]) continue;
      KArgs a = base_args(p);
      set_phase(p, &a, PH_COMBINE, c);
      const hipError_t e = launch_init_b(a, st);
      if (e != hipSuccess) return hip_fail(e, "init step's B");
      continue;
    }
    if (!p->L.totals[ph_main[kind]][c]) continue;
    const int bt = cls_bt(c);
    KArgs a = base_args(p);
    set_step(p, &a, t);
    set_phase(p, &a, ph_main[kind], c);
    // e4m3 Gram-side products in the first fp8_steps steps, bf16 matrices only
    const bool q = cls_prec(c) == kBF16;
    a.fp8 = q && t < p->fp8_steps;
    a.fp8_next = q && t + 1 < p->fp8_steps;
    a.fallback = fallback;
    a.x0b = kind == 2 && t == 0 && p->L.x0b;
    // learned path, step 1: A^2 and its moments are kept until the class is chosen
    a.raw_a2 = p->learned && !fallback && t == 0 && kind == 1;
    if (cls_prec(c) == kF32) {
      const float sp = kind == 0 ? p->sx[t] : kind == 1 ? p->sa[t] : p->sb[t], sq = kind == 1 ? p->sa[t] : p->sx[t];
      a.deq = 1.0f / sp / sq;
      a.oscale = kind == 0 ? p->sa[t] : kind == 1 ? p->sb[t] : p->sx[t + 1];
    }
    // Gram-side products of the FP8 steps run the e4m3 kernels; updates stay bf16
    const int prec = (a.fp8 && kind != 2) ? kFP8 : cls_prec(c);
    hipError_t e;
    if (prec == kFP8 && bt == kTileLarge) {
      // the 256 tile reads e4m3 copies: quantise X_t (or A_t) with its scale first
      set_phase(p, &a, kind == 0 ? PH_QX : PH_QA, c);
      if ((e = launch_quant(kind, a, kQuantGridCap, st)) != hipSuccess) return hip_fail(e, "quantisation launch");
      set_phase(p, &a, ph_main[kind], c);
    }
    const bool small = prec == kF32 || prec == kTiny || (prec == kBF16 && bt != kTileLarge);
    e = prec == kF32M ? launch_f32_gemm(kind, a, st)
        : small ? launch_small_gemm(prec, bt, kind, a, st)
              : launch_gemm(prec, bt, kind, a, bt == kTileLarge ? kGemmGridCapLarge : kGemmGridCap, st);
    if (e != hipSuccess) return hip_fail(e, names[kind]);
    if (ph_red[kind] >= 0 && p->L.totals[ph_red[kind]][c]) {
      set_phase(p, &a, ph_red[kind], c);
      e = prec == kF32M ? launch_f32_reduce(kind, a, st)
          : small ? launch_small_reduce(prec, bt, kind, a, st) : launch_reduce(prec, bt, kind, a, kReduceGridCap, st);
      if (e != hipSuccess) return hip_fail(e, "split-k reduce");
    }
  }
  return PE_OK;
}

// learned path between step 1's A^2 and its update: choose the class, form B
pe_status enqueue_select(const pe_plan* p, hipStream_t st) {
  KArgs a = base_args(p);
  set_step(p, &a, 0);
  hipError_t e = launch_select(a, st);
  if (e != hipSuccess) return hip_fail(e, "select launch");
  for (int c = 0; c < kNCls; ++c) {
    if (!p->L.totals[PH_COMBINE][c]) continue;
    set_phase(p, &a, PH_COMBINE, c);
    a.oscale = p->sb[0];
    if ((e = launch_combine(cls_prec(c), a, st)) != hipSuccess) return hip_fail(e, "combine launch");
  }
  return PE_OK;
}

// Algorithm 4 in segments of fast_restart steps (FP32 classes only): per
// segment the Gram matrix, then per step B_t, D_t and (but for the last step)
// R_{t+1}, and the update X <- q X + D X; see small_fast_kernel.
pe_status enqueue_fast(const pe_plan* p, hipStream_t st) {
  pe_status s = enqueue_norm(p, st, 0);
  if (s != PE_OK) return s;
  hipError_t e;
  const float* next = p->sfast.data();
  float sx = p->sx[0], scale[5] = {};
  // kind 0: Gram of X, 1: symmetric product of two fb buffers
  auto product = [&](int seg, int kind, int fp_, int fq_, int fe1, float c1, int fe2, float c2, float cacc, int fout,
                     float cdiag) -> pe_status {
    KArgs a = base_args(p);
    a.t = seg;
    a.fast = 1;
    a.fp_ = fp_;
    a.fq_ = fq_;
    a.fe1 = fe1;
    a.fe2 = fe2;
    a.c1 = c1;
    a.c2 = c2;
    a.cacc = cacc;
    a.fout = fout;
    a.cdiag = cdiag;
    const float deq = kind == 0 ? 1.0f / sx / sx : 1.0f / scale[fp_] / scale[fq_];
    a.oscale = scale[fout] = *next++;
    for (int c = 0; c < kNCls; ++c) {
      if (!p->L.totals[PH_FSYRK][c]) continue;
      set_phase(p, &a, PH_FSYRK, c);
      a.deq = cls_prec(c) == kF32 ? deq : 1.0f;
      e = cls_prec(c) == kF32M ? launch_f32_fast(kind, a, st) : launch_fast(cls_prec(c), cls_bt(c), kind, a, st);
      if (e != hipSuccess) return hip_fail(e, "fast product");
    }
    return PE_OK;
  };
  // X <- q X + D X
  auto update = [&](int seg, bool last, float q, int dcur) -> pe_status {
    KArgs a = base_args(p);
    a.t = seg;
    a.last = last;
    a.a = q;
    a.b = a.c = 0.0f;
    a.fast = 1;
    a.fp_ = dcur;
    a.deq = 1.0f / scale[dcur] / sx;
    a.oscale = sx = *next++;
    for (int c = 0; c < kNCls; ++c) {
      if (!p->L.totals[PH_UPD][c]) continue;
      set_phase(p, &a, PH_UPD, c);
      e = cls_prec(c) == kF32M ? launch_f32_gemm(2, a, st) : launch_small_gemm(cls_prec(c), cls_bt(c), 2, a, st);
      if (e != hipSuccess) return hip_fail(e, "fast update");
    }
    return PE_OK;
  };
  return fast_walk(p->abc.data(), p->T, p->fast_restart, p->fast_eps, product, update);
}

// power method on each matrix's step-1 Gram matrix and the init coefficients
pe_status enqueue_power(const pe_plan* p, hipStream_t st) {
  KArgs a = base_args(p);
  hipError_t e;
  for (int it = 0; it < p->spectral_init; ++it) {
    a.est_phase = it;
    for (int c = 0; c < kNCls; ++c) {
      if (!p->L.totals[PH_PW][c]) continue;
      set_phase(p, &a, PH_PW, c);
      if ((e = launch_power(0, a, st)) != hipSuccess) return hip_fail(e, "power step");
    }
  }
  a.est_phase = p->spectral_init;
  if ((e = launch_power(1, a, st)) != hipSuccess) return hip_fail(e, "init coefficients");
  return PE_OK;
}

// all steps of the matrices that fit one compute unit
pe_status enqueue_resident(const pe_plan* p, hipStream_t st) {
  if (!p->L.resident) return PE_OK;
  ResSchedule sc;
  sc.T = p->T;
  for (int i = 0; i < 3 * p->T; ++i) sc.abc[i] = p->abc[i];
  KArgs a = base_args(p);
  hipError_t e;
  for (int b = 0; b < 4; ++b) {
    if (!p->L.totals[PH_RES][b]) continue;
    set_phase(p, &a, PH_RES, b);
    if ((e = launch_resident(b, a, sc, st)) != hipSuccess) return hip_fail(e, "resident launch");
  }
  return PE_OK;
}

pe_status enqueue_steps(const pe_plan* p, hipStream_t st, int fallback) {
  if (p->fast_restart > 0) return enqueue_fast(p, st);
  pe_status s = enqueue_norm(p, st, fallback);
  if (s != PE_OK) return s;
  for (int t = 0; t < p->T + p->t0; ++t)
    for (int kind = 0; kind < 3; ++kind) {
      if (t < p->t0 && kind == 1 && (s = enqueue_power(p, st)) != PE_OK) return s;
      if ((s = enqueue_gemm(p, t, kind, st, fallback)) != PE_OK) return s;
      if (p->learned && !fallback && t == 0 && kind == 1 && (s = enqueue_select(p, st)) != PE_OK)
        return s;
    }
  return PE_OK;
}

pe_status enqueue(const pe_plan* p, hipStream_t st) {
  pe_status s = enqueue_resident(p, st);
  if (s != PE_OK || phase_total(p->L, PH_PREP) == 0) return s;
  s = enqueue_steps(p, st, 0);
  if (s != PE_OK || !p->learned || !(p->tau > 0.0f)) return s;
  // estimate ||X X^T - I||_2 of every result; re-run the failed ones with class 4
  KArgs a = base_args(p);
  hipError_t e = launch_est(a, kEstIters, st, offs_ptr(p, PH_EST_A, 0), p->L.totals[PH_EST_A][0],
                            offs_ptr(p, PH_EST_B, 0), p->L.totals[PH_EST_B][0]);
  if (e != hipSuccess) return hip_fail(e, "estimate launch");
  return enqueue_steps(p, st, 1);
}

pe_status plan_init(pe_plan* p, int count, const pe_matrix* mats, const pe_opts* o, void* ws,
                    size_t ws_bytes, hipStream_t st) {
  pe_status s = validate(count, mats, o);
  if (s != PE_OK) return s;
  p->count = count;
  p->fp8_steps = o->compute == PE_COMPUTE_FP8 ? o->fp8_steps : 0;
  p->T = o->T;
  p->norm_mode = o->norm_mode;
  p->spectral_init = o->spectral_init;
  p->t0 = o->spectral_init > 0 ? 1 : 0;
  p->muon_beta = o->muon_beta;
  p->muon_lr = o->muon_lr;
  p->muon_wd = o->muon_wd;
  p->fast_restart = o->fast_restart;
  p->fast_eps = o->fast_eps;
  p->abc.resize(3 * o->T);
  for (int i = 0; i < 3 * o->T; ++i) p->abc[i] = (float)o->abc[i];
  p->learned = learned_mode(o);
  p->mlp = o->predictor;
  p->force_class = o->force_class;
  p->tau = o->fallback_tau;
  Layout sizing;
  build_layout(count, mats, o, nullptr, &sizing);
  if (phase_total(sizing, PH_PREP) == 0 && !sizing.resident) return PE_OK;  // nothing but empty matrices
  if (!ws || ((uintptr_t)ws & 255) || ws_bytes < sizing.bytes) return PE_EWORKSPACE;
  build_layout(count, mats, o, (char*)ws, &p->L);
  warm_launch_grids();
  std::vector<std::vector<double>> tables;
  s = class_tables(p, &tables);
  if (s != PE_OK) return s;
  const PlaneBounds bounds = plane_bounds(tables, p->T, p->t0);
  for (double v : bounds.x) p->sx.push_back(plane_scale(v));
  for (double v : bounds.a) p->sa.push_back(plane_scale(v));
  for (int t = 0; t < p->T + p->t0; ++t) p->sb.push_back(t < p->t0 ? 1.0f : plane_scale(bounds.b[t]));
  if (p->fast_restart > 0) {
    bool grew;
    for (double v : fast_bounds(p->abc.data(), p->T, p->fast_restart, p->fast_eps, &grew)) p->sfast.push_back(plane_scale(v));
  }
  return upload(p, (char*)ws, tables, st);
}

}  // namespace

// ------------------------------------------------ allocation-free entry point
// pe_polar_noalloc keeps its workspace in this file-scope device array instead
// of the caller's: one copy per device, allocated when the code object is
// loaded there and held until the process ends.  In host code `scratch` is
// only a stand-in for the symbol; its device address comes from
// hipGetSymbolAddress, queried once per device (with that device current) and
// cached.
static __device__ __align__(256) char scratch[PE_NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

pe_status scratch_address(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
  if (dev < 0 || dev >= kMaxDevices) {
    g_last_error = "device index beyond the scratch table";
    return PE_EUNSUPPORTED;
  }
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) return hip_fail(e, "hipGetSymbolAddress(scratch)");
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return PE_OK;
}
}  // namespace

// ----------------------------------------------------------------- C ABI
extern "C" {

size_t pe_workspace_size(int32_t count, const pe_matrix* mats, const pe_opts* opts) {
  if (validate(count, mats, opts) != PE_OK) return 0;
  Layout L;
  build_layout(count, mats, opts, nullptr, &L);
  return L.bytes;
}

pe_status pe_polar_batched(int32_t count, const pe_matrix* mats, const pe_opts* opts, void* ws,
                           size_t ws_bytes, void* stream) {
  g_last_error.clear();
  hipStream_t st = (hipStream_t)stream;
  pe_plan p;
  pe_status s = plan_init(&p, count, mats, opts, ws, ws_bytes, st);
  if (s != PE_OK) return s;
  return enqueue(&p, st);
}

pe_status pe_polar(const pe_matrix* mat, const pe_opts* opts, void* ws, size_t ws_bytes, void* stream) {
  if (!mat) return PE_EINVAL;
  return pe_polar_batched(1, mat, opts, ws, ws_bytes, stream);
}

pe_status pe_polar_noalloc(const pe_matrix* mat, const pe_opts* opts, void* stream) {
  g_last_error.clear();
  if (!mat) return PE_EINVAL;
  pe_status s = validate(1, mat, opts);
  if (s != PE_OK) return s;
  Layout sizing;
  build_layout(1, mat, opts, nullptr, &sizing);
  if (sizing.bytes > (size_t)PE_NOALLOC_SCRATCH_BYTES) {
    char buf[160];
    snprintf(buf, sizeof buf, "pe_polar_noalloc: this matrix needs %zu bytes of workspace, the static "
             "scratch holds %zu", sizing.bytes, (size_t)PE_NOALLOC_SCRATCH_BYTES);
    g_last_error = buf;
    return PE_EWORKSPACE;
  }
  void* ws = nullptr;
  if ((s = scratch_address(&ws)) != PE_OK) return s;
  return pe_polar(mat, opts, ws, (size_t)PE_NOALLOC_SCRATCH_BYTES, stream);
}

pe_status pe_plan_create(int32_t count, const pe_matrix* mats, const pe_opts* opts, void* ws,
                         size_t ws_bytes, void* stream, pe_plan** plan) {
  g_last_error.clear();
  if (!plan) return PE_EINVAL;
  *plan = nullptr;
  pe_plan* p = new pe_plan();
  pe_status s = plan_init(p, count, mats, opts, ws, ws_bytes, (hipStream_t)stream);
  if (s != PE_OK) {
    delete p;
    return s;
  }
  *plan = p;
  return PE_OK;
}

pe_status pe_plan_launch(pe_plan* p, void* stream, int32_t use_graph) {
  g_last_error.clear();
  if (!p) return PE_EINVAL;
  hipStream_t st = (hipStream_t)stream;
  if (!use_graph) return enqueue(p, st);
  hipError_t e;
  if (!p->exec) {
    // capture on a private stream (the caller's may be the legacy default stream)
    if ((e = hipStreamCreateWithFlags(&p->cap_stream, hipStreamNonBlocking)) != hipSuccess)
      return hip_fail(e, "capture stream");
    // order the capture after the caller's pending work (tables were uploaded there)
    if ((e = hipStreamSynchronize(st)) != hipSuccess) return hip_fail(e, "sync before capture");
    if ((e = hipStreamBeginCapture(p->cap_stream, hipStreamCaptureModeThreadLocal)) != hipSuccess)
      return hip_fail(e, "begin capture");
    pe_status s = enqueue(p, p->cap_stream);
    hipGraph_t g = nullptr;
    e = hipStreamEndCapture(p->cap_stream, &g);
    if (s != PE_OK) {
      if (g) hipGraphDestroy(g);
      return s;
    }
    if (e != hipSuccess) return hip_fail(e, "end capture");
    p->graph = g;
    if ((e = hipGraphInstantiate(&p->exec, g, nullptr, nullptr, 0)) != hipSuccess) {
      p->exec = nullptr;
      return hip_fail(e, "graph instantiate");
    }
  }
  if ((e = hipGraphLaunch(p->exec, st)) != hipSuccess) return hip_fail(e, "graph launch");
  return PE_OK;
}

pe_status pe_plan_launch_phase(pe_plan* p, int32_t step, int32_t phase, void* stream) {
  g_last_error.clear();
  if (!p || step < 0 || step >= p->T + p->t0 || phase < 0 || phase > 3) return PE_EINVAL;
  // a learned plan's step 1 also selects the class between its phases
  if (p->learned) return PE_EUNSUPPORTED;
  hipStream_t st = (hipStream_t)stream;
  if (step == p->T + p->t0 - 1 && phase == 3) {
    const pe_status s = enqueue_resident(p, st);
    if (s != PE_OK) return s;
  }
  if (phase_total(p->L, PH_PREP) == 0) return PE_OK;
  if (phase == 0) return enqueue_norm(p, st);
  return enqueue_gemm(p, step, phase - 1, st);
}

pe_status pe_plan_destroy(pe_plan* p) {
  if (!p) return PE_OK;
  if (p->exec) hipGraphExecDestroy(p->exec);
  if (p->graph) hipGraphDestroy(p->graph);
  if (p->cap_stream) hipStreamDestroy(p->cap_stream);
  delete p;
  return PE_OK;
}

pe_status pe_plan_selection(pe_plan* p, void* stream, int32_t* classes, float* feats, float* est,
                            int32_t* flags) {
  g_last_error.clear();
  if (!p) return PE_EINVAL;
  if (!p->learned) return PE_EINVAL;
  if (p->count == 0) return PE_OK;
  hipStream_t st = (hipStream_t)stream;
  std::vector<int32_t> rec((size_t)p->count * kSelWords);
  const char* src = (const char*)p->d_descs - p->L.descs_off + p->L.sel_off;
  hipError_t e = hipMemcpyAsync(rec.data(), src, rec.size() * 4, hipMemcpyDeviceToHost, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e != hipSuccess) return hip_fail(e, "selection copy");
  for (int i = 0; i < p->count; ++i) {
    const int32_t* r = rec.data() + (size_t)i * kSelWords;
    const bool run = p->L.descs[i].syrk_nt > 0;  // empty matrices have no record
    if (classes) classes[i] = run ? r[0] : -1;
    if (flags) flags[i] = run ? r[1] : 0;
    if (feats) {
      if (run) memcpy(feats + (size_t)i * kFeat, r + 16, kFeat * 4);
      else memset(feats + (size_t)i * kFeat, 0, kFeat * 4);
    }
    if (est) est[i] = run ? *(const float*)(r + 32) : 0.0f;
  }
  return PE_OK;
}

size_t pe_mlp_workspace_size(int32_t B) {
  if (B <= 0) return 0;
  const size_t nblk = (size_t)(B + 63) / 64;
  return align_up(nblk * kMlpParams * 4) + align_up(nblk * 4);
}

pe_status pe_mlp_forward(const float* params, const float* feats, int32_t B, float* logits,
                         void* stream) {
  g_last_error.clear();
  if (B < 0 || (B > 0 && (!params || !feats || !logits))) return PE_EINVAL;
  if (B == 0) return PE_OK;
  hipError_t e = launch_mlp_forward(params, feats, B, logits, (hipStream_t)stream);
  return e == hipSuccess ? PE_OK : hip_fail(e, "mlp forward");
}

static pe_status mlp_grad_common(const float* params, const float* feats, const int32_t* labels,
                                 int32_t B, float* grad, float* loss, float* upd, float* m, float* v,
                                 int32_t step, float lr, void* ws, size_t ws_bytes, void* stream) {
  g_last_error.clear();
  if (B <= 0 || !params || !feats || !labels) return PE_EINVAL;
  const size_t need = pe_mlp_workspace_size(B);
  if (!ws || ((uintptr_t)ws & 255) || ws_bytes < need) return PE_EWORKSPACE;
  const size_t nblk = (size_t)(B + 63) / 64;
  float* part = (float*)ws;
  float* part_loss = (float*)((char*)ws + align_up(nblk * kMlpParams * 4));
  hipError_t e = launch_mlp_grad(params, feats, labels, B, part, part_loss, grad, loss, upd, m, v,
                                 step, lr, (hipStream_t)stream);
  return e == hipSuccess ? PE_OK : hip_fail(e, "mlp grad");
}

pe_status pe_mlp_grad(const float* params, const float* feats, const int32_t* labels, int32_t B,
                      float* grad, float* loss, void* ws, size_t ws_bytes, void* stream) {
  if (!grad) return PE_EINVAL;
  return mlp_grad_common(params, feats, labels, B, grad, loss, nullptr, nullptr, nullptr, 0, 0.0f,
                         ws, ws_bytes, stream);
}

pe_status pe_mlp_train_step(float* params, float* m, float* v, int32_t step, float lr,
                            const float* feats, const int32_t* labels, int32_t B, float* loss,
                            void* ws, size_t ws_bytes, void* stream) {
  if (!m || !v || step < 1 || !(lr > 0.0f) || !std::isfinite(lr)) return PE_EINVAL;
  return mlp_grad_common(params, feats, labels, B, nullptr, loss, params, m, v, step, lr, ws,
                         ws_bytes, stream);
}

pe_status pe_quantize_e4m3(const void* x, int32_t x_dtype, void* q, int64_t n, float scale,
                           void* stream) {
  g_last_error.clear();
  if (n < 0 || (n > 0 && (!x || !q)) || (x_dtype != PE_F32 && x_dtype != PE_BF16)) return PE_EINVAL;
  if (!(scale > 0.0f) || !std::isfinite(scale)) return PE_EINVAL;
  if (n == 0) return PE_OK;
  hipError_t e = launch_quantize(x, x_dtype == PE_BF16, (uint8_t*)q, n, scale, (hipStream_t)stream);
  return e == hipSuccess ? PE_OK : hip_fail(e, "quantize launch");
}

int32_t pe_tile_count(void) { return 3; }

const char* pe_tile_name(int32_t tile_id) {
  switch (tile_id) {
    case 0: return "auto";
    case 1: return "bt64_bt128_mfma16";
    case 2: return "bt256_w2x4_mfma32";
  }
  return nullptr;
}

pe_status pe_tile_table_load(const char* path) {
  if (!path) return PE_EINVAL;
  FILE* f = fopen(path, "r");
  if (!f) return PE_EINVAL;
  std::map<std::string, int> tab;
  char line[256];
  while (fgets(line, sizeof line, f)) {
    if (line[0] == '#' || line[0] == '\n') continue;
    char cls[128];
    int id = 0;
    if (sscanf(line, "%127s %d", cls, &id) != 2 || id < 1 || id > 2) {
      fclose(f);
      return PE_EINVAL;
    }
    tab[cls] = id;
  }
  fclose(f);
  std::lock_guard<std::mutex> lk(g_tab_mu);
  g_tile_table.swap(tab);
  return PE_OK;
}

const char* pe_shape_class(int32_t compute, int64_t m, int64_t n) {
  thread_local std::string s;
  if (m <= 0 || n <= 0) return "";
  s = shape_class(compute == PE_COMPUTE_F32 ? kF32 : kBF16, std::min(m, n), std::max(m, n));
  return s.c_str();
}

const char* pe_status_string(pe_status st) {
  switch (st) {
    case PE_OK: return "ok";
    case PE_EINVAL: return "invalid argument";
    case PE_EUNSUPPORTED: return "unsupported in this build";
    case PE_ENOCONV: return "Remez exchange did not converge";
    case PE_EWORKSPACE: return "workspace missing, too small or not 256-byte aligned";
    case PE_EHIP: return "HIP runtime error";
  }
  return "unknown status";
}

const char* pe_last_error(void) { return g_last_error.c_str(); }

}  // extern "C"
