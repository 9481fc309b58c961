// Device-side descriptors shared by the kernels and the host runtime.
//
// Layout in HBM (per matrix; all buffers 256-byte aligned, inside the caller's
// workspace).  The iterate is oriented as X = G (m <= n) or X = G^T (m > n),
// so X is s x L with s = min(m, n) <= L = max(m, n) and the Gram matrix is
// s x s (the smaller side).  s and L are padded with zeros to sp, Lp
// (multiples of the update's block tile, 64, 128 or 256).  Zero rows/columns stay exactly zero under
// X <- aX + (bA + cA^2)X, so every kernel runs on the padded shape with no
// bounds checks; only the input read and the final store see m, n.
//   Xf      sp x Lp  fp32   master iterate (row-major; fp32 paths)
//   Xl      sp x Lp  int16  bf16/fp8 paths: the iterate is FP32 in two halves,
//                           its bf16 copy and the low half of the bit pattern,
//                           X = bits (Xb << 16) + Xl
//   Xb, Xb1 sp x Lp  bf16   operand copies of X_t (bf16/fp8 paths), used in turn:
//                           step t reads Xb (t even) or Xb1 (t odd) in the Gram
//                           product and in B X, and its update writes the other
//                           (fp32 path: two fp16 planes each, see below)
//   Af      sp x sp  fp32   A = X X^T (fp32 path)
//   As      sp x sp  bf16   A in bf16 on the bf16/fp8 paths, read by A^2 and by
//                           the bA term of B (fp32 path: planes of A, in the
//                           one of Xb, Xb1 that the step's update will write)
//   Bs      sp x sp  bf16 (fp32 path: planes)   B - beta I, B = bA + cA^2 (beta: see shift_beta)
//                           (bf16 paths, spectrum-aware init step: in two bf16
//                           parts, the second one in As, which is free by then)
//   Xq, Aq  sp x Lp, sp x sp  e4m3  operand copies for the FP8 steps (256 tile)
//   part    split-K partial tiles of the Gram-side products
//   red     per-tile partial sums of squares (fp64) and maxima (fp32) of G
//   trp     per-tile partials of tr(A_t) and ||A_t||_F^2 (fp32), for the shift beta_t
//   scal    per-matrix scalars (scale, amax values), cnt: arrival counters
//
// Operands of the fp32 path.  The matrix cores multiply fp16 16 times faster
// than fp32, so an fp32 operand matrix V is held as two fp16 planes
//   hi = fp16(q V),  lo = fp16(q V - hi)      (hi first, lo one matrix further)
// with a power of two q, 22 significant bits, and a product is
//   V W = (hi hi' + hi lo' + lo hi') / (q q')
// with fp32 accumulation; the dropped lo lo' is 2^-22 of a term (the 64 tile
// keeps it).  Matrices of fewer than 16 rows, whose few terms average nothing
// out, take fp32 operands and fp64 sums on the vector units instead.  q puts a bound
// on the matrix's largest singular value (a scalar recursion on the host over
// the schedule) at 2^14, a quarter of the fp16 range, so no entry overflows and
// the smallest entries lose bits only 2^-38 below it.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pe {

constexpr int kTileTiny = 64;   // GEMM block tiles: 64 x 64, 128 x 128 or 256 x 256
constexpr int kTileSmall = 128;
constexpr int kTileLarge = 256;
constexpr int kPrepTile = 64;   // norm/prep tile
constexpr int kPrepGroup = 4;   // tiles per norm-pass item (one partial sum each); 1 in small calls
constexpr int kFoldPartials = 256;  // partial sums of a matrix that its readers may add up themselves
constexpr int kThreads = 256;   // threads per block (4 wave64)
constexpr int kMaxSteps = 64;

// kTiny: the fp32 path of matrices with fewer than 16 rows, without planes;
// kF32M: FP32 MFMA (f32.hip), X^T in Xb / Xb1, fp32 B and fb
enum Prec : int32_t { kF32 = 0, kBF16 = 1, kFP8 = 2, kTiny = 3, kF32M = 4 };

// scal[] slots
enum : int32_t {
  kScScale = 0,    // sigma = 1 / (1.01 ||G||_F + 1e-7)
  kScAmaxG = 1,    // max |G| (float bits)
  kScFro = 2,      // ||G||_F as float
  kScBeta = 3,     // shift beta_t = tr(B_t)/s of the current step (update: a + beta)
  kScInitA = 5,    // spectrum-aware init: coefficients (a, b) of the init cubic
  kScInitB = 6,
  kScInitQ = 7,    // fp32 path: plane scale of the init step's B
  kScAmaxX = 8,    // +t : max |X_t| (uint bits of a non-negative float), t = 0..63
  kScAmaxA = 72,   // +t : max |A_t| for step t (0-based)
  kScN = 136
};

struct MatDesc {
  const void* G;
  void* Out;
  int64_t ldg, ldo;
  int32_t m, n, s, L;
  int32_t sp, Lp, trans, g_bf16;
  int32_t out_bf16, nb, nbL, sel;
  float* Xf;
  uint16_t* Xl;
  void* Xb;
  void* Xb1;
  float* Af;
  void* As;
  void* Bs;
  float* part;
  double* red;      // [n_prep] doubles then [n_prep] floats
  float* scal;      // [kScN]
  uint32_t* cnt;    // [4]
  float* trp;       // [syrk_nt][2] per-tile partials of tr(A) and ||A||_F^2 (Gram epilogue)
  int32_t n_prep, syrk_nt, upd_nt, gram_split;
  int32_t a2_split, nbs, g_vec, o_vec;  // nbs: tiles per side of the symmetric products;
                                        // g_vec / o_vec: 16-byte loads of G / stores of the bf16 output
  // learned l-predictor (null unless the call selects schedules per matrix)
  int32_t* selp;    // schedule class of this matrix
  int32_t* flagp;   // 1: the fallback re-run recomputes this matrix
  float* A2f;       // sp x sp fp32: A^2 of step 1, before the class is known
  float* mom;       // [syrk_nt][4] per-tile partial moments tr(A^k), k = 1..4
  float* feat;      // [16] features (diagnostic copy)
  float* est;       // [2]: estimate of ||X X^T - I||_2, flag
  float* vec;       // power iteration vectors: v [sp], y [sp], w [Lp]
  // FP8 steps on the 256 tile: e4m3 copies of the Gram-side operands
  uint8_t* Xq;      // sp x Lp: e4m3(q X_t), written by the quantisation pass
  uint8_t* Aq;      // sp x sp: e4m3(q A_t)
  // fast rectangular iteration (FP32): sp x sp buffers, see kFb* below
  float* fb[5];      // fp32 values
  uint16_t* fbp[5];  // operand planes (kFbP: none, the dead copy of X holds them)
  // Muon step (caller's m x n layout): momentum M (FP32) updated by the norm
  // pass, weights W updated by the last step's epilogue
  float* M;
  void* W;
  int64_t ldm, ldw;
  int32_t w_bf16;
  // 1: X_0 is exactly its bf16 copy (bf16 input, bf16/FP8 compute, no Muon
  // momentum): the norm pass stores no low half and the first update reads Xb alone
  int32_t x0b;
};

// Roles of MatDesc::fb in the fast rectangular iteration: the segment's R_t
// (ping-pong), D_t = Q_t - (prod a) I (ping-pong), P = R_t B_t, and B_t.
enum : int32_t { kFbR = 0, kFbD0 = 1, kFbD1 = 2, kFbB = 3, kFbP = 4, kFbNone = -1 };

struct KArgs {
  const MatDesc* descs;  // device array of `count` descriptors
  const int32_t* offs;   // per-matrix prefix offsets of this phase's items, count+1
  int32_t count;
  int32_t total;         // items in this launch
  int32_t t;             // 0-based step
  int32_t last;          // 1 on the final step
  int32_t fp8;           // this step's Gram-side products take e4m3 operands
  int32_t fp8_next;      // the next step's Gram product takes e4m3 operands
  int32_t norm_mode;
  int32_t tmax;          // rows of the selectable coefficient table
  int32_t prep_group;    // 64 x 64 tiles per norm-pass item
  int32_t fold_norm;     // no finalize launch: readers of sigma add up the partial sums
  int32_t alike;         // split_k = 1: nothing that orders sums depends on the launch's size
  float a, b, c;         // coefficients of step t (fixed schedule)
  const float* sel_coef; // [n_sched][tmax][3] or nullptr: per-matrix class schedules
  int32_t raw_a2;        // step-1 A^2 of the learned path: store A^2 and its moments
  int32_t fallback;      // fallback re-run: skip matrices whose flag is 0
  const float* mlp;      // predictor parameters (device) for the selection kernel
  int32_t force_class;   // >= 0: use this class instead of the network's choice
  int32_t fixed_class;
  float tau;             // fallback threshold
  int32_t est_phase;     // phase of the estimate's power iteration; step of the init's
  const int32_t* ord;    // position -> matrix of this phase's item order (nullptr: identity)
  // fast rectangular iteration (small_fast_kernel and the update): operand and
  // epilogue buffers (MatDesc::fb roles) and coefficients of
  //   out = cacc * acc + c1 * E1 + c2 * E2 + cdiag * I
  int32_t fast;          // 1: a launch of the fast iteration
  int32_t fp_, fq_, fe1, fe2, fout;
  float cacc, c1, c2, cdiag;
  int32_t tail;          // first tile of a launch that runs the last tiles as quarters (-1: none)
  float mbeta, mlr, mwd; // Muon momentum coefficient, learning rate, weight decay
  int32_t init_step;     // the spectrum-aware init step: (a, b, 0) from scal[kScInitA/B]
  const int32_t* sel_steps;  // [n_sched]: steps T' of each class's schedule (learned path)
  int32_t x0b;           // first update: every matrix of the call reads X_0 from its bf16 copy
  // fp32 path: 1 / (scales of the launch's two operands), scale of the planes it writes
  float deq, oscale;
};

// Schedule of the resident kernel, which runs all steps of a call.
struct ResSchedule {
  int32_t T;
  float abc[3 * kMaxSteps];
};

// Spectral shift of the update.  In real arithmetic
//   X_{t+1} = a X + B X = (a + beta) X + (B - beta I) X
// for any beta.  The product takes bf16 copies of its operands, whose rounding
// errors enter as (B - beta I) dX and dB X; beta = tr(B) / s, the mean
// eigenvalue of B, minimises ||B - beta I||_F and with it the error carried
// by isotropic rounding noise (on inputs whose singular values sit close
// together, B is close to a multiple of I and the unshifted product rounds away
// most of the update).  tr(B) = b tr(A) + c ||A||_F^2 for symmetric A; the Gram
// epilogue leaves per-tile partials of both, and every caller reduces them in
// the same fixed order, so all blocks agree on beta bit for bit.
template <typename D>
__device__ __forceinline__ float shift_beta(D& d, float b, float c) {
  const int lane = threadIdx.x & 63;
  float tr = 0.0f, fr = 0.0f;
  for (int u = lane; u < d.syrk_nt; u += 64) {
    tr += d.trp[2 * u];
    fr += d.trp[2 * u + 1];
  }
  // butterfly sums: every lane ends with the same bits (addition commutes exactly)
  for (int off = 32; off > 0; off >>= 1) {
    tr += __shfl_xor(tr, off);
    fr += __shfl_xor(fr, off);
  }
  return d.s > 0 ? (b * tr + c * fr) / (float)d.s : 0.0f;
}

constexpr int kClasses = 8;
constexpr int kFeat = 16;
constexpr int kMlpH = 64;
constexpr int kMlpParams = kFeat * kMlpH + kMlpH + kMlpH * kMlpH + kMlpH + kMlpH * kClasses + kClasses;

// Device memory is filled from kernel arguments (copied at launch), so the
// host needs neither pinned staging nor a synchronisation to upload tables.
constexpr int kPutWords = 960;
struct PutChunk {
  uint32_t* dst;
  int32_t nwords;
  int32_t pad;
  uint32_t w[kPutWords];
};

}  // namespace pe
