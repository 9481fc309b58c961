// The FP32 path on FP32 MFMA (v_mfma_f32_16x16x4_f32, 157 TFLOP/s nominal), for
// the calls below.
//
// Schedules whose polynomials grow on [0, 1].  The planes' scales come from bounds
// on |p| and |b y + c y^2| there; a spectrum that stays where they are small (a
// Gaussian 4096 x 4096 has nothing above 0.03) is then held far below its scale,
// and its low bits and in the end all of it are lost: three steps whose B is
// bounded by 38 and 1.2e7 were 3e-4 off at s = 1024, (20, -300, 900) and two
// Newton-Schulz steps gave NaN.  The line lies where the planes are still as
// close to 64 bits as FP32 MFMA (runtime.hip, planes_fit); schedules for [l, 1]
// stay below it (X 2, B 16).  All forms of a call: any output, Muon, learned choice,
// spectrum-aware init, fast iteration.
//
// Long schedules on matrices of some hundreds of rows and more with an FP32
// result.  The small-tile kernels' fp16 planes are two to three times as fast
// and closer to 64 bits at every size; but each further step multiplies what
// rounding leaves in the small singular directions, so that two FP32 summations
// in different orders end up to 4.6e-5 apart (s = 2048, T = 8).  Where that
// distance passes 2e-5 (T = 6: s = 1280 1.9e-5, 1536 2.1e-5; T = 8: s = 512
// 1.9e-5, 768 2.8e-5) FP32 results stay the ones that earlier versions of this
// library gave, and this file's summation order with them.
//
// 128 x 128 tiles, 4 waves in 2 x 2, each 64 x 64 as 4 x 4 fragments; operands
// staged through registers, 32 fp32 of k per LDS stage (144-byte rows: 128 plus
// a pad that spreads the banks), two double-buffered stages.  A lane reads its
// fragment as one 16-byte chunk: rows lane % 16, k chunk lane / 16.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pe_kernels.h"

namespace pe {

constexpr int kRowBytes = 144;
constexpr int kBK = 32;
constexpr int kOpB = 128 * kRowBytes;  // one operand, one stage

__device__ __forceinline__ void f32_mma(const char* sA, const char* sB, int wm, int wn, int lane, f32x4 (&acc)[4][4]) {
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    u32x4 fa[4], fb[4];
    const int koff = ks * 64 + (lane / 16) * 16;
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      fa[f] = *(const u32x4*)(sA + (wm * 64 + f * 16 + (lane % 16)) * kRowBytes + koff);
      fb[f] = *(const u32x4*)(sB + (wn * 64 + f * 16 + (lane % 16)) * kRowBytes + koff);
    }
#pragma unroll
    for (int fm = 0; fm < 4; ++fm)
#pragma unroll
      for (int fn = 0; fn < 4; ++fn) {
        const f32x4 a4 = __builtin_bit_cast(f32x4, fa[fm]), b4 = __builtin_bit_cast(f32x4, fb[fn]);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[fm][fn] = __builtin_amdgcn_mfma_f32_16x16x4f32(a4[e], b4[e], acc[fm][fn], 0, 0, 0);
      }
  }
}

// acc += P[rp0:+128, k0:k1] * Q[rq0:+128, k0:k1]^T, (k1 - k0) % kBK == 0.
__device__ __forceinline__ void f32_product(const float* __restrict__ P, const float* __restrict__ Q, int64_t ld, int rp0,
                                            int rq0, int k0, int k1, char* smem, f32x4 (&acc)[4][4]) {
  constexpr int VEC = 4, CPT = 4;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  // chunk c = tid + 256 j: row c / 8, 16-byte column c % 8
  const int crow = tid >> 3, ccol = tid & 7;
  const PE_GLOBAL float* pP = gview(P) + (size_t)(rp0 + crow) * ld + k0 + ccol * VEC;
  const PE_GLOBAL float* pQ = gview(Q) + (size_t)(rq0 + crow) * ld + k0 + ccol * VEC;
  const size_t jstride = (size_t)32 * ld;  // 32 rows between a thread's chunks
  u32x4 ra[CPT], rb[CPT];
  const int nk = (k1 - k0) / kBK;
#pragma unroll
  for (int j = 0; j < CPT; ++j) {
    ra[j] = *(const PE_GLOBAL u32x4*)(pP + j * jstride);
    rb[j] = *(const PE_GLOBAL u32x4*)(pQ + j * jstride);
  }
  const int soff = crow * kRowBytes + ccol * 16;
#pragma unroll
  for (int j = 0; j < CPT; ++j) {
    *(u32x4*)(smem + soff + j * 32 * kRowBytes) = ra[j];
    *(u32x4*)(smem + kOpB + soff + j * 32 * kRowBytes) = rb[j];
  }
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    // prefetch the next stage (the last iteration re-reads its own stage, which
    // keeps the loop free of branches around the register buffers)
    const size_t adv = (size_t)(kt + 1 < nk ? kt + 1 : kt) * kBK;
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
      ra[j] = *(const PE_GLOBAL u32x4*)(pP + adv + j * jstride);
      rb[j] = *(const PE_GLOBAL u32x4*)(pQ + adv + j * jstride);
    }
    // keep the prefetch at the top of the stage: a whole stage of MFMA work
    // then covers its latency
    __builtin_amdgcn_sched_barrier(0);
    const char* cur = smem + (kt & 1) * 2 * kOpB;
    f32_mma(cur, cur + kOpB, wm, wn, lane, acc);
    char* nxt = smem + ((kt + 1) & 1) * 2 * kOpB;
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
      *(u32x4*)(nxt + soff + j * 32 * kRowBytes) = ra[j];
      *(u32x4*)(nxt + kOpB + soff + j * 32 * kRowBytes) = rb[j];
    }
    __syncthreads();
  }
}

// accumulator element (fm, fn, r): row wm 64 + fm 16 + 4 (lane / 16) + r, column wn 64 + fn 16 + lane % 16
__device__ __forceinline__ int f32_row(int fm) { return ((int)threadIdx.x >> 7) * 64 + fm * 16 + 4 * ((threadIdx.x & 63) >> 4); }
__device__ __forceinline__ int f32_col(int fn) { return (((int)threadIdx.x >> 6) & 1) * 64 + fn * 16 + (threadIdx.x & 15); }

template <int KIND>
__device__ __forceinline__ void f32_epi_syrk(const KArgs& args, CDesc& d, int ti, int tj, const f32x4 (&acc)[4][4], float* red) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const size_t sp = d.sp;
  float alpha = 1.0f, beta = 0.0f, a, b = 0.0f, c = 0.0f;
  if (KIND == KIND_GRAM && args.t == 0) {
    const float sg = d.scal[kScScale];
    alpha = sg * sg;
  }
  const bool raw = KIND == KIND_A2 && args.raw_a2;  // learned path, step 1: A^2 and its moments
  if (KIND == KIND_A2 && !raw) {
    step_coef(args, d, &a, &b, &c);
    beta = shift_beta(d, b, c);
    if (ti == 0 && tj == 0 && threadIdx.x == 0) d.scal[kScBeta] = beta;
  }
  float* dst = KIND == KIND_GRAM ? d.Af : raw ? d.A2f : (float*)d.Bs;
  float trs = 0.0f, frs = 0.0f;
  float mom[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int fm = 0; fm < 4; ++fm) {
    float ar[4][4];
    if (KIND == KIND_A2) {
#pragma unroll
      for (int fn = 0; fn < 4; ++fn)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          ar[fn][r] = gview(d.Af)[(size_t)(ti * 128 + f32_row(fm) + r) * sp + tj * 128 + f32_col(fn)];
    }
#pragma unroll
    for (int fn = 0; fn < 4; ++fn) {
      const int i = ti * 128 + f32_row(fm), j = tj * 128 + f32_col(fn);
      float v[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float x = acc[fm][fn][r];
        if (KIND == KIND_GRAM) {
          v[r] = alpha * x;
          frs = __builtin_fmaf(v[r], v[r], frs);
        } else if (raw) {
          const float av = ar[fn][r];
          v[r] = x;
          if (ti == tj && i + r == j) mom[0] += av;
          mom[1] = __builtin_fmaf(av, av, mom[1]);
          mom[2] = __builtin_fmaf(av, x, mom[2]);
          mom[3] = __builtin_fmaf(x, x, mom[3]);
        } else {
          v[r] = __builtin_fmaf(c, x, b * ar[fn][r]);
          if (ti == tj && i + r == j && j < d.s) v[r] -= beta;
        }
        gview_w(dst)[(size_t)(i + r) * sp + j] = v[r];
      }
      // mirrored tile: row j, columns i..i+3
      if (ti != tj) *(PE_GLOBAL f32x4*)gview_w(dst + (size_t)j * sp + i) = (f32x4){v[0], v[1], v[2], v[3]};
    }
  }
  if (KIND == KIND_GRAM) {
    // the tile's partials of tr(A) and ||A||_F^2 (an off-diagonal tile also
    // stands for its mirror); the diagonal is read back once the tile is stored
    __syncthreads();
    if (ti == tj && threadIdx.x < 128) trs = gview(d.Af)[(size_t)(ti * 128 + threadIdx.x) * sp + tj * 128 + threadIdx.x];
    for (int off = 32; off > 0; off >>= 1) {
      trs += __shfl_xor(trs, off);
      frs += __shfl_xor(frs, off);
    }
    if (lane == 0) {
      red[2 * wave] = trs;
      red[2 * wave + 1] = frs;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      float t0 = 0.0f, t1 = 0.0f;
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        t0 += red[2 * w];
        t1 += red[2 * w + 1];
      }
      const int tile = tri_index(ti, tj, d.nbs);
      d.trp[2 * tile] = t0;
      d.trp[2 * tile + 1] = (ti == tj ? 1.0f : 2.0f) * t1;
    }
  }
  if (raw) {
    // (an off-diagonal tile also stands for its mirror: weight 2 except on tr A)
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      for (int off = 32; off > 0; off >>= 1) mom[k] += __shfl_xor(mom[k], off);
      if (lane == 0) red[k * 4 + wave] = mom[k];
    }
    __syncthreads();
    if (threadIdx.x < 4) {
      const float* q = red + threadIdx.x * 4;
      const float t = ((q[0] + q[1]) + q[2]) + q[3];
      d.mom[(size_t)tri_index(ti, tj, d.nbs) * 4 + threadIdx.x] = threadIdx.x == 0 || ti == tj ? t : 2.0f * t;
    }
  }
}

// X = alpha ((a + beta) X + acc): the master and the next X^T (the two X^T
// buffers Xb and Xb1 take turns), or the caller's output on the last step
template <bool LAST>
__device__ __forceinline__ void f32_epi_update(const KArgs& args, CDesc& d, int tm, int tn, bool past, const f32x4 (&acc)[4][4]) {
  const size_t Lp = d.Lp, sp = d.sp;
  float a, b, c;
  step_coef(args, d, &a, &b, &c);
  // (a matrix past its schedule copies X: a = 1)
  if (!args.fast && !past) a += d.scal[kScBeta];
  const float alpha = args.t == 0 ? d.scal[kScScale] : 1.0f, keep = 1.0f - args.mlr * args.mwd;
  float* XTn = (float*)((args.t & 1) ? d.Xb : d.Xb1);
#pragma unroll
  for (int fm = 0; fm < 4; ++fm) {
    float xr[4][4];
#pragma unroll
    for (int fn = 0; fn < 4; ++fn)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        xr[fn][r] = gview(d.Xf)[(size_t)(tm * 128 + f32_row(fm) + r) * Lp + tn * 128 + f32_col(fn)];
#pragma unroll
    for (int fn = 0; fn < 4; ++fn) {
      const int i = tm * 128 + f32_row(fm), n = tn * 128 + f32_col(fn);
      float v[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = alpha * (a * xr[fn][r] + acc[fm][fn][r]);
      if constexpr (!LAST) {
#pragma unroll
        for (int r = 0; r < 4; ++r) gview_w(d.Xf)[(size_t)(i + r) * Lp + n] = v[r];
        *(PE_GLOBAL f32x4*)gview_w(XTn + (size_t)n * sp + i) = (f32x4){v[0], v[1], v[2], v[3]};
      } else if (n < d.L) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (i + r < d.s) {
            const size_t row = d.trans ? n : i + r, col = d.trans ? i + r : n;
            if (d.Out) {
              const size_t o = row * d.ldo + col;
              if (d.out_bf16) gview_w((uint16_t*)d.Out)[o] = f2bf(v[r]);
              else gview_w((float*)d.Out)[o] = v[r];
            }
            if (d.W) {
              const size_t o = row * d.ldw + col;
              const float w = d.w_bf16 ? bf2f(gview((const uint16_t*)d.W)[o]) : gview((const float*)d.W)[o];
              const float x = __builtin_fmaf(-args.mlr, v[r], keep * w);
              if (d.w_bf16) gview_w((uint16_t*)d.W)[o] = f2bf(x);
              else gview_w((float*)d.W)[o] = x;
            }
          }
      }
    }
  }
}

template <int KIND>
__global__ __launch_bounds__(kThreads, 2) void f32_gemm_kernel(KArgs args) {
  __shared__ __attribute__((aligned(16))) char smem[4 * kOpB + 64];
  for (int slot = blockIdx.x; slot < args.total; slot += gridDim.x) {
    const int item = xcd_item(slot, args.total);
    const int pos = find_mat(args.offs, args.count, item);
    CDesc& d = const_desc(args, args.ord ? const_i32(args.ord, pos) : pos);
    if (skip_matrix(args, d)) continue;
    const bool past = past_schedule(args, d);
    if (past && KIND != KIND_UPD_LAST) continue;
    const int local = item - const_i32(args.offs, pos);
    f32x4 acc[4][4];
#pragma unroll
    for (int fm = 0; fm < 4; ++fm)
#pragma unroll
      for (int fn = 0; fn < 4; ++fn) acc[fm][fn] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    if constexpr (KIND == KIND_UPD || KIND == KIND_UPD_LAST) {
      int tm, tn;
      banded_decode(local, d.nb, d.nbL, &tm, &tn);
      const float* B = args.fast ? d.fb[args.fp_] : (const float*)d.Bs;
      if (!past) f32_product(B, (const float*)((args.t & 1) ? d.Xb1 : d.Xb), d.sp, tm * 128, tn * 128, 0, d.sp, smem, acc);
      f32_epi_update<KIND == KIND_UPD_LAST>(args, d, tm, tn, past, acc);
    } else {
      const int split = KIND == KIND_GRAM ? d.gram_split : d.a2_split;
      const int tile = local / split, ksp = local % split;
      int ti, tj;
      tri_decode_banded(tile, d.nbs, &ti, &tj);
      const float* Op = KIND == KIND_GRAM ? d.Xf : d.Af;
      const int K = KIND == KIND_GRAM ? d.Lp : d.sp;
      int k0, k1;
      split_range(K, split, ksp, kBK, &k0, &k1);
      // a degree-3 step (c = 0 in the fixed schedule) needs no A^2
      if (KIND == KIND_A2 && !args.sel_coef && args.c == 0.0f) k1 = k0;
      if (k1 > k0) f32_product(Op, Op, K, ti * 128, tj * 128, k0, k1, smem, acc);
      if (split == 1) {
        f32_epi_syrk<KIND>(args, d, ti, tj, acc, (float*)(smem + 4 * kOpB));
      } else {
        // partial tile: float4 q of thread t at ((tile split + ksp) 16 + q) 256 + t
        float* part = d.part + (size_t)(tile * split + ksp) * 16384;
#pragma unroll
        for (int q = 0; q < 16; ++q)
          *(PE_GLOBAL f32x4*)gview_w(part + (q * kThreads + threadIdx.x) * 4) = acc[q >> 2][q & 3];
      }
    }
    __syncthreads();  // the stages are free for the next tile
  }
}

template <int KIND>
__global__ __launch_bounds__(kThreads) void f32_reduce_kernel(KArgs args) {
  __shared__ float red[16];
  for (int item = blockIdx.x; item < args.total; item += gridDim.x) {
    const int mi = find_mat(args.offs, args.count, item);
    CDesc& d = const_desc(args, mi);
    if (skip_matrix(args, d) || past_schedule(args, d)) continue;
    const int tile = item - const_i32(args.offs, mi), split = KIND == KIND_GRAM ? d.gram_split : d.a2_split;
    int ti, tj;
    tri_decode_banded(tile, d.nbs, &ti, &tj);
    f32x4 acc[4][4];
    const float* part = d.part + (size_t)tile * split * 16384;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      f32x4 s = *(const PE_GLOBAL f32x4*)gview(part + (q * kThreads + threadIdx.x) * 4);
      for (int k = 1; k < split; ++k) s += *(const PE_GLOBAL f32x4*)gview(part + (size_t)k * 16384 + (q * kThreads + threadIdx.x) * 4);
      acc[q >> 2][q & 3] = s;
    }
    f32_epi_syrk<KIND>(args, d, ti, tj, acc, red);
    __syncthreads();
  }
}

// Products of the fast rectangular iteration (see small_fast_kernel), on FP32
// buffers: D alternates between two, R is no operand of the product that
// replaces it.
template <int KIND>
__global__ __launch_bounds__(kThreads, 2) void f32_fast_kernel(KArgs args) {
  __shared__ __attribute__((aligned(16))) char smem[4 * kOpB];
  for (int slot = blockIdx.x; slot < args.total; slot += gridDim.x) {
    const int item = xcd_item(slot, args.total);
    const int pos = find_mat(args.offs, args.count, item);
    CDesc& d = const_desc(args, pos);
    int ti, tj;
    tri_decode_banded(item - const_i32(args.offs, pos), d.nbs, &ti, &tj);
    f32x4 acc[4][4];
#pragma unroll
    for (int fm = 0; fm < 4; ++fm)
#pragma unroll
      for (int fn = 0; fn < 4; ++fn) acc[fm][fn] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    if constexpr (KIND == KIND_GRAM) f32_product(d.Xf, d.Xf, d.Lp, ti * 128, tj * 128, 0, d.Lp, smem, acc);
    else f32_product(d.fb[args.fp_], d.fb[args.fq_], d.sp, ti * 128, tj * 128, 0, d.sp, smem, acc);
    const size_t sp = d.sp;
    float ca = args.cacc;
    if (KIND == KIND_GRAM && args.t == 0) ca *= d.scal[kScScale] * d.scal[kScScale];
    const float *E1 = args.fe1 >= 0 ? d.fb[args.fe1] : nullptr, *E2 = args.fe2 >= 0 ? d.fb[args.fe2] : nullptr;
    float* out = d.fb[args.fout];
#pragma unroll
    for (int fm = 0; fm < 4; ++fm)
#pragma unroll
      for (int fn = 0; fn < 4; ++fn) {
        const int i = ti * 128 + f32_row(fm), j = tj * 128 + f32_col(fn);
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const size_t o = (size_t)(i + r) * sp + j;
          float x = ca * acc[fm][fn][r];
          if (E1) x = __builtin_fmaf(args.c1, gview(E1)[o], x);
          if (E2) x = __builtin_fmaf(args.c2, gview(E2)[o], x);
          if (i + r == j && j < d.s) x += args.cdiag;
          v[r] = x;
          gview_w(out)[o] = x;
        }
        if (ti != tj) *(PE_GLOBAL f32x4*)gview_w(out + (size_t)j * sp + i) = (f32x4){v[0], v[1], v[2], v[3]};
      }
    __syncthreads();  // the stages are free for the next tile
  }
}

hipError_t launch_f32_fast(int kind, const KArgs& a, hipStream_t st) {
  if (a.total <= 0) return hipSuccess;
  auto k = kind == KIND_GRAM ? f32_fast_kernel<KIND_GRAM> : f32_fast_kernel<KIND_A2>;
  hipLaunchKernelGGL(k, dim3(a.total < 512 ? a.total : 512), dim3(kThreads), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_f32_gemm(int kind, const KArgs& a, hipStream_t st) {
  if (a.total <= 0) return hipSuccess;
  auto k = kind == KIND_GRAM ? f32_gemm_kernel<KIND_GRAM> : kind == KIND_A2 ? f32_gemm_kernel<KIND_A2>
         : a.last            ? f32_gemm_kernel<KIND_UPD_LAST> : f32_gemm_kernel<KIND_UPD>;
  hipLaunchKernelGGL(k, dim3(a.total < 512 ? a.total : 512), dim3(kThreads), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_f32_reduce(int kind, const KArgs& a, hipStream_t st) {
  if (a.total <= 0) return hipSuccess;
  auto k = kind == KIND_GRAM ? f32_reduce_kernel<KIND_GRAM> : f32_reduce_kernel<KIND_A2>;
  hipLaunchKernelGGL(k, dim3(a.total < 1024 ? a.total : 1024), dim3(kThreads), 0, st, a);
  return hipGetLastError();
}

}  // namespace pe
