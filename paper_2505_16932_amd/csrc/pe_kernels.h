// Device helpers shared by the kernel files: conversions, descriptor access,
// waits and barriers, and the item orders of the persistent kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pe_device.h"

namespace pe {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short i16x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef short i16x4 __attribute__((ext_vector_type(4)));

// Streaming (non-temporal) stores and loads, for data that a launch touches
// once: outputs that only later launches read should not displace from the L2
// the operand panels that neighbouring tiles of the same launch re-read.
template <typename T>
__device__ __forceinline__ void st_stream(T* p, T v) { __builtin_nontemporal_store(v, p); }
__device__ __forceinline__ void st_stream(uint2* p, uint2 v) {
  __builtin_nontemporal_store((u32x2){v.x, v.y}, (u32x2*)p);
}
// streaming only where S holds; an ordinary store otherwise
template <bool S, typename T>
__device__ __forceinline__ void st_hint(T* p, T v) {
  if constexpr (S) st_stream(p, v);
  else *p = v;
}

// KIND_UPD0: the first update when X_0 is exactly its bf16 copy (MatDesc::x0b);
// KIND_UPDI: the spectrum-aware init step's on the bf16 paths (B in two parts)
enum Kind : int { KIND_GRAM = 0, KIND_A2 = 1, KIND_UPD = 2, KIND_UPD_LAST = 3, KIND_UPD0 = 4, KIND_UPDI = 5 };

// Descriptor pointers are generic; loads through these global-address-space
// views compile to global_load (not flat_load), which keeps vmcnt/lgkmcnt apart.
#define PE_GLOBAL __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ const PE_GLOBAL T* gview(const T* p) {
  return (const PE_GLOBAL T*)p;
}
template <typename T>
__device__ __forceinline__ PE_GLOBAL T* gview_w(T* p) {
  return (PE_GLOBAL T*)p;
}

// ---------------------------------------------------------------- helpers
__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);  // quiet NaN
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
// two floats as packed bf16, round to nearest even (v_cvt_pk_bf16_f32)
typedef float f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack2_bf16(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){lo, hi}, bf16x2));
}
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
// next plane of two floats: their fp16 values, which are taken out of them
__device__ __forceinline__ uint32_t peel2_f16(float* x, float* y) {
  const f16x2 h = __builtin_convertvector((f32x2){*x, *y}, f16x2);
  const f32x2 back = __builtin_convertvector(h, f32x2);
  *x -= back[0];
  *y -= back[1];
  return __builtin_bit_cast(uint32_t, h);
}
// The iterate of the bf16 paths in two 16-bit halves: hi the bf16 copy that the
// products read (nearest, halves away from zero), lo the low half of the FP32
// bit pattern read as a signed number, bits = (hi << 16) + lo.  Exact, in four
// bytes per element instead of an FP32 copy beside the bf16 one.
__device__ __forceinline__ void join2_f32(uint32_t hi, uint32_t lo, float* x, float* y) {
  *x = __int_as_float((int)(hi << 16) + (int)(int16_t)(lo & 0xffffu));
  *y = __int_as_float((int)(hi & 0xffff0000u) + ((int)lo >> 16));
}
__device__ __forceinline__ void split2_f32(float x, float y, uint32_t* hi, uint32_t* lo) {
  const uint32_t u = __float_as_uint(x), v = __float_as_uint(y);
  *hi = ((u + 0x8000u) >> 16) | ((v + 0x8000u) & 0xffff0000u);
  *lo = (u & 0xffffu) | (v << 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// Tables that no kernel of the call writes (descriptors, item offsets), read
// at indexes all lanes share: through the constant address space they load
// into scalar registers, a whole descriptor's fields in one or two round trips.
#define PE_CONST __attribute__((address_space(4)))
typedef const PE_CONST MatDesc CDesc;
__device__ __forceinline__ CDesc& const_desc(const KArgs& args, int mi) {
  return ((CDesc*)(uintptr_t)args.descs)[mi];
}
__device__ __forceinline__ int const_i32(const int32_t* p, int i) {
  return ((const PE_CONST int32_t*)(uintptr_t)p)[i];
}

__device__ __forceinline__ int find_mat(const int32_t* offs, int count, int item) {
  int lo = 0, hi = count - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (const_i32(offs, mid) <= item) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Scale of X_0 from ||G||_F (Appendix A.1 listing, or Algorithm 1)
__device__ __forceinline__ float norm_sigma(double fro, int mode) {
  return (float)(mode == 1 ? 1.0 / (fro + 1e-2) : 1.0 / (1.01 * fro + 1e-7));
}

// sum of a wave's values, the same bits in every lane
__device__ __forceinline__ double wave_sum(double x) {
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
  return x;
}

// ||X||_F^2 of the caller's matrix, from the norm pass's partial sums
__device__ __forceinline__ double matrix_square_sum(CDesc& d) {
  double acc = 0.0;
  for (int i = threadIdx.x & 63; i < d.n_prep; i += 64) acc += gview(d.red)[i];
  return wave_sum(acc);
}

// sigma of a matrix: from the finalize launch, or (small calls, which save that
// launch) from the partial sums, which every wave adds up alike
__device__ __forceinline__ float matrix_sigma(const KArgs& args, CDesc& d) {
  if (!args.fold_norm) return d.scal[kScScale];
  return norm_sigma(sqrt(matrix_square_sum(d)), args.norm_mode);
}

// In the fallback re-run only the matrices whose estimate failed are recomputed.
template <typename D>
__device__ __forceinline__ bool skip_matrix(const KArgs& args, D& d) {
  return args.fallback && (d.flagp == nullptr || *d.flagp == 0);
}

// Learned path: the matrix's class schedule has ended (step t >= its T'); its
// kernels skip it, and the last step only copies X to the caller's output.
template <typename D>
__device__ __forceinline__ int schedule_steps(const KArgs& args, D& d) {
  if (!args.sel_steps || !d.selp) return kMaxSteps + 1;
  int cls = *d.selp;
  if (cls < 0 || cls >= kClasses) cls = args.fixed_class;
  return args.sel_steps[cls];
}
template <typename D>
__device__ __forceinline__ bool past_schedule(const KArgs& args, D& d) { return args.t >= schedule_steps(args, d); }

// bf16 operand copies of the iterate (bf16 / e4m3 paths): step t reads X_t
// from one of the two buffers, in the Gram product and as the k-rows of B X,
// while its update writes X_{t+1} into the other (every tile of the update
// reads all of X_t, so it cannot be overwritten in place)
template <typename D>
__device__ __forceinline__ const uint16_t* xb_at(D& d, int t) { return (const uint16_t*)((t & 1) ? d.Xb1 : d.Xb); }
template <typename D>
__device__ __forceinline__ const uint16_t* xb_cur(const KArgs& args, D& d) { return xb_at(d, args.t); }
template <typename D>
__device__ __forceinline__ uint16_t* xb_next(const KArgs& args, D& d) {
  return (uint16_t*)((args.t & 1) ? d.Xb : d.Xb1);
}

template <typename D>
__device__ __forceinline__ void step_coef(const KArgs& args, D& d, float* a, float* b, float* c) {
  if (args.init_step) {
    // spectrum-aware init: the cubic chosen per matrix from its power bound
    *a = d.scal[kScInitA];
    *b = d.scal[kScInitB];
    *c = 0.0f;
  } else if (args.sel_coef) {
    // the class slot is written before any product that reads coefficients
    // (finalize: fixed class; select: the chosen one); an out-of-range value
    // still falls back to the fixed class instead of leaving the table
    int cls = *d.selp;
    if (cls < 0 || cls >= kClasses) cls = args.fixed_class;
    const float* p = args.sel_coef + ((size_t)cls * args.tmax + args.t) * 3;
    *a = p[0]; *b = p[1]; *c = p[2];
  } else {
    *a = args.a; *b = args.b; *c = args.c;
  }
}

// 16-byte chunk of a 128-byte stage row: XOR-ed by the row pair's number, which
// spreads the reads of one chunk of 32 rows over all banks
__device__ __forceinline__ int dl_swz(int row, int chunk) { return chunk ^ ((row >> 1) & 7); }

// s_waitcnt vmcnt(n) (gfx9 encoding: vmcnt[3:0] | vmcnt[5:4] << 14; exp/lgkm at max)
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// Workgroup barrier that orders LDS accesses for the compiler without the
// memory fences of __syncthreads (which would also wait for every
// outstanding global load): the empty asm statements with a memory clobber
// keep the compiler from moving loads or stores across the s_barrier; the
// hardware ordering comes from the explicit waits placed before it.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// s_waitcnt lgkmcnt(0) with vmcnt and expcnt left at their maxima
__device__ __forceinline__ void wait_lgkm0() { __builtin_amdgcn_s_waitcnt(0xC07F); }

// Persistent blocks take items b, b + G, b + 2G, ... (G = gridDim.x, a multiple
// of 8 or all of the items).  Blocks are dispatched round-robin over the 8 XCDs
// (block b on XCD b % 8), each with its own L2.  This permutation gives the
// blocks of an XCD neighbouring positions of the item order, so tiles that
// share operand panels run on the same L2: in a full round one contiguous
// range, in the last, partial one (sorted by length like the others, and the
// last to even out the work) runs of 16 dealt to the XCDs in turn.
__device__ __forceinline__ int xcd_item(int slot, int total) {
  const int G = gridDim.x, first = slot / G * G, b = slot - first, n = min(G, total - first);
  const int x = b & 7, i = b >> 3;
  const int runs = n == G ? 0 : n >> 7, r = n - 128 * runs;
  if (i < 16 * runs) return first + ((i >> 4) * 8 + x) * 16 + (i & 15);
  return first + 128 * runs + x * (r >> 3) + min(x, r & 7) + i - 16 * runs;
}

// Tile (tm, tn) of an nb x nbn grid from a position in "banded" order: bands of
// GM tile rows, tm fastest inside a band, so consecutive positions form
// GM-tall blocks that share both operand panels.
__device__ __forceinline__ void banded_decode(int local, int nb, int nbn, int* tm, int* tn) {
  constexpr int GM = 8;
  const int band = local / (GM * nbn);
  const int first = band * GM;
  const int rows = min(GM, nb - first);
  const int r = local - band * GM * nbn;
  *tm = first + r % rows;
  *tn = r / rows;
}

// upper-triangle tile index -> (ti, tj), ti <= tj, row-major over ti
__device__ __forceinline__ void tri_decode(int u, int nb, int* ti, int* tj) {
  int r = 0, rowlen = nb;
  while (u >= rowlen) { u -= rowlen; ++r; --rowlen; }
  *ti = r;
  *tj = r + u;
}

// Upper-triangle tile (ti <= tj) from a position in banded order: bands of
// GM tile rows; inside a band, columns left to right, the band's rows (those
// with ti <= tj) fastest.  Consecutive positions then share column panels and
// cycle through GM row panels, as in banded_decode, so the tiles that one XCD
// runs together touch few distinct operand panels.  A band of R rows starting
// at row r0 holds R(R+1)/2 tiles in its first R columns, then R per column.
__device__ __forceinline__ void tri_decode_banded(int u, int nb, int* ti, int* tj) {
  constexpr int GM = 8;
  int r0 = 0;
  for (;;) {
    const int R = min(GM, nb - r0);
    const int tri = R * (R + 1) / 2;
    const int cnt = tri + (nb - r0 - R) * R;
    if (u < cnt) {
      if (u < tri) {
        int c = 0;
        while ((c + 1) * (c + 2) / 2 <= u) ++c;
        *tj = r0 + c;
        *ti = r0 + (u - c * (c + 1) / 2);
      } else {
        const int v = u - tri;
        *tj = r0 + R + v / R;
        *ti = r0 + v % R;
      }
      return;
    }
    u -= cnt;
    r0 += R;
  }
}

// inverse of tri_decode (row-major index, used for per-tile partial sums)
__device__ __forceinline__ int tri_index(int ti, int tj, int nb) {
  return ti * nb - (ti * (ti - 1)) / 2 + (tj - ti);
}

__device__ __forceinline__ void split_range(int K, int split, int ksp, int BK, int* k0, int* k1) {
  int per = (K + split - 1) / split;
  per = (per + BK - 1) / BK * BK;
  *k0 = min(K, ksp * per);
  *k1 = min(K, *k0 + per);
}

// Wave-level max of non-negative floats, one atomic per wave.
__device__ __forceinline__ void wave_amax_atomic(float v, float* slot) {
  for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
  if ((threadIdx.x & 63) == 0) atomicMax((unsigned int*)slot, __float_as_uint(v));
}

__device__ __forceinline__ uint2 pack4_bf16(const float (&v)[4]) {
  uint2 pk;
  pk.x = (uint32_t)f2bf(v[0]) | ((uint32_t)f2bf(v[1]) << 16);
  pk.y = (uint32_t)f2bf(v[2]) | ((uint32_t)f2bf(v[3]) << 16);
  return pk;
}

}  // namespace pe
