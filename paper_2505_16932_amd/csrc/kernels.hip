// gfx950 kernels of the Polar Express online stage (Section 3.5 and the
// Appendix A.1 listing: X_0 = G / (1.01 ||G||_F + 1e-7); per step
// A = X X^T, B = b A + c A^2, X = a X + B X).
//
// The norm pass, the bf16 and e4m3 products on the 256 tile, the e4m3 products
// of small matrices, the power method and the init step's B; the 64 and 128 tiles
// are in tiles.hip, FP32 MFMA in f32.hip, matrices of at most 64 rows in resident.hip.  Each kernel
// is launched once per phase over the items of every matrix of a call ("grouped"
// launches; a single matrix is a group of one) and walks its items in a
// grid-stride loop:
//   prep_kernel   one HBM pass over G: orientation, sum of squares (FP32 per
//                 lane and item, FP64 fixed-order sum of the items' partials
//                 => deterministic), max |G|, and the unscaled copies of X_0
//                 (bf16 paths: the bf16 copy, plus the low halves unless the
//                 bf16 copy is exact; FP32 paths: X_0); the scale sigma is folded
//                 into step 1's epilogues (A_1 = sigma^2 G G^T, X_1 = sigma (a G
//                 + B_1 G)).
//   gemm_kernel   persistent blocks over block tiles of 256 (8 waves in 2 x 4,
//                 32x32x16 MFMA, one block per CU), or of 128 for the e4m3
//                 Gram-side products of small matrices; bf16 operands go from
//                 HBM straight into a two-stage LDS ring, FP32 accumulation.
//                 KIND_GRAM:  A = X X^T, upper-triangle tiles only, mirrored
//                             store (SYRK);
//                 KIND_A2:    B = b A + c A A^T (A symmetric, so A^2 = A A^T is
//                             again a SYRK), epilogue re-reads A;
//                 KIND_UPD:   X = a X + B X; reads X_t itself (k along its rows)
//                             with transposing LDS reads; the epilogue reads and
//                             writes X in two 16-bit halves (the high one is the
//                             next step's operand), or writes the caller's output
//                             on the last step (KIND_UPD_LAST); KIND_UPD0 is the
//                             first update reading X_0 from its exact bf16 copy.
//                 In the e4m3 steps the Gram-side products read e4m3 copies
//                 (quant_kernel) on the 256 tile, or convert bf16 operands
//                 while staging them on the 128 tile.
//                 Split-K for the Gram-side products writes partial tiles;
//                 splitk_reduce_kernel sums them in split order (deterministic)
//                 and runs the same epilogue.
// The Gram-side GEMMs are "NT": C[i][j] = sum_k P[i][k] Q[j][k] with both
// operands row-major along k, which is what the MFMA lane layout wants; the
// update's second operand is row-major along n and is transposed by the LDS
// reads.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "pe_kernels.h"

namespace pe {
// ------------------------------------------------------------------ prep
// One 64 x 64 tile of the oriented, padded X per iteration of the block loop.
// Thread t owns two 8-element row chunks of the source block (rows t/8 and
// t/8 + 32, columns 8*(t%8)..+8) and, after an LDS transpose, the matching
// chunks of the transposed block.  Each tile writes its own partial sum of
// squares (FP64) and max |G|; finalize_kernel reduces them in fixed order.
__device__ __forceinline__ void load8(CDesc& d, int gr, int gc, int srn, int scn, float (&v)[8]) {
  if (gr < srn && d.g_vec && gc + 8 <= scn) {
    const size_t off = (size_t)gr * d.ldg + gc;
    if (d.g_bf16) {
      const u32x4 c = *(const PE_GLOBAL u32x4*)(gview((const uint16_t*)d.G) + off);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[2 * e] = __uint_as_float(c[e] << 16);
        v[2 * e + 1] = __uint_as_float(c[e] & 0xffff0000u);
      }
    } else {
      const PE_GLOBAL f32x4* q = (const PE_GLOBAL f32x4*)(gview((const float*)d.G) + off);
      const f32x4 c0 = q[0], c1 = q[1];
#pragma unroll
      for (int e = 0; e < 4; ++e) { v[e] = c0[e]; v[4 + e] = c1[e]; }
    }
    return;
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    float x = 0.0f;
    if (gr < srn && gc + e < scn) {
      const size_t off = (size_t)gr * d.ldg + gc + e;
      x = d.g_bf16 ? bf2f(((const uint16_t*)d.G)[off]) : ((const float*)d.G)[off];
    }
    v[e] = x;
  }
}

template <int P>
__device__ __forceinline__ void store8_f32(float* dst, const float (&v)[8]) {
  st_stream((f32x4*)dst, f32x4{v[0], v[1], v[2], v[3]});
  st_stream((f32x4*)(dst + 4), f32x4{v[4], v[5], v[6], v[7]});
}
// row-major X row chunk: the bf16 paths' two halves (the low one unless the
// bf16 copy, in the first of the two buffers, holds X_0 exactly), or FP32
template <int P>
__device__ __forceinline__ void store_x_chunk(CDesc& d, size_t o, const float (&v)[8]) {
  if constexpr (P == kBF16) {
    u32x4 hi, lo;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      uint32_t a, b;
      split2_f32(v[2 * e], v[2 * e + 1], &a, &b);
      hi[e] = a;
      lo[e] = b;
    }
    st_stream((u32x4*)((uint16_t*)d.Xb + o), hi);
    if (!d.x0b) st_stream((u32x4*)(d.Xl + o), lo);
  } else {
    store8_f32<P>(d.Xf + o, v);
  }
}
// X^T chunk, FP32 MFMA's operand of B X: row n, columns i..i+7
__device__ __forceinline__ void store_xt_chunk(CDesc& d, int n, int i, const float (&v)[8]) {
  store8_f32<kF32M>((float*)d.Xb + (size_t)n * d.sp + i, v);
}
template <int P>
__global__ __launch_bounds__(kThreads) void prep_kernel(KArgs args) {
  __shared__ float tile[kPrepTile][kPrepTile + 1];
  __shared__ float red_s[kThreads / 64];
  __shared__ float red_f[kThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int rr = tid >> 3, cc = (tid & 7) * 8;
  // one item = prep_group consecutive 64 x 64 tiles (row-major tile order);
  // the partial sums of an item are reduced once, in a fixed order
  for (int item = blockIdx.x; item < args.total; item += gridDim.x) {
    const int mi = find_mat(args.offs, args.count, item);
    CDesc& d = const_desc(args, mi);
    if (skip_matrix(args, d)) continue;
    const int local = item - const_i32(args.offs, mi);
    const int ntk = d.Lp / kPrepTile, ntiles = ntk * (d.sp / kPrepTile);
    const int srn = d.trans ? d.L : d.s, scn = d.trans ? d.s : d.L;
    // sum of squares in FP32 per lane and within the item; the items' partials
    // are summed across the matrix in FP64 (finalize_kernel, or each reader)
    float ss = 0.0f;
    float amax = 0.0f;
#pragma unroll 1
    for (int u = 0; u < args.prep_group; ++u) {
      const int tix = local * args.prep_group + u;
      if (tix >= ntiles) break;
      const int i0 = (tix / ntk) * kPrepTile;   // rows of X (s side)
      const int k0 = (tix % ntk) * kPrepTile;   // cols of X (L side)
      // source block in G's own layout
      const int sr0 = d.trans ? k0 : i0, sc0 = d.trans ? i0 : k0;
      float v[2][8];
#pragma unroll
      for (int j = 0; j < 2; ++j) load8(d, sr0 + rr + 32 * j, sc0 + cc, srn, scn, v[j]);
      if (d.M) {
        // Muon momentum (Section 1.1): M <- beta M + (1 - beta) G in place, and
        // the iteration runs on the new M (padding stays zero).  The thread's
        // 16 values are all loaded before any is stored (16-byte accesses when
        // the row chunk is inside the matrix and aligned).
        const bool mvec = ((uintptr_t)d.M % 16 == 0) && (d.ldm % 4 == 0);
        float mo[2][8];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int gr = sr0 + rr + 32 * j;
          const PE_GLOBAL float* mrow = gview(d.M) + (size_t)gr * d.ldm + sc0 + cc;
          if (gr < srn && mvec && sc0 + cc + 8 <= scn) {
            const f32x4 lo = *(const PE_GLOBAL f32x4*)mrow, hi = *(const PE_GLOBAL f32x4*)(mrow + 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              mo[j][e] = lo[e];
              mo[j][e + 4] = hi[e];
            }
          } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) mo[j][e] = (gr < srn && sc0 + cc + e < scn) ? mrow[e] : 0.0f;
          }
        }
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int gr = sr0 + rr + 32 * j;
          PE_GLOBAL float* mrow = gview_w(d.M) + (size_t)gr * d.ldm + sc0 + cc;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            mo[j][e] = __builtin_fmaf(args.mbeta, mo[j][e], (1.0f - args.mbeta) * v[j][e]);
            if (gr < srn && sc0 + cc + e < scn) v[j][e] = mo[j][e];
          }
          if (gr < srn && mvec && sc0 + cc + 8 <= scn) {
            *(PE_GLOBAL f32x4*)mrow = (f32x4){mo[j][0], mo[j][1], mo[j][2], mo[j][3]};
            *(PE_GLOBAL f32x4*)(mrow + 4) = (f32x4){mo[j][4], mo[j][5], mo[j][6], mo[j][7]};
          } else {
#pragma unroll
            for (int e = 0; e < 8; ++e)
              if (gr < srn && sc0 + cc + e < scn) mrow[e] = mo[j][e];
          }
        }
      }
      // a transposed copy of the block goes through LDS: X itself when G is
      // tall, X^T for FP32 MFMA
      const bool transpose = P == kF32M || d.trans;
      if (transpose && u > 0) __syncthreads();  // the previous tile's transposed reads are done
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int r = rr + 32 * j;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          if (transpose) tile[r][cc + e] = v[j][e];
          ss = __builtin_fmaf(v[j][e], v[j][e], ss);
          amax = fmaxf(amax, fabsf(v[j][e]));
        }
        if (!d.trans) store_x_chunk<P>(d, (size_t)(i0 + r) * d.Lp + k0 + cc, v[j]);
        else if (P == kF32M) store_xt_chunk(d, k0 + r, i0 + cc, v[j]);
      }
      if (transpose) {
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          const int q = rr + 32 * j;
          float w[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) w[e] = tile[cc + e][q];
          if (!d.trans) store_xt_chunk(d, k0 + q, i0 + cc, w);
          else store_x_chunk<P>(d, (size_t)(i0 + q) * d.Lp + k0 + cc, w);
        }
      }
    }
    for (int off = 32; off > 0; off >>= 1) {
      ss += __shfl_xor(ss, off);
      amax = fmaxf(amax, __shfl_xor(amax, off));
    }
    if (lane == 0) { red_s[wave] = ss; red_f[wave] = amax; }
    __syncthreads();
    if (tid == 0) {
      d.red[local] = (double)((red_s[0] + red_s[1]) + (red_s[2] + red_s[3]));
      ((float*)(d.red + d.n_prep))[local] = fmaxf(fmaxf(red_f[0], red_f[1]), fmaxf(red_f[2], red_f[3]));
    }
    __syncthreads();  // the next item's first tile reuses the LDS tile and the reduction slots
  }
}

// One block per matrix: fixed-order reduction of the tile partials (the same
// result for any launch geometry), then sigma = 1 / (1.01 ||G||_F + 1e-7)
// (or 1 / (||G||_F + 1e-2)); clears the amax slots the FP8 steps accumulate into.
__global__ __launch_bounds__(kThreads) void finalize_kernel(KArgs args) {
  __shared__ double red_d[kThreads / 64];
  __shared__ float red_f[kThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int mi = blockIdx.x; mi < args.count; mi += gridDim.x) {
    CDesc& d = const_desc(args, mi);
    if (d.n_prep == 0 || skip_matrix(args, d)) continue;
    double acc = 0.0;
    float am = 0.0f;
    const float* rf = (const float*)(d.red + d.n_prep);
    for (int i = tid; i < d.n_prep; i += kThreads) {
      acc += d.red[i];
      am = fmaxf(am, rf[i]);
    }
    for (int off = 32; off > 0; off >>= 1) {
      acc += __shfl_xor(acc, off);
      am = fmaxf(am, __shfl_xor(am, off));
    }
    __syncthreads();
    if (lane == 0) { red_d[wave] = acc; red_f[wave] = am; }
    __syncthreads();
    if (tid == 0) {
      const double tot = (red_d[0] + red_d[1]) + (red_d[2] + red_d[3]);
      const double fro = sqrt(tot);
      d.scal[kScScale] = norm_sigma(fro, args.norm_mode);
      d.scal[kScAmaxG] = fmaxf(fmaxf(red_f[0], red_f[1]), fmaxf(red_f[2], red_f[3]));
      d.scal[kScFro] = (float)fro;
    }
    for (int i = kScAmaxX + tid; i < kScN; i += kThreads) d.scal[i] = 0.0f;
    // learned path, first pass: the class slot holds the fixed class until the
    // selection kernel overwrites it, and no matrix is marked for the re-run
    if (d.selp && !args.fallback && tid == 0) {
      *d.selp = args.fixed_class;
      *d.flagp = 0;
    }
  }
}

// ------------------------------------------------------------- GEMM core
// Block tile BT x BT of MFMA fragments F x F, F = BT/8: BT = 256 (bf16 and
// e4m3; 32 x 32 fragments) and BT = 128 (the e4m3 steps' Gram-side products of
// small matrices; 16 x 16).  The wave grid is WaveCfg below.
template <int BT>
struct TileCfg {
  static constexpr int F = BT / 8;                   // fragment edge
  static constexpr int ACC = F == 16 ? 4 : 16;       // accumulator floats per fragment
  static constexpr int RG = F == 16 ? 1 : 4;         // groups of 4 consecutive rows per fragment
};

template <int N>
struct AccT;
template <>
struct AccT<4> { typedef f32x4 type; };
template <>
struct AccT<16> { typedef float type __attribute__((ext_vector_type(16))); };

// Waves of a GEMM block and their grid over the BT x BT tile: two wave rows
// of BT/2 tile rows each; WGN wave columns of WTN tile columns, each holding
// FN fragments of F x F.  The bf16 256 tile runs 8 waves (2 per SIMD, wave
// tile 128 x 64): one wave's LDS reads, barrier waits and epilogue memory
// latency then overlap the other's MFMAs.  The FP8 256 tile uses the same
// layout; the e4m3 128 tile runs 4 waves.
template <int P, int BT>
struct WaveCfg {
  static constexpr int NW = ((P == kBF16 || P == kFP8) && BT == 256) ? 8 : 4;
  static constexpr int NT = NW * 64;
  static constexpr int WGN = NW / 2;
  static constexpr int F = BT / 8;
  static constexpr int FN = 8 / WGN;
  static constexpr int WTN = FN * F;
};

// ------------------------------------------------- bf16 direct-to-LDS main loop
// The bf16 path's main loop.  Operands go from HBM straight into LDS with
// global_load_lds_dwordx4 (lane i of a wave writes 16 bytes at LDS base + 16 i),
// so no registers stage them and no wait on a load sits in front of an LDS
// store.  Stages hold 64 k, 128 bytes per row, in a ring of two: with rows of 64
// bytes such a load covers sixteen half cache lines and runs at half the rate
// (33 against 55 bytes per clock and CU from L2), about as long as the MFMAs of
// the stage take (eight layers of 4096-wide matrices: Gram product 7.5 -> 6.9 ms,
// A^2 4.0 -> 3.75, update 14.9 -> 14.7; e4m3 Gram product of one layer 586 -> 554
// us).  A row's eight 16-byte chunks are stored XOR-swizzled by (row / 2) % 8,
// which spreads the fragment reads of consecutive rows over all banks.
template <int BT>
struct DlCfg {
  static constexpr int BK = 64;                  // k per stage
  static constexpr int NS = 2;                   // stages in the LDS ring
  static constexpr int ROWB = 128;               // bytes per row per stage
  static constexpr int OPB = BT * ROWB;          // one operand, one stage
  static constexpr int STB = 2 * OPB;            // one stage
  static constexpr int LDS = NS * STB;
  static constexpr int NW = WaveCfg<kBF16, BT>::NW;
  static constexpr int IPW = OPB / 1024 / NW;    // 1-KB loads per wave per operand per stage
  static constexpr int LPS = 2 * IPW;            // load instructions per wave per stage
};

// The update's second operand can also be X itself, row-major with k along
// its rows (XR): a stage then holds 32 rows of X (k) by BT columns (n), and
// the fragments are read with transposing LDS reads.  16-byte chunk c of
// stage row r sits at chunk c ^ xr_swz(r): each transposing read covers four
// consecutive rows per 16 lanes, and the swizzle puts them on distinct banks.
template <int BT>
__device__ __forceinline__ int xr_swz(int r) {
  static_assert(BT == 256, "the smaller tiles have their own");
  return (r & 3) << 2;
}

// P and Q are row-major along k (row strides ld, ldQ); XR: Q is row-major X, k
// along its rows, already offset to the tile's first column.
template <int BT, bool XR = false>
__device__ __forceinline__ void dl_issue_stage(const PE_GLOBAL uint16_t* P, const PE_GLOBAL uint16_t* Q,
                                               int64_t ld, int64_t ldQ, int kofs, char* slot, int wave, int lane) {
  typedef DlCfg<BT> C;
  if constexpr (XR) {
    constexpr int CPR = BT / 8;                      // 16-byte chunks per stage row
#pragma unroll
    for (int j = 0; j < C::IPW; ++j) {
      const int blk = j * C::NW + wave;             // 1-KB block = 64 / CPR rows
      const int row = blk * (64 / CPR);
      // the row's swizzle is the same for every j: one lane offset for all
      const int lc = (lane % CPR) ^ xr_swz<BT>(wave * (64 / CPR) + lane / CPR);  // logical chunk this lane fetches
      const PE_GLOBAL char* g = (const PE_GLOBAL char*)(Q + (size_t)(kofs + row) * ldQ) +
                                (uint32_t)((lane / CPR) * (int)ldQ * 2 + lc * 16);
      __builtin_amdgcn_global_load_lds((const void*)g,
                                       (__attribute__((address_space(3))) void*)(slot + C::OPB + blk * 1024),
                                       16, 0, 0);
    }
  }
#pragma unroll
  for (int op = 0; op < (XR ? 1 : 2); ++op) {
    const PE_GLOBAL uint16_t* base = op == 0 ? P : Q;
    const int64_t rs = op == 0 ? ld : ldQ;
#pragma unroll
    for (int j = 0; j < C::IPW; ++j) {
      const int blk = j * C::NW + wave;             // 1-KB block = 8 rows
      const int lc = dl_swz(wave * 8 + (lane >> 3), lane & 7);  // logical chunk this lane fetches
      const PE_GLOBAL char* g = (const PE_GLOBAL char*)(base + (size_t)(blk * 8) * rs + kofs) +
                                (uint32_t)((lane >> 3) * (int)rs * 2 + lc * 16);
      __builtin_amdgcn_global_load_lds((const void*)g,
                                       (__attribute__((address_space(3))) void*)(slot + op * C::OPB + blk * 1024),
                                       16, 0, 0);
    }
  }
}

// Transposing read of an XR stage (rows k, BT columns n): with every 16
// lanes addressing rows r0..r0+3 (lane q: row r0 + q / 4, columns n0 + 4 (q % 4)
// .. + 3), lane q receives the four k values of column n0 + q.
template <int BT>
__device__ __forceinline__ u32x2 xr_read(const char* sB, int r, int nn) {
  const char* p = sB + r * (BT * 2) + (((nn >> 3) ^ xr_swz<BT>(r)) << 4) + (nn & 4) * 2;
  return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                       (__attribute__((address_space(3))) i16x4*)(p)));
}

// Fragments of one 16-deep k-step of the 256 tile (32x32x16 MFMA, 8 waves):
// rows lane % 32 of four 32-row fragments of the first operand and two of the
// second, 16-byte chunk 2 * sub + lane / 32 of the stage's 128-byte row.
struct Frags32 {
  u32x4 a[4], b[2];
};

template <bool XR = false>
__device__ __forceinline__ void dl_read_frags32(const char* stage, int sub, int wm, int wn, int lane,
                                                Frags32& f) {
  constexpr int OPB = DlCfg<256>::OPB;
  const int lc = 2 * sub + (lane >> 5);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int ra = wm * 128 + i * 32 + (lane & 31);
    f.a[i] = *(const u32x4*)(stage + ra * 128 + dl_swz(ra, lc) * 16);
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    if constexpr (XR) {
      // 32x32x16: lane l takes k = 16 sub + 8 (l / 32) .. + 7 of column l % 32
      // of the fragment, whose columns are 32 wn + 128 i .. (upd_col)
      const int r = 16 * sub + 8 * (lane >> 5) + ((lane & 15) >> 2);
      const int nn = wn * 32 + i * 128 + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
      const u32x2 lo = xr_read<256>(stage + OPB, r, nn), hi = xr_read<256>(stage + OPB, r + 4, nn);
      f.b[i] = (u32x4){lo[0], lo[1], hi[0], hi[1]};
    } else {
      const int rb = wn * 64 + i * 32 + (lane & 31);
      f.b[i] = *(const u32x4*)(stage + OPB + rb * 128 + dl_swz(rb, lc) * 16);
    }
  }
}

// SWAP: operands exchanged, so that a lane holds consecutive columns of one row
// (of the update tile) instead of consecutive rows of one column
template <bool SWAP, typename A>
__device__ __forceinline__ void dl_mfma32(const Frags32& f, A (&acc)[4][2]) {
#pragma unroll
  for (int fm = 0; fm < 4; ++fm)
#pragma unroll
    for (int fn = 0; fn < 2; ++fn)
      acc[fm][fn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, SWAP ? f.b[fn] : f.a[fm]),
                                                            __builtin_bit_cast(bf16x8, SWAP ? f.a[fm] : f.b[fn]), acc[fm][fn], 0, 0, 0);
}

// acc += P[rp0:+BT, k0:k1] * Q[rq0:+BT, k0:k1]^T (bf16), k0 and k1 multiples of 64;
// XR: acc += P[rp0:+BT, k0:k1] * Q[k0:k1, rq0:+BT]
template <int BT, typename A, int FN, bool XR = false>
__device__ __forceinline__ void gemm_nt_tile_dl(const uint16_t* __restrict__ P,
                                                const uint16_t* __restrict__ Q, int64_t ld, int64_t ldQ,
                                                int rp0, int rq0, int k0, int k1, char* smem,
                                                A (&acc)[4][FN]) {
  typedef DlCfg<BT> C;
  typedef WaveCfg<kBF16, BT> W;
  static_assert(FN == W::FN, "accumulator grid");
  static_assert(BT == 256 && W::NW == 8 && C::NS == 2 && C::LPS == 8, "pipelined loop is written for the 8-wave 256 tile");
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / W::WGN, wn = wave % W::WGN;
  const PE_GLOBAL uint16_t* pP = gview(P) + (size_t)rp0 * ld + k0;
  const PE_GLOBAL uint16_t* pQ = XR ? gview(Q) + (size_t)k0 * ldQ + rq0 : gview(Q) + (size_t)rq0 * ldQ + k0;
  const int nk = (k1 - k0) / C::BK;
  // prologue: stages 0 and 1 in flight (a stage past the end re-reads the last
  // one, which keeps the count of outstanding loads per iteration fixed)
  __syncthreads();  // the previous tile's readers are done with the ring
  dl_issue_stage<BT, XR>(pP, pQ, ld, ldQ, 0, smem, wave, lane);
  dl_issue_stage<BT, XR>(pP, pQ, ld, ldQ, (nk > 1 ? 1 : 0) * C::BK, smem + C::STB, wave, lane);
  // Four 16-deep k-steps per stage, software-pipelined: the fragments of the
  // next k-step are read from LDS while the MFMAs of the current one run, and
  // the stage barrier sits before the last k-step, whose fragments are already
  // in registers, so neither LDS latency nor the barrier stands between two
  // MFMA groups; the loads of stage kt + 2 go out behind it, into the slot just
  // read, four k-steps before they are needed.  Explicit waits at the end of
  // each k-step leave nothing in flight at the loop header, and scheduling
  // fences keep the compiler's scheduler from re-serialising reads and MFMAs.
  constexpr int NRD = XR ? 8 : 6;  // LDS reads per k-step (8 with transposing reads), spread over the 8 MFMAs
  Frags32 f0, f1;
  auto step = [&](const char* st, int sub, Frags32& next, const Frags32& now) {
    __builtin_amdgcn_sched_barrier(0);
    dl_read_frags32<XR>(st, sub, wm, wn, lane, next);
    dl_mfma32<XR>(now, acc);
#pragma unroll
    for (int q = 0; q < NRD; ++q) {
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    }
    if constexpr (NRD < 8) __builtin_amdgcn_sched_group_barrier(0x008, 8 - NRD, 0);
    __builtin_amdgcn_sched_barrier(0);
    wait_lgkm0();
  };
  wait_vmcnt<C::LPS>();
  lds_barrier();  // stage 0 visible
  dl_read_frags32<XR>(smem, 0, wm, wn, lane, f0);
  wait_lgkm0();
  for (int kt = 0; kt < nk; ++kt) {
    char* cur = smem + (kt & 1) * C::STB;
    step(cur, 1, f1, f0);
    step(cur, 2, f0, f1);
    step(cur, 3, f1, f0);
    // own loads of stage kt + 1 landed; after the barrier everyone's have, and
    // every wave has read stage kt
    wait_vmcnt<0>();
    lds_barrier();
    __builtin_amdgcn_sched_barrier(0);
    dl_issue_stage<BT, XR>(pP, pQ, ld, ldQ, (kt + 2 < nk ? kt + 2 : nk - 1) * C::BK, cur, wave, lane);
    const int nx = kt + 1 < nk ? kt + 1 : kt;
    dl_read_frags32<XR>(smem + (nx & 1) * C::STB, 0, wm, wn, lane, f0);
    dl_mfma32<XR>(f1, acc);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      __builtin_amdgcn_sched_group_barrier(0x010, 1, 1);
      if (q < NRD) __builtin_amdgcn_sched_group_barrier(0x100, 1, 1);
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 1);
    }
    __builtin_amdgcn_sched_barrier(0);
    wait_lgkm0();
    __builtin_amdgcn_sched_barrier(0);
  }
  wait_vmcnt<0>();  // no LDS write may still be in flight when the ring is reused
}

// ------------------------------------------------------------- FP8 (e4m3)
// Per-tensor scale: the largest power of two q with amax * 1.01 * q <= 448, so
// x * q is exact and never exceeds the largest e4m3 magnitude (the 1.01 covers
// the bf16 rounding of values whose maximum was taken in fp32).
__device__ __forceinline__ float fp8_scale(float amax) {
  if (!(amax > 0.0f) || !(amax < 3.0e38f)) return 1.0f;
  int e;
  frexpf(448.0f / (amax * 1.01f), &e);
  return ldexpf(1.0f, e - 1);
}

// four floats -> four OCP e4m3 bytes (hardware conversion, round to nearest even)
__device__ __forceinline__ uint32_t pack4_e4m3(float f0, float f1, float f2, float f3) {
  int w = __builtin_amdgcn_cvt_pk_fp8_f32(f0, f1, 0, false);
  w = __builtin_amdgcn_cvt_pk_fp8_f32(f2, f3, w, true);
  return (uint32_t)w;
}

// eight bf16 (one 16-byte chunk) scaled by q -> eight e4m3 bytes
__device__ __forceinline__ uint2 bf16x8_to_e4m3(u32x4 c, float q) {
  uint2 r;
  r.x = pack4_e4m3(__uint_as_float(c[0] << 16) * q, __uint_as_float(c[0] & 0xffff0000u) * q,
                   __uint_as_float(c[1] << 16) * q, __uint_as_float(c[1] & 0xffff0000u) * q);
  r.y = pack4_e4m3(__uint_as_float(c[2] << 16) * q, __uint_as_float(c[2] & 0xffff0000u) * q,
                   __uint_as_float(c[3] << 16) * q, __uint_as_float(c[3] & 0xffff0000u) * q);
  return r;
}

// FP8 stage layout: the bf16 operand is read from HBM and quantised on its way
// into LDS.  BT = 128: 128 k per stage, 16x16x128 f8f6f4 MFMA (lane: 32 bytes
// at k = 32*(lane/16)); BT = 256: 64 k per stage, 32x32x64 f8f6f4 MFMA (lane:
// 32 bytes at k = 32*(lane/32)).  Rows carry a 16-byte pad.
template <int BT>
struct Fp8Cfg {
  static constexpr int F = BT / 8;
  static constexpr int KQ = BT == 128 ? 128 : 64;   // k per stage
  static constexpr int ROWB = KQ + 16;              // LDS bytes per row
  static constexpr int OPB = BT * ROWB;
  static constexpr int LDS = 4 * OPB;
  static constexpr int CPR = KQ / 8;                // 16-byte bf16 chunks per row
  static constexpr int CPT = BT * CPR / kThreads;   // chunks per thread per operand (8)
  static constexpr int RSTRIDE = kThreads / CPR;    // rows between a thread's chunks
};

template <int BT, typename A>
__device__ __forceinline__ void mma_stage_fp8(const char* sA, const char* sB, int wm, int wn,
                                              int lane, A (&acc)[4][4]) {
  typedef Fp8Cfg<BT> C;
  constexpr int F = C::F;
  i32x8 fa[4], fb[4];
  const int koff = (lane / F) * 32;
#pragma unroll
  for (int f = 0; f < 4; ++f) {
    const char* pa = sA + (wm * (BT / 2) + f * F + (lane % F)) * C::ROWB + koff;
    const char* pb = sB + (wn * (BT / 2) + f * F + (lane % F)) * C::ROWB + koff;
    const u32x4 a0 = *(const u32x4*)pa, a1 = *(const u32x4*)(pa + 16);
    const u32x4 b0 = *(const u32x4*)pb, b1 = *(const u32x4*)(pb + 16);
    fa[f] = i32x8{(int)a0[0], (int)a0[1], (int)a0[2], (int)a0[3],
                  (int)a1[0], (int)a1[1], (int)a1[2], (int)a1[3]};
    fb[f] = i32x8{(int)b0[0], (int)b0[1], (int)b0[2], (int)b0[3],
                  (int)b1[0], (int)b1[1], (int)b1[2], (int)b1[3]};
  }
#pragma unroll
  for (int fm = 0; fm < 4; ++fm) {
#pragma unroll
    for (int fn = 0; fn < 4; ++fn) {
      // format 0 = e4m3 for both operands, E8M0 block scales 127 = 1.0
      acc[fm][fn] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(fa[fm], fb[fn], acc[fm][fn],
                                                                     0, 0, 0, 127, 0, 127);
    }
  }
}

// acc += q(P)[rp0:+BT, k0:k1] * q(Q)[rq0:+BT, k0:k1]^T with bf16 operands in HBM
// quantised to e4m3 with scales qp, qq; (k1 - k0) % KQ == 0.
template <int BT, typename A>
__device__ __forceinline__ void gemm_nt_tile_fp8(const uint16_t* __restrict__ P,
                                                 const uint16_t* __restrict__ Q, int64_t ld,
                                                 int rp0, int rq0, int k0, int k1, float qp, float qq,
                                                 char* smem, A (&acc)[4][4]) {
  typedef Fp8Cfg<BT> C;
  constexpr int CPT = C::CPT;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int crow = tid / C::CPR, ccol = tid % C::CPR;
  const PE_GLOBAL uint16_t* pP = gview(P) + (size_t)(rp0 + crow) * ld + k0 + ccol * 8;
  const PE_GLOBAL uint16_t* pQ = gview(Q) + (size_t)(rq0 + crow) * ld + k0 + ccol * 8;
  const size_t jstride = (size_t)C::RSTRIDE * ld;
  u32x4 ra[CPT], rb[CPT];
  const int nk = (k1 - k0) / C::KQ;
#pragma unroll
  for (int j = 0; j < CPT; ++j) {
    ra[j] = *(const PE_GLOBAL u32x4*)(pP + j * jstride);
    rb[j] = *(const PE_GLOBAL u32x4*)(pQ + j * jstride);
  }
  const int soff = crow * C::ROWB + ccol * 8;
#pragma unroll
  for (int j = 0; j < CPT; ++j) {
    *(uint2*)(smem + soff + j * C::RSTRIDE * C::ROWB) = bf16x8_to_e4m3(ra[j], qp);
    *(uint2*)(smem + C::OPB + soff + j * C::RSTRIDE * C::ROWB) = bf16x8_to_e4m3(rb[j], qq);
  }
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    const size_t adv = (size_t)(kt + 1 < nk ? kt + 1 : kt) * C::KQ;
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
      ra[j] = *(const PE_GLOBAL u32x4*)(pP + adv + j * jstride);
      rb[j] = *(const PE_GLOBAL u32x4*)(pQ + adv + j * jstride);
    }
    // keep the prefetch at the top of the stage: a whole stage of MFMA work
    // then covers its latency
    __builtin_amdgcn_sched_barrier(0);
    const char* cur = smem + (kt & 1) * 2 * C::OPB;
    mma_stage_fp8<BT>(cur, cur + C::OPB, wm, wn, lane, acc);
    char* nxt = smem + ((kt + 1) & 1) * 2 * C::OPB;
#pragma unroll
    for (int j = 0; j < CPT; ++j) {
      *(uint2*)(nxt + soff + j * C::RSTRIDE * C::ROWB) = bf16x8_to_e4m3(ra[j], qp);
      *(uint2*)(nxt + C::OPB + soff + j * C::RSTRIDE * C::ROWB) = bf16x8_to_e4m3(rb[j], qq);
    }
    __syncthreads();
  }
}

// ---------------------------------------- FP8 Gram-side main loop, 256 tile
// Once a step's operand maximum is known (X_t: the previous update or the norm
// pass; A_t: the Gram epilogue), a quantisation pass writes its e4m3 copy
// e4m3(q x) (quant_kernel); the product then streams one byte per element
// through the direct-to-LDS ring (128 k per 128-byte row, two
// v_mfma_scale_f32_32x32x64_f8f6f4 k-steps per stage), half the bytes of the
// bf16 ring, and the epilogue multiplies by 1/q^2.  The conversion
// v_cvt_scalef32_pk_fp8_bf16 computes e4m3(x / scale) with round to nearest
// even (two values per instruction); scale = 1/q, a power of two, makes it
// e4m3(q x) exactly.
__device__ __forceinline__ int cvt4_e4m3(uint32_t u0, uint32_t u1, float inv_q) {
  i16x2 r = {0, 0};
  r = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(r, __builtin_bit_cast(bf16x2, u0), inv_q, false);
  r = __builtin_amdgcn_cvt_scalef32_pk_fp8_bf16(r, __builtin_bit_cast(bf16x2, u1), inv_q, true);
  return __builtin_bit_cast(int, r);
}

// Direct-to-LDS issue of one 128-k stage of two e4m3 operands (128 bytes per
// row: the same row geometry and swizzle as a 64-k bf16 stage).
__device__ __forceinline__ void dl_issue_stage_q8(const PE_GLOBAL uint8_t* P, const PE_GLOBAL uint8_t* Q,
                                                  int64_t ld, int kofs, char* slot, int wave, int lane) {
  typedef DlCfg<256> C;
#pragma unroll
  for (int op = 0; op < 2; ++op) {
    const PE_GLOBAL uint8_t* base = op == 0 ? P : Q;
#pragma unroll
    for (int j = 0; j < C::IPW; ++j) {
      const int blk = j * C::NW + wave;             // 1-KB block = 8 rows
      const int lc = dl_swz(wave * 8 + (lane >> 3), lane & 7);
      const PE_GLOBAL uint8_t* g = base + (size_t)(blk * 8) * ld + kofs + (uint32_t)((lane >> 3) * (int)ld + lc * 16);
      __builtin_amdgcn_global_load_lds((const void*)g,
                                       (__attribute__((address_space(3))) void*)(slot + op * C::OPB + blk * 1024),
                                       16, 0, 0);
    }
  }
}

// e4m3 fragments of one half of a 128-k stage for v_mfma_scale_f32_32x32x64_f8f6f4:
// lane l holds row l % 32 and k = 64 sub + 32 (l / 32) + 0..31, i.e. the 16-byte
// chunks 4 sub + 2 (l / 32) and the next of its 128-byte row.
struct FragsQ8 {
  i32x8 a[4], b[2];
};

__device__ __forceinline__ i32x8 q8_row(const char* op, int row, int kh) {
  const char* r = op + row * 128;
  const u32x4 c0 = *(const u32x4*)(r + dl_swz(row, 2 * kh) * 16);
  const u32x4 c1 = *(const u32x4*)(r + dl_swz(row, 2 * kh + 1) * 16);
  return i32x8{(int)c0[0], (int)c0[1], (int)c0[2], (int)c0[3], (int)c1[0], (int)c1[1], (int)c1[2], (int)c1[3]};
}

__device__ __forceinline__ void q8_read(const char* st, int sub, int wm, int wn, int lane, FragsQ8& f) {
  constexpr int OPB = DlCfg<256>::OPB;
  const int kh = 2 * sub + (lane >> 5);
#pragma unroll
  for (int i = 0; i < 4; ++i) f.a[i] = q8_row(st, wm * 128 + i * 32 + (lane & 31), kh);
#pragma unroll
  for (int i = 0; i < 2; ++i) f.b[i] = q8_row(st + OPB, wn * 64 + i * 32 + (lane & 31), kh);
}

template <typename A>
__device__ __forceinline__ void q8_mfma(const FragsQ8& f, A (&acc)[4][2]) {
#pragma unroll
  for (int fm = 0; fm < 4; ++fm)
#pragma unroll
    for (int fn = 0; fn < 2; ++fn)
      // format 0 = e4m3 for both operands, E8M0 block scales 127 = 1.0
      acc[fm][fn] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(f.a[fm], f.b[fn], acc[fm][fn],
                                                                    0, 0, 0, 127, 0, 127);
}

// acc += P[rp0:+256, k0:k1] * Q[rq0:+256, k0:k1]^T with e4m3 operands in HBM
// (already scaled by the quantisation pass); (k1 - k0) % 128 == 0.  Ring of
// two 128-k stages (64 KB each).  One fragment set per wave (two would not fit
// beside the 128 accumulators); the second wave on each SIMD covers the LDS
// latency.
template <typename A>
__device__ __forceinline__ void gemm_nt_tile_dl_q8(const uint8_t* __restrict__ P,
                                                   const uint8_t* __restrict__ Q, int64_t ld, int rp0,
                                                   int rq0, int k0, int k1, char* smem, A (&acc)[4][2]) {
  typedef DlCfg<256> C;
  typedef WaveCfg<kFP8, 256> W;
  static_assert(W::NW == 8 && C::NS == 2 && C::LPS == 8, "ring of the 8-wave 256 tile");
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / W::WGN, wn = wave % W::WGN;
  const PE_GLOBAL uint8_t* pP = (const PE_GLOBAL uint8_t*)P + (size_t)rp0 * ld + k0;
  const PE_GLOBAL uint8_t* pQ = (const PE_GLOBAL uint8_t*)Q + (size_t)rq0 * ld + k0;
  const int nk = (k1 - k0) / 128;
  __syncthreads();  // the previous tile's readers are done with the ring
  dl_issue_stage_q8(pP, pQ, ld, 0, smem, wave, lane);
  dl_issue_stage_q8(pP, pQ, ld, (nk > 1 ? 1 : 0) * 128, smem + C::STB, wave, lane);
  for (int s = 0; s < nk; ++s) {
    // own loads of stage s landed (stage s + 1 may be pending); after the
    // barrier everyone's have
    char* cur = smem + (s & 1) * C::STB;
    wait_vmcnt<C::LPS>();
    lds_barrier();
    FragsQ8 f;
    q8_read(cur, 0, wm, wn, lane, f);
    q8_mfma(f, acc);
    q8_read(cur, 1, wm, wn, lane, f);
    wait_lgkm0();
    lds_barrier();  // every wave has read stage s: its slot takes stage s + 2
    dl_issue_stage_q8(pP, pQ, ld, (s + 2 < nk ? s + 2 : nk - 1) * 128, cur, wave, lane);
    q8_mfma(f, acc);
  }
  wait_vmcnt<0>();  // no LDS write may still be in flight when the ring is reused
}

// Scale of step t's Gram-side operand (kind GRAM: X_t, kind A2: A_t).
__device__ __forceinline__ float fp8_operand_scale(CDesc& d, int kind, int t) {
  float amax;
  if (kind == KIND_GRAM)
    amax = t == 0 ? d.scal[kScAmaxG] : __uint_as_float(((const uint32_t*)d.scal)[kScAmaxX + t]);
  else
    amax = __uint_as_float(((const uint32_t*)d.scal)[kScAmaxA + t]);
  return fp8_scale(amax);
}

// ------------------------------------------------------------- epilogues
// Accumulator element (fm, fn, g, r) is C[row][col] of the block tile with
//   F = 16: row = wm*BT/2 + fm*16 + 4*(lane/16) + r,           col = wn*BT/2 + fn*16 + lane%16
//   F = 32: row = wm*BT/2 + fm*32 + 8*g + 4*(lane/32) + r,     col = wn*WTN + fn*32 + lane%32
// with acc register index 4*g + r (WTN = BT/2 with 4 waves, BT/4 with 8); each
// (fm, fn, g) is four consecutive rows.
template <int BT>
__device__ __forceinline__ int acc_row(int wm, int fm, int g, int lane) {
  constexpr int F = TileCfg<BT>::F;
  return F == 16 ? wm * (BT / 2) + fm * 16 + 4 * (lane >> 4)
                 : wm * (BT / 2) + fm * 32 + 8 * g + 4 * (lane >> 5);
}
template <int P, int BT>
__device__ __forceinline__ int acc_col(int wn, int fn, int lane) {
  constexpr int F = TileCfg<BT>::F;
  return wn * WaveCfg<P, BT>::WTN + fn * F + (lane % F);
}
// The epilogues read one FP32 matrix (A for B = bA + cA^2, X for X = aX + BX)
// at the accumulator positions and write others, possibly the same buffer.
// A lane's inputs of one fragment row fm (4 fragments) are loaded before the
// stores of the previous row are issued, so the loads of a row overlap instead
// of each one waiting behind the stores the compiler must keep ahead of it.
template <int P, int BT>
struct FragRow {
  float x[WaveCfg<P, BT>::FN][TileCfg<BT>::RG][4];  // [fn][row group][r]
};

// red: LDS scratch of at least 4 * NW doubles for the epilogue's block
// reductions (the GEMM kernel gives a tail of its one LDS array, past the
// operand ring and the staging area: a kernel with a single LDS object keeps
// the compiler's LDS-DMA wait tracking from turning into a full vmcnt(0) wait
// after every stage's loads).
// A is exactly symmetric as stored (a tile's mirror holds the same bf16
// values, and a diagonal tile sums the same products in the same order at (i,j)
// and (j,i)), so the four consecutive rows i..i+3 of a lane at column j are the
// contiguous A[j][i..i+3]: one 8-byte load instead of four 2-byte ones.
template <int P, int BT>
__device__ __forceinline__ void load_frag_row_sym(const uint16_t* __restrict__ A, size_t ld, int row0,
                                                  int col0, int wm, int wn, int fm, int lane,
                                                  FragRow<P, BT>& f) {
#pragma unroll
  for (int fn = 0; fn < WaveCfg<P, BT>::FN; ++fn)
#pragma unroll
    for (int g = 0; g < TileCfg<BT>::RG; ++g) {
      const size_t o = (size_t)(col0 + acc_col<P, BT>(wn, fn, lane)) * ld + row0 + acc_row<BT>(wm, fm, g, lane);
      const u32x2 w = *gview((const u32x2*)(A + o));
      f.x[fn][g][0] = __uint_as_float(w[0] << 16);
      f.x[fn][g][1] = __uint_as_float(w[0] & 0xffff0000u);
      f.x[fn][g][2] = __uint_as_float(w[1] << 16);
      f.x[fn][g][3] = __uint_as_float(w[1] & 0xffff0000u);
    }
}

// A transposed bf16 tile of the 256 tile (the update's X^T, a SYRK tile's
// mirror) staged in the operand ring: 256 rows of 256 bf16, padded to 528
// bytes so a 16-byte-aligned row start spreads the column-wise writes over the
// banks
constexpr int kXtStageRow = 528;
constexpr int kXtStageBytes = 256 * kXtStageRow;

// STAGE (bf16 operands of the 256 tile): the tile goes to LDS transposed,
// column by column, and leaves it as whole rows twice: the staged rows are the
// mirror tile's rows, and the tile's own rows are gathered from the staged
// columns with transposing LDS reads (ds_read_b64_tr_b16: within each 16
// lanes, lane 4a+j receives element j of the 8-byte rows addressed by lanes a,
// a+4, a+8, a+12).  Stored directly, the mirror would leave the L2 in 8-byte
// pieces of 64 rows per instruction and the tile in 2-byte ones.
template <int P, int BT, bool STAGE, typename A, int FN>
__device__ __forceinline__ void epi_syrk(const KArgs& args, CDesc& d, int kind, int ti,
                                         int tj, float deq, const A (&acc)[4][FN], double* red,
                                         char* smem) {
  typedef TileCfg<BT> C;
  typedef WaveCfg<P, BT> W;
  static_assert(FN == W::FN, "accumulator grid");
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = wave / W::WGN, wn = wave % W::WGN;
  const size_t sp = d.sp;
  // only B = bA + cA^2 needs the step's coefficients
  float a = 0.0f, b = 0.0f, c = 0.0f;
  if (kind == KIND_A2 && !args.raw_a2) step_coef(args, d, &a, &b, &c);
  float alpha = deq;
  if (kind == KIND_GRAM && args.t == 0) {
    const float sg = d.scal[kScScale];
    alpha *= sg * sg;
  }
  const float calpha = c * deq;
  // B - beta I: the shift leaves the diagonal of the real s x s block
  const bool shifted = kind == KIND_A2 && !args.raw_a2;
  const float beta = shifted ? shift_beta(d, b, c) : 0.0f;
  if (shifted && ti == 0 && tj == 0 && threadIdx.x == 0) d.scal[kScBeta] = beta;
  float amax = 0.0f;
  float trs = 0.0f, frs = 0.0f;  // Gram: this lane's share of tr(A) and of ||A||_F^2 over the tile
  // learned path: this lane's share of the tile's moment partials (FP32; the
  // tiles' partials are summed in FP64 by the selection kernel)
  float mom[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  // the A^2 kinds read A's bf16 copy
  const bool reads_a = kind == KIND_A2;
  static_assert(!STAGE || BT == 256, "mirror staging: tiles of 256");
  const bool stage = STAGE && !(kind == KIND_A2 && args.raw_a2);
  if (stage) __syncthreads();  // every wave is done with the operand ring
  FragRow<P, BT> pre[2];
  auto load_a = [&](int fm, FragRow<P, BT>& f) {
    load_frag_row_sym<P, BT>((const uint16_t*)d.As, sp, ti * BT, tj * BT, wm, wn, fm, lane, f);
  };
  if (reads_a) load_a(0, pre[0]);
#pragma unroll
  for (int fm = 0; fm < 4; ++fm) {
    if (reads_a && fm + 1 < 4) load_a(fm + 1, pre[(fm + 1) & 1]);
    const FragRow<P, BT>& cur = pre[fm & 1];
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) {
#pragma unroll
      for (int g = 0; g < C::RG; ++g) {
        const int i = ti * BT + acc_row<BT>(wm, fm, g, lane);
        const int j = tj * BT + acc_col<P, BT>(wn, fn, lane);
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const size_t o = (size_t)(i + r) * sp + j;
          const float x = acc[fm][fn][4 * g + r];
          if (kind == KIND_GRAM) {
            v[r] = alpha * x;
            if constexpr (!STAGE) ((uint16_t*)d.As)[o] = f2bf(v[r]);
            // the spectrum-aware init's power method reads an FP32 copy of A
            if (args.init_step) d.Af[o] = v[r];
            amax = fmaxf(amax, fabsf(v[r]));
            // (staged tiles take their sum of squares from LDS during the copy-out)
            if constexpr (!STAGE) frs = __builtin_fmaf(v[r], v[r], frs);
          } else if (args.raw_a2) {
            // learned path, step 1: keep A^2 and accumulate tr(A^k) partials;
            // the combine kernel forms B once the schedule class is known
            const float a2 = deq * x;
            const float av = cur.x[fn][g][r];
            v[r] = a2;
            d.A2f[o] = a2;
            if (ti == tj && i + r == j) mom[0] += av;
            mom[1] = __builtin_fmaf(av, av, mom[1]);
            mom[2] = __builtin_fmaf(av, a2, mom[2]);
            mom[3] = __builtin_fmaf(a2, a2, mom[3]);
          } else {
            // same operation order as the learned path's combine kernel
            v[r] = __builtin_fmaf(calpha, x, b * cur.x[fn][g][r]);
            if (ti == tj && i + r == j && j < d.s) v[r] -= beta;
            if constexpr (!STAGE) ((uint16_t*)d.Bs)[o] = f2bf(v[r]);
          }
        }
        if (kind == KIND_GRAM && args.init_step && ti != tj)
          *(float4*)(d.Af + (size_t)j * sp + i) = make_float4(v[0], v[1], v[2], v[3]);
        if (ti != tj && kind == KIND_A2 && args.raw_a2) {
          *(float4*)(d.A2f + (size_t)j * sp + i) = make_float4(v[0], v[1], v[2], v[3]);
        } else if (stage) {
          *(uint2*)(smem + (j - tj * BT) * kXtStageRow + (i - ti * BT) * 2) = pack4_bf16(v);
        } else if (ti != tj) {
          // mirrored tile: row j, columns i..i+3 (contiguous)
          const size_t o = (size_t)j * sp + i;
          *(uint2*)((uint16_t*)(kind == KIND_GRAM ? d.As : d.Bs) + o) = pack4_bf16(v);
        }
      }
    }
  }
  if constexpr (STAGE) if (stage) {
    __syncthreads();
    uint16_t* dst = (uint16_t*)(kind == KIND_GRAM ? d.As : d.Bs);
    if (ti != tj) {
      // mirror rows j = tj*BT + r, columns ti*BT .. +255: 256 rows x 32 chunks of 16 bytes
      uint16_t* mir = dst + (size_t)tj * BT * sp + (size_t)ti * BT;
      for (int ch = threadIdx.x; ch < 256 * 32; ch += W::NT) {
        const int r = ch >> 5, cc = ch & 31;
        *(u32x4*)(mir + (size_t)r * sp + cc * 8) = *(const u32x4*)(smem + r * kXtStageRow + cc * 16);
      }
    }
    // the tile's own rows: each 16 lanes take tile columns 8 jb .. 8 jb + 7
    // (staged rows) of 16 tile rows (staged columns) per step; lane s then
    // holds row 16 ib + s, eight columns, as one 16-byte store
    static_assert(W::NT / 16 == 32, "one 16-lane group per 8 columns");
    const int jb = threadIdx.x >> 4, s = threadIdx.x & 15;
    uint16_t* own = dst + (size_t)ti * BT * sp + (size_t)tj * BT + 8 * jb;
#pragma unroll 4
    for (int ib = 0; ib < 16; ++ib) {
      u32x2 h[2];
#pragma unroll
      for (int rd = 0; rd < 2; ++rd) {
        const char* p = smem + (8 * jb + 4 * rd + (s >> 2)) * kXtStageRow + (16 * ib + 4 * (s & 3)) * 2;
        h[rd] = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                              (__attribute__((address_space(3))) i16x4*)(p)));
      }
      *(u32x4*)(own + (size_t)(16 * ib + s) * sp) = (u32x4){h[0][0], h[0][1], h[1][0], h[1][1]};
      if (kind == KIND_GRAM) {
#pragma unroll
        for (int rd = 0; rd < 2; ++rd)
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const float lo = __uint_as_float(h[rd][e] << 16), hi = __uint_as_float(h[rd][e] & 0xffff0000u);
            frs = __builtin_fmaf(lo, lo, frs);
            frs = __builtin_fmaf(hi, hi, frs);
          }
      }
    }
    // (the next tile's prologue starts with a barrier before it refills the ring)
  }
  // the A^2 product of the same step quantises A with this maximum
  if (kind == KIND_GRAM && args.fp8) wave_amax_atomic(amax, d.scal + kScAmaxA + args.t);
  if (kind == KIND_GRAM) {
    // the tile's partials of tr(A) and ||A||_F^2 (an off-diagonal tile also
    // stands for its mirror), summed in a fixed order; the diagonal is read
    // back once the tile is stored (from the staging area, else from memory:
    // the block's own stores are visible to it after the barrier)
    float* rf = (float*)red;
    __syncthreads();  // tile stored; the previous tile's reader of rf is done
    // (the init step's F^2 = tr A feeds w^2 = F^2 - z^2, which cancels: it
    // takes the FP32 copy of A, not the bf16 one)
    if (ti == tj && threadIdx.x < BT) {
      const int q = threadIdx.x;
      if (args.init_step) trs = d.Af[(size_t)(ti * BT + q) * sp + tj * BT + q];
      else if constexpr (STAGE) trs = bf2f(*(const uint16_t*)(smem + q * kXtStageRow + q * 2));
      else trs = bf2f(((const uint16_t*)d.As)[(size_t)(ti * BT + q) * sp + tj * BT + q]);
    }
    for (int off = 32; off > 0; off >>= 1) {
      trs += __shfl_xor(trs, off);
      frs += __shfl_xor(frs, off);
    }
    if (lane == 0) {
      rf[2 * wave] = trs;
      rf[2 * wave + 1] = frs;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      float t0 = 0.0f, t1 = 0.0f;
#pragma unroll
      for (int w = 0; w < W::NW; ++w) {
        t0 += rf[2 * w];
        t1 += rf[2 * w + 1];
      }
      const int tileid = tri_index(ti, tj, d.nbs);
      d.trp[2 * tileid] = t0;
      d.trp[2 * tileid + 1] = (ti == tj ? 1.0f : 2.0f) * t1;
    }
  }
  if (kind == KIND_A2 && args.raw_a2) {
    // fixed-order block reduction of the tile's moment partials
    // (an off-diagonal tile also stands for its mirror: weight 2 except on tr A)
    const int tileid = tri_index(ti, tj, d.nbs);
    const float wgt = ti == tj ? 1.0f : 2.0f;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      float x = mom[k];
      for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
      mom[k] = x;
    }
    float* rf = (float*)red;
    __syncthreads();
    if (lane == 0)
      for (int k = 0; k < 4; ++k) rf[k * W::NW + wave] = mom[k];
    __syncthreads();
    if (threadIdx.x < 4) {
      const int k = threadIdx.x;
      float t = 0.0f;
#pragma unroll
      for (int w = 0; w < W::NW; ++w) t += rf[k * W::NW + w];
      d.mom[(size_t)tileid * 4 + k] = k == 0 ? t : wgt * t;
    }
  }
}


// ------------------------------------------------ update epilogue, 256 tile
// X <- alpha ((a + beta) X + (B - beta I) X).  With one 8-wave block per CU
// nothing runs beside it, so it is built for few, wide accesses in flight
// early: the accumulators go to LDS in two passes of 128 tile rows (rows
// 64 p .. 64 p + 63 of each wave row in pass p; a lane holds four consecutive
// columns of a row), and leave it as row chunks of eight values, 512
// contiguous bytes per array and 32 lanes.  The chunks' halves of X are loaded
// two groups ahead: the first while the accumulators are staged, the next ones
// while a group is computed and stored.  Eight bytes per element (read lo, hi;
// write lo, hi) where an FP32 master beside the bf16 copy took ten.
constexpr int kUpdRow = 1040;                  // bytes of a staged row: 256 floats and a pad
constexpr int kUpdStageBytes = 128 * kUpdRow;
// float index of (row, column) in a pass's stage; four-float groups are XOR-ed
// by the row's eight-row block, which spreads the column-wise reads of a
// transposed output
__device__ __forceinline__ int upd_idx(int row, int col) { return row * (kUpdRow / 4) + (col ^ (((row >> 3) & 7) << 2)); }

__device__ __forceinline__ void upd_read8(const float* cs, int row, int col, float (&v)[8]) {
  const f32x4 a = *(const f32x4*)(cs + upd_idx(row, col)), b = *(const f32x4*)(cs + upd_idx(row, col + 4));
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    v[e] = a[e];
    v[e + 4] = b[e];
  }
}

// 8 values of a row of the caller's output (row gr, columns gc..) and the Muon
// weight step on the same positions (from the bf16 X where X leaves as bf16, so
// that the two agree)
__device__ __forceinline__ void upd_result(const KArgs& args, CDesc& d, int gr, int gc, int rows, int cols, const float (&v)[8]) {
  if (gr >= rows || gc >= cols) return;
  const bool whole = gc + 8 <= cols;
  u32x4 h;
#pragma unroll
  for (int e = 0; e < 4; ++e) h[e] = pack2_bf16(v[2 * e], v[2 * e + 1]);
  if (d.Out) {
    const size_t o = (size_t)gr * d.ldo + gc;
    if (d.out_bf16) {
      uint16_t* q = (uint16_t*)d.Out + o;
      if (whole && d.o_vec) st_stream((u32x4*)q, h);
      else
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (gc + e < cols) st_stream(q + e, (uint16_t)(h[e >> 1] >> (16 * (e & 1))));
    } else {
      float* q = (float*)d.Out + o;
      if (whole && ((uintptr_t)d.Out % 16 == 0) && d.ldo % 4 == 0) {
        st_stream((f32x4*)q, (f32x4){v[0], v[1], v[2], v[3]});
        st_stream((f32x4*)(q + 4), (f32x4){v[4], v[5], v[6], v[7]});
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (gc + e < cols) st_stream(q + e, v[e]);
      }
    }
  }
  if (d.W) {
    const float keep = 1.0f - args.mlr * args.mwd;
    const bool rounded = d.Out && d.out_bf16;
    const size_t o = (size_t)gr * d.ldw + gc;
    const bool vec = whole && ((uintptr_t)d.W % 16 == 0) && d.ldw % (d.w_bf16 ? 8 : 4) == 0;
    float w[8];
    if (vec && d.w_bf16) {
      const u32x4 raw = *(const PE_GLOBAL u32x4*)(gview((const uint16_t*)d.W) + o);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        w[2 * e] = __uint_as_float(raw[e] << 16);
        w[2 * e + 1] = __uint_as_float(raw[e] & 0xffff0000u);
      }
    } else if (vec) {
      const PE_GLOBAL f32x4* q = (const PE_GLOBAL f32x4*)(gview((const float*)d.W) + o);
      const f32x4 lo = q[0], hi = q[1];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        w[e] = lo[e];
        w[e + 4] = hi[e];
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        w[e] = 0.0f;
        if (gc + e < cols) w[e] = d.w_bf16 ? bf2f(gview((const uint16_t*)d.W)[o + e]) : gview((const float*)d.W)[o + e];
      }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float x = rounded ? bf2f((uint16_t)(h[e >> 1] >> (16 * (e & 1)))) : v[e];
      w[e] = __builtin_fmaf(-args.mlr, x, keep * w[e]);
    }
    if (vec && d.w_bf16) {
      *(PE_GLOBAL u32x4*)(gview_w((uint16_t*)d.W) + o) =
          (u32x4){pack2_bf16(w[0], w[1]), pack2_bf16(w[2], w[3]), pack2_bf16(w[4], w[5]), pack2_bf16(w[6], w[7])};
    } else if (vec) {
      PE_GLOBAL f32x4* q = (PE_GLOBAL f32x4*)(gview_w((float*)d.W) + o);
      q[0] = (f32x4){w[0], w[1], w[2], w[3]};
      q[1] = (f32x4){w[4], w[5], w[6], w[7]};
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (gc + e < cols) {
          if (d.w_bf16) gview_w((uint16_t*)d.W)[o + e] = f2bf(w[e]);
          else gview_w((float*)d.W)[o + e] = w[e];
        }
    }
  }
}

template <int KIND, typename A>
__device__ __forceinline__ void epi_update(const KArgs& args, CDesc& d, int tm, int tn, bool past, const A (&acc)[4][2], char* smem) {
  constexpr bool LAST = KIND == KIND_UPD_LAST, X0B = KIND == KIND_UPD0;
  typedef WaveCfg<kBF16, 256> W;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / W::WGN, wn = wave % W::WGN;
  float* cs = (float*)smem;
  const size_t Lp = d.Lp;
  // X_t of a matrix past its schedule is where its last step left it
  const uint16_t* Xh = xb_at(d, past ? schedule_steps(args, d) : args.t);
  uint16_t* Xn = xb_next(args, d);
  // chunk u (0..7) of pass p: stage row, and offset of its first element
  auto stage_row = [&](int u) { return u * 16 + (tid >> 5); };
  auto tile_row = [&](int p, int sr) { return (sr >> 6) * 128 + p * 64 + (sr & 63); };
  const int col = (tid & 31) * 8;
  u32x4 hi[2][4], lo[2][4];
  auto load_group = [&](int p, int h, u32x4 (&a)[4], u32x4 (&b)[4]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const size_t o = (size_t)(tm * 256 + tile_row(p, stage_row(h * 4 + q))) * Lp + tn * 256 + col;
      a[q] = *(const PE_GLOBAL u32x4*)(gview(Xh) + o);
      if constexpr (!X0B) b[q] = __builtin_nontemporal_load((const PE_GLOBAL u32x4*)(gview((const uint16_t*)d.Xl) + o));
    }
  };
  load_group(0, 0, hi[0], lo[0]);
  float a, b, c;
  step_coef(args, d, &a, &b, &c);
  // the B operand holds B - beta I (a matrix past its schedule copies X: a = 1)
  if (!past) a += d.scal[kScBeta];
  const float alpha = (args.t == 0) ? d.scal[kScScale] : 1.0f;
  float amax = 0.0f;
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    __syncthreads();  // the operand ring, or the previous pass, has been read
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int fn = 0; fn < 2; ++fn)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const auto& x = acc[2 * p + f][fn];
          *(f32x4*)(cs + upd_idx(wm * 64 + f * 32 + (lane & 31), wn * 32 + fn * 128 + 8 * g + 4 * (lane >> 5))) =
              (f32x4){x[4 * g], x[4 * g + 1], x[4 * g + 2], x[4 * g + 3]};
        }
    load_group(p, 1, hi[1], lo[1]);
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int sr = stage_row(h * 4 + q), row = tm * 256 + tile_row(p, sr);
        float v[8], x[8];
        upd_read8(cs, sr, col, v);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if constexpr (X0B) {
            x[2 * e] = __uint_as_float(hi[h][q][e] << 16);
            x[2 * e + 1] = __uint_as_float(hi[h][q][e] & 0xffff0000u);
          } else {
            join2_f32(hi[h][q][e], lo[h][q][e], &x[2 * e], &x[2 * e + 1]);
          }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          v[e] = alpha * (a * x[e] + v[e]);
          amax = fmaxf(amax, fabsf(v[e]));
        }
        if constexpr (!LAST) {
          const size_t o = (size_t)row * Lp + tn * 256 + col;
          u32x4 nh, nl;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            uint32_t h, l;
            split2_f32(v[2 * e], v[2 * e + 1], &h, &l);
            nh[e] = h;
            nl[e] = l;
          }
          *(PE_GLOBAL u32x4*)(gview_w(Xn) + o) = nh;
          __builtin_nontemporal_store(nl, (PE_GLOBAL u32x4*)(gview_w(d.Xl) + o));
        } else if (!d.trans) {
          upd_result(args, d, row, tn * 256 + col, d.s, d.L, v);
        } else {
          *(f32x4*)(cs + upd_idx(sr, col)) = (f32x4){v[0], v[1], v[2], v[3]};
          *(f32x4*)(cs + upd_idx(sr, col + 4)) = (f32x4){v[4], v[5], v[6], v[7]};
        }
      }
      // the registers of this group take the next pass's first one
      if (h == 0 && p == 0) load_group(1, 0, hi[0], lo[0]);
    }
    if constexpr (LAST) {
      if (d.trans) {
        // the caller's rows are tile columns: 8 consecutive tile rows of one
        // column per thread, eight threads along the 64 rows of a wave row
        __syncthreads();
        for (int u = tid; u < 256 * 16; u += W::NT) {
          const int n = u >> 4, r0 = (u & 15) * 8;
          float v[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = cs[upd_idx(r0 + e, n)];
          upd_result(args, d, tn * 256 + n, tm * 256 + tile_row(p, r0), d.L, d.s, v);
        }
      }
    }
  }
  if (!LAST && args.fp8_next) wave_amax_atomic(amax, d.scal + kScAmaxX + args.t + 1);
}

// ------------------------------------------------------------- kernels
template <int P, int KIND, int BT>
__global__ __launch_bounds__((WaveCfg<P, BT>::NT), (BT == 128 ? 2 : 1)) void gemm_kernel(KArgs args) {
  typedef TileCfg<BT> C;
  typedef WaveCfg<P, BT> W;
  typedef typename AccT<C::ACC>::type Acc;
  constexpr int BK = P == kFP8 ? (BT == 256 ? 128 : Fp8Cfg<BT>::KQ) : DlCfg<BT>::BK;
  constexpr bool UPD = KIND == KIND_UPD || KIND == KIND_UPD_LAST || KIND == KIND_UPD0;
  static_assert(P == kBF16 ? BT == 256 : (P == kFP8 && !UPD), "bf16 on the 256 tile; e4m3 Gram-side products");
  // the 256 tile stages a SYRK tile's mirror, or the update's tile, in the
  // buffer of its direct-to-LDS operand ring
  constexpr bool kStageMirror = BT == 256;
  constexpr int LDSB0 = BT == 256 ? DlCfg<256>::LDS : Fp8Cfg<BT>::LDS;
  constexpr int LDSS = BT != 256 ? 0 : UPD ? kUpdStageBytes : kXtStageBytes;
  constexpr int LDSB = LDSB0 < LDSS ? LDSS : LDSB0;
  // SYRK kinds: a small tail past the ring for the epilogue's block reductions
  constexpr int kRedTail = (KIND == KIND_GRAM || KIND == KIND_A2) ? 256 : 0;
  static_assert(kRedTail == 0 || kRedTail >= 4 * W::NW * 8, "moment reduction fits the tail");
  __shared__ __attribute__((aligned(16))) char smem[LDSB + kRedTail];
  for (int slot = blockIdx.x; slot < args.total; slot += gridDim.x) {
    const int item = xcd_item(slot, args.total);
    const int pos = find_mat(args.offs, args.count, item);
    CDesc& d = const_desc(args, args.ord ? const_i32(args.ord, pos) : pos);
    if (skip_matrix(args, d)) continue;
    const bool past = past_schedule(args, d);
    if (past && KIND != KIND_UPD_LAST) continue;
    const int local = item - const_i32(args.offs, pos);
    Acc acc[4][W::FN];
#pragma unroll
    for (int fm = 0; fm < 4; ++fm)
#pragma unroll
      for (int fn = 0; fn < W::FN; ++fn) acc[fm][fn] = Acc{};
    if constexpr (UPD) {
      int tm, tn;
      banded_decode(local, d.nb, d.nbL, &tm, &tn);
      // the update reads X_t itself (row-major, k along its rows); a matrix past
      // its schedule: no product, the epilogue copies X
      // (the init step's B has a second part)
      const int parts = past ? 0 : args.init_step ? 2 : 1;
      for (int h = 0; h < parts; ++h)
        gemm_nt_tile_dl<BT, Acc, W::FN, true>((const uint16_t*)(h ? d.As : d.Bs), xb_cur(args, d), d.sp, d.Lp, tm * BT,
                                               tn * BT, 0, d.sp, smem, acc);
      epi_update<KIND>(args, d, tm, tn, past, acc, smem);
    } else {
      const int split = KIND == KIND_GRAM ? d.gram_split : d.a2_split;
      const int tile = local / split, ksp = local % split;
      int ti, tj;
      tri_decode_banded(tile, d.nbs, &ti, &tj);
      const uint16_t* Op = KIND == KIND_GRAM ? xb_cur(args, d) : (const uint16_t*)d.As;
      const int K = KIND == KIND_GRAM ? d.Lp : d.sp;
      int k0, k1;
      split_range(K, split, ksp, BK, &k0, &k1);
      // a degree-3 step (c = 0 in the fixed schedule) needs no A^2: the
      // epilogue forms B = b A - beta I from an empty product
      if (KIND == KIND_A2 && !args.sel_coef && args.c == 0.0f) k1 = k0;
      float deq = 1.0f;
      if constexpr (P == kFP8) {
        const float q = fp8_operand_scale(d, KIND, args.t);
        deq = 1.0f / (q * q);
        if constexpr (BT == 256) {
          // e4m3 copies written by the quantisation pass (scale q already applied)
          const uint8_t* Oq = KIND == KIND_GRAM ? d.Xq : d.Aq;
          if (k1 > k0) gemm_nt_tile_dl_q8(Oq, Oq, K, ti * BT, tj * BT, k0, k1, smem, acc);
        } else {
          if (k1 > k0) gemm_nt_tile_fp8<BT>(Op, Op, K, ti * BT, tj * BT, k0, k1, q, q, smem, acc);
        }
      } else {
        if (k1 > k0)
          gemm_nt_tile_dl<BT>(Op, Op, K, K, ti * BT, tj * BT, k0, k1, smem, acc);
      }
      if (split == 1) {
        epi_syrk<P, BT, kStageMirror>(args, d, KIND, ti, tj, deq, acc, (double*)(smem + LDSB), smem);
      } else {
        // partial tile: float4 q of thread t at ((tile*split + ksp)*Q + q)*NT + t
        constexpr int Q = 4 * W::FN * C::ACC / 4;
        float4* part = (float4*)d.part + ((size_t)(tile * split + ksp) * Q) * W::NT;
#pragma unroll
        for (int fm = 0; fm < 4; ++fm)
#pragma unroll
          for (int fn = 0; fn < W::FN; ++fn)
#pragma unroll
            for (int g = 0; g < C::ACC / 4; ++g) {
              const int q = (fm * W::FN + fn) * (C::ACC / 4) + g;
              part[q * W::NT + threadIdx.x] =
                  make_float4(acc[fm][fn][4 * g], acc[fm][fn][4 * g + 1], acc[fm][fn][4 * g + 2],
                              acc[fm][fn][4 * g + 3]);
            }
      }
    }
  }
}

// ------------------------------------------------ spectrum-aware init
// Power method on the step-1 Gram matrix A = X X^T (appendix on matrices with
// large spectral gaps, k = 1): v_0 = the sign vector of Knuth's hash of the
// index (+-1/sqrt(s)), v <- A v / ||A v||; after the last step
// z = sqrt(||A v||) <= sigma_1, F^2 = tr A, w = sqrt(F^2 - z^2), and when
// z > w the cubic through (w, 1) and (z, 1):
//   a = (z^2 + z w + w^2) / (z w (z + w)),  b = -1 / (z w (z + w))
// (identity otherwise) is applied as an extra first step X <- a X + b A X.
// One launch per power step: y_k = A v_k with v_k = y_{k-1} / ||y_{k-1}||, where
// every wave adds up the norm of the previous product itself (a few KB, in one
// fixed order) instead of a launch of its own doing it once (16 steps on 1024 x
// 4096 and 1024 x 1024: 32 launches, 177 us, before; 17 launches now).  The two
// halves of d.vec take turns as y.
// ||y|| over [0, sp) (padding is zero), the same bits in every lane
template <typename F = float>
__device__ __forceinline__ F pw_norm(const float* y, int sp) {
  const int lane = threadIdx.x & 63;
  F ss = 0;
  for (int i = 4 * lane; i < sp; i += 256) {
    const f32x4 v = *(const PE_GLOBAL f32x4*)gview(y + i);
#pragma unroll
    for (int e = 0; e < 4; ++e) ss = fma((F)v[e], (F)v[e], ss);
  }
  for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
  return sqrt(ss);
}
// what pw_matvec_kernel multiplies the previous product by
__device__ __forceinline__ float pw_inverse(const float* prev, int sp) {
  const float nrm = pw_norm(prev, sp);
  return nrm > 0.0f ? 1.0f / nrm : 0.0f;
}

// one wave per row, four rows per item, from the FP32 A (the fp32 path's own A;
// on the bf16 paths the copy the init step's Gram epilogue writes: w^2 = tr A -
// z^2 cancels, and its error grows as z^2 / w^2 times that of z, which bf16 A
// would make useless).  est_phase: the step k.
__global__ __launch_bounds__(256) void pw_matvec_kernel(KArgs args) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int item = blockIdx.x; item < args.total; item += gridDim.x) {
    const int mi = find_mat(args.offs, args.count, item);
    CDesc& d = const_desc(args, mi);
    const int r = (item - const_i32(args.offs, mi)) * 4 + wave, sp = d.sp;
    if (r >= sp) continue;
    const float* row = d.Af + (size_t)r * sp;
    const float* prev = d.vec + (size_t)((args.est_phase + 1) & 1) * sp;
    float acc = 0.0f;
    if (args.est_phase == 0) {
      const float sc = rsqrtf((float)d.s);
      for (int j = 4 * lane; j < sp; j += 256) {
        const f32x4 a = *(const PE_GLOBAL f32x4*)gview(row + j);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t h = (uint32_t)(j + e) * 2654435761u;
          acc = __builtin_fmaf(a[e], j + e < d.s ? ((h & 0x80000000u) ? -sc : sc) : 0.0f, acc);
        }
      }
    } else {
      const float inv = pw_inverse(prev, sp);
      for (int j = 4 * lane; j < sp; j += 256) {
        const f32x4 a = *(const PE_GLOBAL f32x4*)gview(row + j), v = *(const PE_GLOBAL f32x4*)gview(prev + j);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = __builtin_fmaf(a[e], v[e] * inv, acc);
      }
    }
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    if (lane == 0) d.vec[(size_t)(args.est_phase & 1) * sp + r] = acc;
  }
}

// After the last power step (est_phase: their number): the init coefficients.
// w^2 = F^2 - z^2 cancels by kappa = z^2 / w^2, so both are formed in FP64 and
// from the same matrix: z^2 = ||A v|| / ||v|| with the norm that v was left with,
// and F^2 = tr A or, on the fp32 paths, where the diagonal of A may lack the
// products of low planes (4e-8 of it, all of one sign), the norm pass's sum times
// the square of sigma that scaled A.  In FP32 their rounding was 6e-8 kappa
// of w^2 (2048 x 2304, kappa 1e5: 8.3e-3 of the result against 64 bits).
__global__ __launch_bounds__(64) void pw_coef_kernel(KArgs args) {
  const int lane = threadIdx.x & 63;
  for (int mi = blockIdx.x; mi < args.count; mi += gridDim.x) {
    CDesc& d = const_desc(args, mi);
    if (d.syrk_nt == 0) continue;
    const float *y = d.vec + (size_t)((args.est_phase + 1) & 1) * d.sp, *prev = d.vec + (size_t)(args.est_phase & 1) * d.sp;
    const double nv = args.est_phase == 1 ? rsqrtf((float)d.s) * sqrt((double)d.s) : pw_inverse(prev, d.sp) * pw_norm<double>(prev, d.sp);
    const double z2 = nv > 0.0 ? pw_norm<double>(y, d.sp) / nv : 0.0;
    double F2 = 0.0;
    if (d.Xl) {
      for (int u = lane; u < d.syrk_nt; u += 64) F2 += d.trp[2 * u];
      F2 = wave_sum(F2);
    } else {
      const float sigma = matrix_sigma(args, d);
      F2 = matrix_square_sum(d) * (sigma * sigma);
    }
    if (lane == 0) {
      float a = 1.0f, b = 0.0f;
      const double z = sqrt(z2), w2 = F2 - z2;
      if (z > 0.0 && w2 > 0.0) {
        const double w = sqrt(w2);
        if (z > w) {
          const double den = z * w * (z + w);
          a = (float)((z * z + z * w + w * w) / den);
          b = (float)(-1.0 / den);
        }
      }
      d.scal[kScInitA] = a;
      d.scal[kScInitB] = b;
      // fp32 path: B = b A - beta I has entries up to 2 |b| (A's norm is at most 1)
      int ex = 0;
      if (b != 0.0f) frexpf(2.0f * fabsf(b), &ex);
      d.scal[kScInitQ] = ldexpf(1.0f, 14 - ex);
    }
  }
}

// B = b A - beta I of the init step on the bf16 paths, one row per item, from
// the FP32 A and in two bf16 parts (Bs, and As, whose A no one reads any more).
// The cubic cancels at the outlying value (16 - 15 where that is 15 times the
// rest) and the schedule's slope there is some hundreds, so a relative error of
// B's top eigenvalue reaches the result 3000 times as large; from the bf16 A,
// whose rounding is the same for all entries of one mantissa and does not average
// out, it was 2e-6 to 1.4e-4 (960 x 640: 7.1e-3 against 64 bits).  A pass over A
// at memory speed.
__global__ __launch_bounds__(256) void init_b_kernel(KArgs args) {
  for (int item = blockIdx.x; item < args.total; item += gridDim.x) {
    const int mi = find_mat(args.offs, args.count, item);
    CDesc& d = const_desc(args, mi);
    const int row = item - const_i32(args.offs, mi), sp = d.sp;
    const float b = d.scal[kScInitB], beta = shift_beta(d, b, 0.0f);
    if (row == 0 && threadIdx.x == 0) d.scal[kScBeta] = beta;
    const size_t base = (size_t)row * sp;
    for (int j = 4 * threadIdx.x; j < sp; j += 4 * blockDim.x) {
      const f32x4 a = *(const PE_GLOBAL f32x4*)gview(d.Af + base + j);
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = b * a[e] - (j + e == row && row < d.s ? beta : 0.0f);
      const uint32_t h0 = pack2_bf16(v[0], v[1]), h1 = pack2_bf16(v[2], v[3]);
      *(PE_GLOBAL u32x2*)(gview_w((uint16_t*)d.Bs) + base + j) = (u32x2){h0, h1};
      *(PE_GLOBAL u32x2*)(gview_w((uint16_t*)d.As) + base + j) =
          (u32x2){pack2_bf16(v[0] - __uint_as_float(h0 << 16), v[1] - __uint_as_float(h0 & 0xffff0000u)),
                  pack2_bf16(v[2] - __uint_as_float(h1 << 16), v[3] - __uint_as_float(h1 & 0xffff0000u))};
    }
  }
}

// e4m3 copy of step t's Gram-side operand (KIND_GRAM: X_t from Xb into Xq;
// KIND_A2: A_t from As into Aq) with the step's per-tensor scale.  One item is
// 16384 elements (four chunks of 16 per thread, all loads issued first); the
// padded sizes are multiples of 65536.
template <int KIND>
__global__ __launch_bounds__(kThreads) void quant_kernel(KArgs args) {
  constexpr int kChunks = 4;
  for (int item = blockIdx.x; item < args.total; item += gridDim.x) {
    const int mi = find_mat(args.offs, args.count, item);
    CDesc& d = const_desc(args, mi);
    if (skip_matrix(args, d) || past_schedule(args, d)) continue;
    const size_t base = (size_t)(item - const_i32(args.offs, mi)) * kChunks * kThreads * 16;
    const uint16_t* src = KIND == KIND_GRAM ? xb_cur(args, d) : (const uint16_t*)d.As;
    uint8_t* dst = KIND == KIND_GRAM ? d.Xq : d.Aq;
    const float inv_q = 1.0f / fp8_operand_scale(d, KIND, args.t);
    u32x4 c[kChunks][2];
#pragma unroll
    for (int k = 0; k < kChunks; ++k) {
      const size_t e0 = base + ((size_t)k * kThreads + threadIdx.x) * 16;
      c[k][0] = *(const PE_GLOBAL u32x4*)(gview(src) + e0);
      c[k][1] = *(const PE_GLOBAL u32x4*)(gview(src) + e0 + 8);
    }
#pragma unroll
    for (int k = 0; k < kChunks; ++k) {
      const size_t e0 = base + ((size_t)k * kThreads + threadIdx.x) * 16;
      const u32x4 o = {(uint32_t)cvt4_e4m3(c[k][0][0], c[k][0][1], inv_q), (uint32_t)cvt4_e4m3(c[k][0][2], c[k][0][3], inv_q),
                       (uint32_t)cvt4_e4m3(c[k][1][0], c[k][1][1], inv_q), (uint32_t)cvt4_e4m3(c[k][1][2], c[k][1][3], inv_q)};
      st_stream((u32x4*)(dst + e0), o);
    }
  }
}

template <int P, int KIND, int BT>
__global__ __launch_bounds__((WaveCfg<P, BT>::NT)) void splitk_reduce_kernel(KArgs args) {
  typedef TileCfg<BT> C;
  typedef WaveCfg<P, BT> W;
  typedef typename AccT<C::ACC>::type Acc;
  constexpr int Q = 4 * W::FN * C::ACC / 4;
  __shared__ double red[4 * W::NW];
  for (int item = blockIdx.x; item < args.total; item += gridDim.x) {
    const int mi = find_mat(args.offs, args.count, item);
    CDesc& d = const_desc(args, mi);
    if (skip_matrix(args, d) || past_schedule(args, d)) continue;
    const int tile = item - const_i32(args.offs, mi);
    const int split = KIND == KIND_GRAM ? d.gram_split : d.a2_split;
    int ti, tj;
    tri_decode_banded(tile, d.nbs, &ti, &tj);
    Acc acc[4][W::FN];
    const float4* part = (const float4*)d.part + ((size_t)tile * split * Q) * W::NT;
#pragma unroll
    for (int fm = 0; fm < 4; ++fm)
#pragma unroll
      for (int fn = 0; fn < W::FN; ++fn)
#pragma unroll
        for (int g = 0; g < C::ACC / 4; ++g) {
          const int q = (fm * W::FN + fn) * (C::ACC / 4) + g;
          float4 s = part[q * W::NT + threadIdx.x];
          for (int k = 1; k < split; ++k) {
            const float4 p = part[((size_t)k * Q + q) * W::NT + threadIdx.x];
            s.x += p.x; s.y += p.y; s.z += p.z; s.w += p.w;
          }
          acc[fm][fn][4 * g] = s.x;
          acc[fm][fn][4 * g + 1] = s.y;
          acc[fm][fn][4 * g + 2] = s.z;
          acc[fm][fn][4 * g + 3] = s.w;
        }
    float deq = 1.0f;
    if constexpr (P == kFP8) {
      const float q = fp8_operand_scale(d, KIND, args.t);
      deq = 1.0f / (q * q);
    }
    epi_syrk<P, BT, false>(args, d, KIND, ti, tj, deq, acc, red, nullptr);
  }
}

// q[i] = e4m3(x[i] * scale) with the conversion the FP8 path uses.
// bf16 input with a power-of-two scale takes the instruction of the FP8
// steps' quantisation pass (e4m3(x / (1/scale)), exact); other inputs scale in
// fp32 and convert with v_cvt_pk_fp8_f32.
__global__ void quantize_e4m3_kernel(const void* x, int x_bf16, uint8_t* q, int64_t n, float scale,
                                     int pow2) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    if (x_bf16 && pow2) {
      const uint32_t u = ((const uint16_t*)x)[i];
      q[i] = (uint8_t)((uint32_t)cvt4_e4m3(u, 0u, 1.0f / scale) & 0xffu);
    } else {
      const float v = x_bf16 ? bf2f(((const uint16_t*)x)[i]) : ((const float*)x)[i];
      q[i] = (uint8_t)(pack4_e4m3(v * scale, 0.0f, 0.0f, 0.0f) & 0xffu);
    }
  }
}

__global__ void put_words_kernel(PutChunk c) {
  for (int i = threadIdx.x; i < c.nwords; i += blockDim.x) c.dst[i] = c.w[i];
}

// ------------------------------------------------------------- launchers
hipError_t launch_finalize(const KArgs& a, hipStream_t st) {
  const int g = a.count < 1024 ? (a.count > 0 ? a.count : 1) : 1024;
  hipLaunchKernelGGL(finalize_kernel, dim3(g), dim3(kThreads), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_put(const PutChunk& c, hipStream_t st) {
  hipLaunchKernelGGL(put_words_kernel, dim3(1), dim3(kThreads), 0, st, c);
  return hipGetLastError();
}

// Blocks of a kernel that fit on the device at once (occupancy calculator x CU
// count), cached per device and kernel; 0 if the runtime cannot say.  A
// grid-stride kernel launched with more blocks than this runs the surplus in
// a second round that leaves most of the device idle.
static int resident_blocks(const void* kernel, int threads) {
  constexpr int kDev = 16, kSlots = 64;
  static const void* keys[kDev][kSlots];
  static int vals[kDev][kSlots];
  static std::mutex mu;
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kDev) return 0;
  std::lock_guard<std::mutex> lock(mu);
  for (int i = 0; i < kSlots; ++i) {
    if (keys[dev][i] == kernel) return vals[dev][i];
    if (keys[dev][i]) continue;
    int ncu = 0, per = 0;
    if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, threads, 0) != hipSuccess) {
      (void)hipGetLastError();  // a failed query must not read as a failed launch
      return 0;
    }
    keys[dev][i] = kernel;
    vals[dev][i] = per * ncu;
    return vals[dev][i];
  }
  return 0;
}

template <typename K>
static int grid_for(int total, int cap, K kernel, int threads) {
  const int res = resident_blocks(reinterpret_cast<const void*>(kernel), threads);
  if (res > 0 && res < cap) cap = res;
  return total < cap ? (total > 0 ? total : 1) : cap;
}

template <int P, int BT>
static void warm_t() {
  constexpr int nt = WaveCfg<P, BT>::NT;
  resident_blocks(reinterpret_cast<const void*>(gemm_kernel<P, KIND_GRAM, BT>), nt);
  resident_blocks(reinterpret_cast<const void*>(gemm_kernel<P, KIND_A2, BT>), nt);
  if constexpr (P == kBF16) {
    resident_blocks(reinterpret_cast<const void*>(gemm_kernel<P, KIND_UPD, BT>), nt);
    resident_blocks(reinterpret_cast<const void*>(gemm_kernel<P, KIND_UPD_LAST, BT>), nt);
    resident_blocks(reinterpret_cast<const void*>(gemm_kernel<P, KIND_UPD0, BT>), nt);
  }
  resident_blocks(reinterpret_cast<const void*>(splitk_reduce_kernel<P, KIND_GRAM, BT>), nt);
  resident_blocks(reinterpret_cast<const void*>(splitk_reduce_kernel<P, KIND_A2, BT>), nt);
}

// Fills the resident-block cache of the current device, so that launches
// recorded into a graph later make no runtime queries.
void warm_launch_grids() {
  resident_blocks(reinterpret_cast<const void*>(prep_kernel<kF32>), kThreads);
  resident_blocks(reinterpret_cast<const void*>(prep_kernel<kF32M>), kThreads);
  resident_blocks(reinterpret_cast<const void*>(prep_kernel<kBF16>), kThreads);
  resident_blocks(reinterpret_cast<const void*>(quant_kernel<KIND_GRAM>), kThreads);
  resident_blocks(reinterpret_cast<const void*>(quant_kernel<KIND_A2>), kThreads);
  warm_t<kBF16, 256>();
  warm_t<kFP8, 128>();
  warm_t<kFP8, 256>();
}

hipError_t launch_prep(int prec, const KArgs& a, int grid_cap, hipStream_t st) {
  auto k = prec == kBF16 ? prep_kernel<kBF16> : prec == kF32M ? prep_kernel<kF32M> : prep_kernel<kF32>;
  hipLaunchKernelGGL(k, dim3(grid_for(a.total, grid_cap, k, kThreads)), dim3(kThreads), 0, st, a);
  return hipGetLastError();
}

template <int P, int BT>
static void launch_gemm_t(int kind, const KArgs& a, int cap, hipStream_t st) {
  auto k = kind == KIND_GRAM ? gemm_kernel<P, KIND_GRAM, BT> : gemm_kernel<P, KIND_A2, BT>;
  if constexpr (P == kBF16)
    if (kind == KIND_UPD)
      k = a.last ? gemm_kernel<P, KIND_UPD_LAST, BT> : a.x0b ? gemm_kernel<P, KIND_UPD0, BT> : gemm_kernel<P, KIND_UPD, BT>;
  constexpr int nt = WaveCfg<P, BT>::NT;
  hipLaunchKernelGGL(k, dim3(grid_for(a.total, cap, k, nt)), dim3(nt), 0, st, a);
}

template <int P, int BT>
static void launch_reduce_t(int kind, const KArgs& a, int cap, hipStream_t st) {
  auto k = kind == KIND_GRAM ? splitk_reduce_kernel<P, KIND_GRAM, BT> : splitk_reduce_kernel<P, KIND_A2, BT>;
  constexpr int nt = WaveCfg<P, BT>::NT;
  hipLaunchKernelGGL(k, dim3(grid_for(a.total, cap, k, nt)), dim3(nt), 0, st, a);
}

hipError_t launch_update_tail(KArgs a, hipStream_t st);

// The bf16 256 tile, and the e4m3 Gram-side products on either tile.  An update
// whose last round has at most a fourth of its tiles runs those as smaller ones,
// one per CU, in a launch of their own: the round would take as long as a full
// one (48 GPT-small matrices, 1296 tiles, 16 in the sixth round: 229 -> 206 + 12
// us per update; two 3072 x 3072, 288 tiles: 1694 -> 1543 us per call, one 4096 x
// 5120, 320 tiles: 2176 -> 1992).  With half a round left it gives nothing (512 x
// 2048 x 24, 384 tiles: 545.7 and 547.2; 2048 x 4096 x 3: 1451 and 1425).
hipError_t launch_gemm(int prec, int bt, int kind, const KArgs& all, int grid_cap, hipStream_t st) {
  KArgs a = all;
  if (kind == KIND_UPD) {
    const int round = grid_for(1 << 30, grid_cap, gemm_kernel<kBF16, KIND_UPD, 256>, WaveCfg<kBF16, 256>::NT);
    const int rest = !a.alike && a.total > round && a.total % round <= round / 4 ? a.total % round : 0;
    a.total -= rest;
    launch_gemm_t<kBF16, 256>(kind, a, grid_cap, st);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || !rest) return e;
    a.tail = a.total;
    a.total = rest;
    return launch_update_tail(a, st);
  }
  if (prec != kFP8) launch_gemm_t<kBF16, 256>(kind, a, grid_cap, st);
  else if (bt == 256) launch_gemm_t<kFP8, 256>(kind, a, grid_cap, st);
  else launch_gemm_t<kFP8, 128>(kind, a, grid_cap, st);
  return hipGetLastError();
}

// phase 0: one power step (a.est_phase), 1: the init coefficients
hipError_t launch_power(int phase, const KArgs& a, hipStream_t st) {
  if (phase == 0) {
    const int g = a.total < 2048 ? (a.total > 0 ? a.total : 1) : 2048;
    hipLaunchKernelGGL(pw_matvec_kernel, dim3(g), dim3(256), 0, st, a);
  } else {
    const int g = a.count < 1024 ? (a.count > 0 ? a.count : 1) : 1024;
    hipLaunchKernelGGL(pw_coef_kernel, dim3(g), dim3(64), 0, st, a);
  }
  return hipGetLastError();
}

hipError_t launch_init_b(const KArgs& a, hipStream_t st) {
  hipLaunchKernelGGL(init_b_kernel, dim3(a.total < 4096 ? a.total : 4096), dim3(256), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_quant(int kind, const KArgs& a, int grid_cap, hipStream_t st) {
  auto k = kind == KIND_GRAM ? quant_kernel<KIND_GRAM> : quant_kernel<KIND_A2>;
  hipLaunchKernelGGL(k, dim3(grid_for(a.total, grid_cap, k, kThreads)), dim3(kThreads), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_reduce(int prec, int bt, int kind, const KArgs& a, int grid_cap, hipStream_t st) {
  if (prec != kFP8) launch_reduce_t<kBF16, 256>(kind, a, grid_cap, st);
  else if (bt == 256) launch_reduce_t<kFP8, 256>(kind, a, grid_cap, st);
  else launch_reduce_t<kFP8, 128>(kind, a, grid_cap, st);
  return hipGetLastError();
}

hipError_t launch_quantize(const void* x, int x_bf16, uint8_t* q, int64_t n, float scale,
                           hipStream_t st) {
  const int64_t blocks = (n + kThreads - 1) / kThreads;
  const int g = (int)(blocks < 4096 ? (blocks > 0 ? blocks : 1) : 4096);
  int e2 = 0;
  const int pow2 = frexpf(scale, &e2) == 0.5f;
  hipLaunchKernelGGL(quantize_e4m3_kernel, dim3(g), dim3(kThreads), 0, st, x, x_bf16, q, n, scale, pow2);
  return hipGetLastError();
}

}  // namespace pe
