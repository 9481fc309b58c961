// gfx950 kernels of the small block tiles, 64 x 64 and 128 x 128 (bf16 and fp32
// paths; the fp32 path's operands are fp16 planes, see pe_device.h):
// the grouped products of kernels.hip for matrices whose 256-wide tiles would
// leave most of the chip idle or pad away too much of the work.
//
// What bounds them: on one matrix of a few hundred to a few thousand rows a
// launch has at most a few hundred tiles, its operands sit in memory behind
// the previous launch's write-back, and the time is latency -- the descriptor
// loads, the operand loads of each k-stage, the epilogue's own loads and
// narrow stores -- not the MFMA rate.  So:
//  * the operand ring is as deep as the LDS allows (one block per CU when the
//    launch has no more tiles than CUs), which puts 128 KB of loads in flight
//    per CU before the first wait;
//  * a stage is 64 deep, 128 bytes per row: direct-to-LDS loads of 64-byte row
//    pieces run at 33 bytes per clock and CU, of 128-byte pieces at 55, and the
//    64 tile's products could use 128 (4096 x 1024: Gram product 20.7 -> 17.8 us;
//    48 GPT-small matrices: 118 -> 105; 4096 x 1024 in all 270 -> 249);
//  * the 64 tile gives each of its four waves every fourth k-stage and
//    a ring of its own, so its main loop has no barrier at all; the four
//    partial tiles are summed through LDS in a fixed order;
//  * what the epilogue reads (X, A, the shift's partial sums) is loaded before
//    the main loop;
//  * the tile leaves through LDS as row-major FP32, 16 consecutive values per
//    thread: every global access of the epilogue is a 16-byte access of a
//    contiguous row, the mirror tile of a symmetric product and a transposed
//    output included (they are read back column by column from a swizzled LDS
//    tile).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "pe_kernels.h"

namespace pe {

// BT: tile edge; KW: groups of waves that share out the k-stages (a group is
// one wave on the 64 tile, four waves in 2 x 2 on the 128 tile; a wave always
// holds 64 x 64 accumulators); NS: stages of BK k in each group's ring; PL:
// planes per operand (1: bf16; 2: the fp32 path's fp16 planes; 0: fp32 itself,
// matrices of fewer than 16 rows).
template <int BT_, int KW_, int NS_, int PL_ = 1, int BK_ = 64>
struct SmallTile {
  static constexpr int BT = BT_, KW = KW_, NS = NS_, PL = PL_, BK = BK_;
  static constexpr int WPG = BT == 64 ? 1 : 4;       // waves per group
  static constexpr int NW = KW * WPG, NT = NW * 64;
  static constexpr int OPB = BT * BK * 2;            // one operand plane, one k-stage
  static constexpr int STB = 2 * PL * OPB;           // one stage (PL = 0: tiny_product's staging instead)
  static constexpr int CB = BT * (BT + 4) * 4;       // bytes of the staged tile
  static constexpr int CPR = BT / 16;                // 16-value chunks per tile row
  static constexpr int NCH = BT * CPR / NT;          // chunks per thread
  static constexpr int LPW = OPB / 1024 / WPG;       // 1-KB loads per wave, plane and stage
  static constexpr int LPS = 2 * PL * LPW;           // load instructions per wave and stage
  static constexpr int REGION = NS * STB > CB ? NS * STB : CB;
  static constexpr int LDS = PL == 0 ? CB + 2 * 16 * 132 * 4 : KW * REGION;
  // chunk p of this thread: tile row and first column
  static __device__ __forceinline__ int row(int p) { return (p * NT + (int)threadIdx.x) / CPR; }
  static __device__ __forceinline__ int col() { return ((int)threadIdx.x % CPR) * 16; }
};
constexpr int kSmallTail = 256;  // block reductions of the epilogues, past the ring

// Staged tile: row-major with the 16-float units of a row XOR-ed by the row's
// own 16-row unit, so that rows are read in 16-byte pieces and columns (16
// rows apart between neighbouring lanes) without more than two-way conflicts.
template <int BT>
__device__ __forceinline__ int cs_idx(int row, int col) {
  return row * (BT + 4) + (col ^ (((row >> 4) & (BT / 16 - 1)) << 4));
}

template <int BT>
__device__ __forceinline__ void cs_load(const float* cs, int row, int col, float (&v)[16]) {
  const float* p = cs + cs_idx<BT>(row, col);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const f32x4 x = *(const f32x4*)(p + 4 * q);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[4 * q + e] = x[e];
  }
}
template <int BT>
__device__ __forceinline__ void cs_store(float* cs, int row, int col, const float (&v)[16]) {
  float* p = cs + cs_idx<BT>(row, col);
#pragma unroll
  for (int q = 0; q < 4; ++q) *(f32x4*)(p + 4 * q) = (f32x4){v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
}
// column `col` of the staged tile, rows row..row+15
template <int BT>
__device__ __forceinline__ void cs_load_t(const float* cs, int row, int col, float (&v)[16]) {
#pragma unroll
  for (int e = 0; e < 16; ++e) v[e] = cs[cs_idx<BT>(row + e, col)];
}

__device__ __forceinline__ void load16(const float* src, float (&v)[16]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const f32x4 x = *(const PE_GLOBAL f32x4*)(gview(src) + 4 * q);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[4 * q + e] = x[e];
  }
}
__device__ __forceinline__ void load16(const uint16_t* src, float (&v)[16]) {
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const u32x4 x = *(const PE_GLOBAL u32x4*)(gview(src) + 8 * q);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[8 * q + 2 * e] = __uint_as_float(x[e] << 16);
      v[8 * q + 2 * e + 1] = __uint_as_float(x[e] & 0xffff0000u);
    }
  }
}
// 16 values of the two-halves iterate
__device__ __forceinline__ void load16_halves(const uint16_t* hi, const uint16_t* lo, float (&v)[16]) {
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const u32x4 h = *(const PE_GLOBAL u32x4*)(gview(hi) + 8 * q), l = *(const PE_GLOBAL u32x4*)(gview(lo) + 8 * q);
#pragma unroll
    for (int e = 0; e < 4; ++e) join2_f32(h[e], l[e], &v[8 * q + 2 * e], &v[8 * q + 2 * e + 1]);
  }
}
__device__ __forceinline__ void store16_halves(uint16_t* hi, uint16_t* lo, const float (&v)[16]) {
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    u32x4 h, l;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      uint32_t a, b;
      split2_f32(v[8 * q + 2 * e], v[8 * q + 2 * e + 1], &a, &b);
      h[e] = a;
      l[e] = b;
    }
    *(PE_GLOBAL u32x4*)(gview_w(hi) + 8 * q) = h;
    *(PE_GLOBAL u32x4*)(gview_w(lo) + 8 * q) = l;
  }
}
__device__ __forceinline__ void store16(float* dst, const float (&v)[16]) {
#pragma unroll
  for (int q = 0; q < 4; ++q)
    *(PE_GLOBAL f32x4*)(gview_w(dst) + 4 * q) = (f32x4){v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
}
__device__ __forceinline__ void store16(uint16_t* dst, const float (&v)[16]) {
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    u32x4 w;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      w[e] = pack2_bf16(v[8 * q + 2 * e], v[8 * q + 2 * e + 1]);
    *(PE_GLOBAL u32x4*)(gview_w(dst) + 8 * q) = w;
  }
}

// ------------------------------------------------------------ operand ring
// 16-byte chunk c of a stage row r sits at chunk small_swz(r, c).  A fragment
// read (16 rows, chunk lane / 16) is served a quarter wave at a time, rows 0-3
// and 12-15 of one chunk beside rows 4-11 of the next; both orders (rows of 128
// and of 64 bytes) put them on distinct banks.
template <int BK>
__device__ __forceinline__ int small_swz(int r, int c) {
  if constexpr (BK == 64) return dl_swz(r, c);
  const int b0 = (r >> 2) & 1, b1 = (r >> 3) & 1;
  return c ^ (((b0 ^ b1) << 1) | b1);
}

// X read with its k rows (update): 16-byte chunk c of stage row r sits at chunk
// c ^ xr_swz(r); the four rows of a 16-lane transposing read, and the four
// 16-lane groups (8 rows apart), then fall on distinct banks.
template <int BT>
__device__ __forceinline__ int small_xr_swz(int r) {
  return BT == 64 ? (((r >> 1) & 1) | (((r >> 3) & 1) << 1)) << 1 : ((r & 3) | (((r >> 3) & 1) << 2)) << 1;
}

// Operands of a product: rows of BK k from row stride ld (Q with ldQ, or, with
// XR, BK rows of X, BT columns, row stride ldQ); the second plane of each lies
// plP / plQ elements behind the first.
struct Operands {
  const PE_GLOBAL uint16_t *P, *Q;
  int64_t ld, ldQ;
  size_t plP, plQ;
};

// Loads of one stage by one wave (stage layout: P's planes, then Q's).  The
// 1-KB blocks of a group's waves alternate, so that a lane's offset, swizzle
// included, is the same for all of a wave's blocks or (one-wave groups) for
// every other one.
template <typename C, bool XR>
__device__ __forceinline__ void small_issue(const Operands& o, int kofs, char* slot, int lw, int lane) {
  constexpr int BT = C::BT, WPG = C::WPG;
#pragma unroll
  for (int op = 0; op < 2; ++op) {
#pragma unroll
    for (int j = 0; j < C::LPW; ++j) {
      const int blk = j * WPG + lw, like = (WPG == 1 ? j & 1 : 0) * WPG + lw;  // like: a block of the same swizzle
      const PE_GLOBAL char* g;
      if (op == 1 && XR) {
        constexpr int CPR = BT / 8, RPB = 64 / CPR;   // 16-byte chunks per stage row, rows per block
        const int lc = (lane % CPR) ^ small_xr_swz<BT>(like * RPB + lane / CPR);
        g = (const PE_GLOBAL char*)(o.Q + (size_t)(kofs + blk * RPB) * o.ldQ) + (uint32_t)((lane / CPR) * (int)o.ldQ * 2 + lc * 16);
      } else {
        constexpr int CPR = C::BK / 8, RPB = 64 / CPR;
        const int64_t ld = op ? o.ldQ : o.ld;
        const int lc = small_swz<C::BK>(like * RPB + lane / CPR, lane % CPR);
        g = (const PE_GLOBAL char*)((op ? o.Q : o.P) + (size_t)(blk * RPB) * ld + kofs) + (uint32_t)((lane / CPR) * (int)ld * 2 + lc * 16);
      }
#pragma unroll
      for (int pl = 0; pl < C::PL; ++pl)
        __builtin_amdgcn_global_load_lds(
            (const void*)(g + 2 * pl * (op ? o.plQ : o.plP)),
            (__attribute__((address_space(3))) void*)(slot + (op * C::PL + pl) * C::OPB + blk * 1024), 16, 0, 0);
    }
  }
}

template <int BT>
__device__ __forceinline__ u32x2 small_xr_read(const char* sB, int r, int nn) {
  const char* p = sB + r * (BT * 2) + (((nn >> 3) ^ small_xr_swz<BT>(r)) << 4) + (nn & 4) * 2;
  return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                       (__attribute__((address_space(3))) i16x4*)(p)));
}

// Fragments of one 32-deep k-step (`ks` of the stage) for a wave's 64 x 64
// accumulators (rows row0.., columns col0.. of the tile).
template <int PL>
struct SmallFrags {
  u32x4 a[PL][4], b[PL][4];
};
template <typename C, bool XR>
__device__ __forceinline__ void small_read(const char* st, int ks, int row0, int col0, int lane, SmallFrags<C::PL>& f) {
  constexpr int BT = C::BT, OPB = C::OPB, PL = C::PL, ROWB = 2 * C::BK;
  const int lc = 4 * ks + (lane >> 4);
#pragma unroll
  for (int pl = 0; pl < PL; ++pl) {
    const char* sA = st + pl * OPB;
    const char* sB = st + (PL + pl) * OPB;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int ra = row0 + q * 16 + (lane & 15);
      f.a[pl][q] = *(const u32x4*)(sA + ra * ROWB + small_swz<C::BK>(ra, lc) * 16);
      if constexpr (XR) {
        const int r = 8 * lc + ((lane & 15) >> 2);
        const int nn = col0 + q * 16 + 4 * (lane & 3);
        const u32x2 lo = small_xr_read<BT>(sB, r, nn), hi = small_xr_read<BT>(sB, r + 4, nn);
        f.b[pl][q] = (u32x4){lo[0], lo[1], hi[0], hi[1]};
      } else {
        const int rb = col0 + q * 16 + (lane & 15);
        f.b[pl][q] = *(const u32x4*)(sB + rb * ROWB + small_swz<C::BK>(rb, lc) * 16);
      }
    }
  }
}

// The operands enter the MFMA in exchanged order, so a lane holds four
// consecutive columns of one row: acc[fm][fn][r] is element (16 fm + lane % 16,
// 16 fn + 4 (lane / 16) + r).
template <typename C>
__device__ __forceinline__ void small_mfma(const SmallFrags<C::PL>& f, f32x4 (&acc)[4][4]) {
  if constexpr (C::PL == 1) {
#pragma unroll
    for (int fm = 0; fm < 4; ++fm)
#pragma unroll
      for (int fn = 0; fn < 4; ++fn)
        acc[fm][fn] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f.b[0][fn]),
                                                              __builtin_bit_cast(bf16x8, f.a[0][fm]), acc[fm][fn], 0, 0, 0);
  } else {
    // (lo, lo) on the 64 tile, whose launches are bound by latency; (hi, lo),
    // (lo, hi), (hi, hi)
    constexpr int pa[4] = {1, 1, 0, 0}, pb[4] = {1, 0, 1, 0};
#pragma unroll
    for (int q = C::BT == 64 ? 0 : 1; q < 4; ++q)
#pragma unroll
      for (int fm = 0; fm < 4; ++fm)
#pragma unroll
        for (int fn = 0; fn < 4; ++fn)
          acc[fm][fn] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, f.b[pb[q]][fn]),
                                                               __builtin_bit_cast(f16x8, f.a[pa[q]][fm]), acc[fm][fn], 0, 0, 0);
  }
}

// wait until at most n stages of loads (n < NS) are outstanding in this wave
template <int LPS, int NS>
__device__ __forceinline__ void wait_stages(int n) {
  if constexpr (NS > 1) {
    if (n >= NS - 1) wait_vmcnt<(NS - 1) * LPS>();
    else wait_stages<LPS, NS - 1>(n);
  } else {
    wait_vmcnt<0>();
  }
}

// The tile's product over k in [k0, k1) (multiples of 64) into the staged LDS
// tile, one partial tile per group, C::REGION bytes apart.  P2 (k0 = 0): the
// product of P + P2, both of k1 columns.  (__restrict__: the
// alias scopes it leaves on the direct-to-LDS loads keep the compiler from
// waiting for all of them before every transposing LDS read.)  `inputs` loads
// what the epilogue reads; it runs once the first stages are on their way, so
// that all of a tile's first loads share one round trip.
template <typename C, bool XR, bool TWO = false, typename F>
__device__ __forceinline__ void small_product(const uint16_t* __restrict__ P, const uint16_t* __restrict__ Q, int64_t ld,
                                              int64_t ldQ, size_t plP, size_t plQ, int rp0, int rq0, int k0, int k1,
                                              char* smem, F&& inputs, const uint16_t* __restrict__ P2 = nullptr) {
  constexpr int BT = C::BT, NS = C::NS, KW = C::KW;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int group = wave / C::WPG, lw = wave % C::WPG;
  const Operands o = {gview(P) + (size_t)rp0 * ld, XR ? gview(Q) + rq0 : gview(Q) + (size_t)rq0 * ldQ,
                      ld, ldQ, plP, plQ};
  const int nk = (k1 - k0) / C::BK * (TWO ? 2 : 1);
  f32x4 acc[4][4];
#pragma unroll
  for (int fm = 0; fm < 4; ++fm)
#pragma unroll
    for (int fn = 0; fn < 4; ++fn) acc[fm][fn] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  // this group's stages: group, group + KW, ...; groups of several waves meet
  // at the block's barrier, so all run the longest group's count
  const int n = (nk - group + KW - 1) / KW, rounds = C::WPG > 1 ? (nk + KW - 1) / KW : n;
  char* ring = smem + group * C::REGION;
  auto issue = [&](int i, char* slot) {
    const int kofs = k0 + (group + KW * i) * C::BK;
    if (TWO && kofs >= k1) {
      Operands o2 = o;
      o2.P = gview(P2) + (size_t)rp0 * ld;
      small_issue<C, XR>(o2, kofs - k1, slot, lw, lane);
    } else {
      small_issue<C, XR>(o, kofs, slot, lw, lane);
    }
  };
  // a slot is refilled as soon as it has been read: all slots start full
#pragma unroll
  for (int i = 0; i < NS; ++i)
    if (i < n) issue(i, ring + i * C::STB);
  inputs();
  const int row0 = C::WPG > 1 ? (lw >> 1) * 64 : 0, col0 = C::WPG > 1 ? (lw & 1) * 64 : 0;
  for (int i = 0; i < rounds; ++i) {
    char* slot = ring + (i % NS) * C::STB;
    // own loads of stage i landed (the NS - 1 stages after it may be pending);
    // after the barrier the group's have
    wait_stages<C::LPS, NS>(n - 1 - i);
    if constexpr (C::WPG > 1) lds_barrier();
    asm volatile("" ::: "memory");
    SmallFrags<C::PL> f;
    if (C::WPG == 1 || i < n) {
#pragma unroll
      for (int ks = 0; ks < C::BK / 32; ++ks) {
        if (ks > 0) small_mfma<C>(f, acc);
        small_read<C, XR>(slot, ks, row0, col0, lane, f);
      }
    }
    wait_lgkm0();  // the slot's reads have returned, after the barrier everyone's
    if constexpr (C::WPG > 1) lds_barrier();
    asm volatile("" ::: "memory");
    if (i + NS < n) issue(i + NS, slot);
    if (C::WPG == 1 || i < n) small_mfma<C>(f, acc);
  }
  if constexpr (C::WPG > 1) __syncthreads();  // the tile overlays the group's ring
  float* cs = (float*)ring;
#pragma unroll
  for (int fm = 0; fm < 4; ++fm)
#pragma unroll
    for (int fn = 0; fn < 4; ++fn)
      *(f32x4*)(cs + cs_idx<BT>(row0 + fm * 16 + (lane & 15), col0 + fn * 16 + 4 * (lane >> 4))) = acc[fm][fn];
  __syncthreads();
}

// The same for matrices of fewer than 16 rows, whose errors have nothing to
// average out against (a 2 x 2 result of the plane products was 1.8e-5 off):
// fp32 operands, fp64 sums on the vector units.  Symmetric products: P and Q
// rows along k, one thread per element of the leading 16 x 16 block; update
// (XR): Q is X, 16 thread rows of 4 columns each.  A few hundred kFLOP.
template <bool XR>
__device__ __forceinline__ void tiny_product(const float* P, const float* Q, size_t ld, size_t ldQ, int rq0, int k0, int k1,
                                             int s, char* smem) {
  float* cs = (float*)smem;
  float* sp = (float*)(smem + 64 * 68 * 4);   // P's chunk: 16 rows of 132 floats; Q's behind it
  float* sq = sp + 16 * 132;
  const int tid = threadIdx.x, i = tid >> 4, j = tid & 15;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  if constexpr (XR) {
    for (int u = tid; u < 256; u += kThreads) sp[(u >> 4) * 17 + (u & 15)] = (u >> 4) < s && (u & 15) < s ? P[(size_t)(u >> 4) * ld + (u & 15)] : 0.0f;
    __syncthreads();
    for (int k = k0; k < s && k < k1; ++k) {
      const f32x4 x = *(const PE_GLOBAL f32x4*)gview(Q + (size_t)k * ldQ + rq0 + 4 * j);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] += (double)sp[i * 17 + k] * (double)x[e];
    }
  } else {
    for (int kc = k0; kc < k1; kc += 128) {
      const int n = min(128, k1 - kc);
      __syncthreads();  // the previous chunk's readers are done
      for (int u = tid; u < 16 * 128; u += kThreads) {
        const int r = u >> 7, c = u & 127;
        const bool in = r < s && c < n;
        sp[r * 132 + c] = in ? P[(size_t)r * ld + kc + c] : 0.0f;
        sq[r * 132 + c] = in ? Q[(size_t)r * ldQ + kc + c] : 0.0f;
      }
      __syncthreads();
      for (int c = 0; c < 128; c += 4) {
        const f32x4 a = *(const f32x4*)(sp + i * 132 + c), b = *(const f32x4*)(sq + j * 132 + c);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += (double)a[e] * (double)b[e];
      }
    }
  }
  for (int u = tid; u < 64 * 68; u += kThreads) cs[u] = 0.0f;
  __syncthreads();
  if constexpr (XR) *(f32x4*)(cs + cs_idx<64>(i, 4 * j)) = (f32x4){(float)acc[0], (float)acc[1], (float)acc[2], (float)acc[3]};
  else cs[cs_idx<64>(i, j)] = (float)((acc[0] + acc[1]) + (acc[2] + acc[3]));
  __syncthreads();
}

// chunk p of the staged product, partial tiles summed in group order
template <typename C>
__device__ __forceinline__ void small_gather(const char* smem, int p, float (&x)[16]) {
  const int row = C::row(p), col = C::col();
  cs_load<C::BT>((const float*)smem, row, col, x);
#pragma unroll
  for (int w = 1; w < (C::PL == 0 ? 1 : C::KW); ++w) {
    float y[16];
    cs_load<C::BT>((const float*)(smem + w * C::REGION), row, col, y);
#pragma unroll
    for (int e = 0; e < 16; ++e) x[e] += y[e];
  }
}

// The fp32 path's X_0 planes hold G times the power of two below sigma, which
// rounds nothing; the rest of sigma, in [1, 2), goes into the epilogues of the
// launches that read them.
__device__ __forceinline__ float pow2_part(float s) { return __uint_as_float(__float_as_uint(s) & 0x7f800000u); }
__device__ __forceinline__ float x0_rest(float sigma) { return sigma / pow2_part(sigma); }

// 16 values into the fp16 planes of an operand (pl elements apart), scaled
template <int PL>
__device__ __forceinline__ void store16_planes(uint16_t* dst, size_t pl, float q, const float (&v)[16]) {
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    float r[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = v[8 * h + e] * q;
#pragma unroll
    for (int k = 0; k < PL; ++k) {
      u32x4 w;
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = peel2_f16(&r[2 * e], &r[2 * e + 1]);
      *(PE_GLOBAL u32x4*)(gview_w(dst) + k * pl + 8 * h) = w;
    }
  }
}

// an operand's chunk: bf16, or the planes
template <int PL>
__device__ __forceinline__ void store16_operand(uint16_t* dst, size_t pl, float q, const float (&v)[16]) {
  if constexpr (PL == 0) store16((float*)dst, v);
  else if constexpr (PL == 1) store16(dst, v);
  else store16_planes<PL>(dst, pl, q, v);
}

// Operand copy of A.  On the fp32 path it lives in the copy of X that the
// step's update will write: between the Gram product and the update that one
// holds nothing, and L >= s.
template <int PL>
__device__ __forceinline__ uint16_t* a_operand(const KArgs& args, CDesc& d) {
  return PL > 1 ? xb_next(args, d) : (uint16_t*)d.As;
}

// ------------------------------------------------------------- epilogues
// Symmetric products: KIND_GRAM stores A (and its mirror), KIND_A2 stores
// B - beta I (or, on the learned path's first step, A^2 and its moments).
// x: the product's chunks; ar: A at the same positions (KIND_A2).  cs: the
// staged tile (for the mirror); red: kSmallTail bytes.
template <typename C, int KIND>
__device__ __forceinline__ void small_epi_syrk(const KArgs& args, CDesc& d, int ti, int tj, float sigma, float beta, float b, float c,
                                               float (&x)[C::NCH][16], const float (&ar)[C::NCH][16],
                                               float* cs, float* red) {
  constexpr int BT = C::BT;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const size_t sp = d.sp;
  float alpha = C::PL > 1 ? args.deq : 1.0f;
  if (KIND == KIND_GRAM && args.t == 0) {
    const float sg = C::PL > 1 ? x0_rest(sigma) : sigma;
    alpha *= sg * sg;
  }
  const bool raw = KIND == KIND_A2 && args.raw_a2;
  uint16_t* dst = KIND == KIND_GRAM ? a_operand<C::PL>(args, d) : (uint16_t*)d.Bs;
  const float q = C::PL > 1 && KIND == KIND_A2 && args.init_step ? d.scal[kScInitQ] : args.oscale;
  constexpr int ES = C::PL == 0 ? 2 : 1;                    // operand elements per uint16_t step
  const bool operand = !raw && !(C::PL == 0 && KIND == KIND_GRAM);  // (fp32 A serves as its own operand)
  float* dstf = KIND == KIND_GRAM ? (C::PL != 1 || args.init_step ? d.Af : nullptr) : (raw ? d.A2f : nullptr);
  // A^2's epilogue reads the FP32 A on the upper tiles only; the power method and
  // the learned path's combine read all of it (2048 x 2048, FP32: 864 -> 849 us per call)
  const bool mirrorf = KIND != KIND_GRAM || args.init_step || args.sel_coef;
  float part[4] = {0.0f, 0.0f, 0.0f, 0.0f};  // Gram: tr A, ||A||^2; raw A^2: moments 1..4
#pragma unroll
  for (int p = 0; p < C::NCH; ++p) {
    const int row = C::row(p), col = C::col();
    const int i = ti * BT + row, j = tj * BT + col;
    const int dd = ti == tj ? row - col : -1;  // chunk element on the diagonal (outside 0..15: none)
    const float bd = i < d.s ? beta : 0.0f;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      float v = x[p][e];
      if (KIND == KIND_GRAM || C::PL > 1) v *= alpha;
      if (KIND == KIND_GRAM) {
        part[1] = __builtin_fmaf(v, v, part[1]);
      } else if (raw) {
        const float av = ar[p][e];
        part[0] += dd == e ? av : 0.0f;
        part[1] = __builtin_fmaf(av, av, part[1]);
        part[2] = __builtin_fmaf(av, v, part[2]);
        part[3] = __builtin_fmaf(v, v, part[3]);
      } else {
        // same operation order as the learned path's combine kernel
        v = __builtin_fmaf(c, v, b * ar[p][e]);
        v -= dd == e ? bd : 0.0f;
      }
      x[p][e] = v;
    }
    if (KIND == KIND_GRAM && ti == tj) {
      // the init step's F^2 = tr A takes the FP32 diagonal, the others what is stored
#pragma unroll
      for (int e = 0; e < 16; ++e)
        part[0] += dd == e ? (C::PL != 1 || args.init_step ? x[p][e] : bf2f(f2bf(x[p][e]))) : 0.0f;
    }
    const size_t o = (size_t)i * sp + j;
    if (operand) store16_operand<C::PL>(dst + ES * o, sp * sp, q, x[p]);
    if (dstf) store16(dstf + o, x[p]);
    if (ti != tj) cs_store<BT>(cs, row, col, x[p]);
  }
  if (ti != tj) {
    __syncthreads();
#pragma unroll
    for (int p = 0; p < C::NCH; ++p) {
      const int row = C::row(p), col = C::col();
      float v[16];
      cs_load_t<BT>(cs, col, row, v);
      const size_t o = (size_t)(tj * BT + row) * sp + ti * BT + col;
      if (operand) store16_operand<C::PL>(dst + ES * o, sp * sp, q, v);
      if (dstf && mirrorf) store16(dstf + o, v);
    }
  }
  if (KIND == KIND_GRAM || raw) {
    // the tile's partials, summed in a fixed order (an off-diagonal tile also
    // stands for its mirror: weight 2 except on the traces)
    constexpr int NP = KIND == KIND_GRAM ? 2 : 4;
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      for (int off = 32; off > 0; off >>= 1) part[k] += __shfl_xor(part[k], off);
      if (lane == 0) red[k * C::NW + wave] = part[k];
    }
    __syncthreads();
    if (threadIdx.x < NP) {
      const int k = threadIdx.x;
      float t = 0.0f;
#pragma unroll
      for (int q = 0; q < C::NW; ++q) t += red[k * C::NW + q];
      const float w = (k == 0 || ti == tj) ? t : 2.0f * t;
      const int tile = tri_index(ti, tj, d.nbs);
      if (KIND == KIND_GRAM) d.trp[2 * tile + k] = w;
      else d.mom[(size_t)tile * 4 + k] = w;
    }
  }
}

// 16 values of a row of the caller's output (row gr, columns gc..) and the Muon
// weight step W <- (1 - lr wd) W - lr X_T on the same positions (the last tiles of
// a 256-tile update: from the bf16 X where X leaves as bf16, like its other tiles);
// 16-byte accesses where the row allows them
__device__ __forceinline__ void store_result(const KArgs& args, CDesc& d, int gr, int gc, int rows, int cols,
                                             const float (&v)[16]) {
  if (gr >= rows || gc >= cols) return;
  const bool whole = gc + 16 <= cols;
  if (d.Out) {
    const size_t o = (size_t)gr * d.ldo + gc;
    if (d.out_bf16) {
      uint16_t* q = (uint16_t*)d.Out + o;
      if (whole && d.o_vec) store16(q, v);
      else
#pragma unroll
        for (int e = 0; e < 16; ++e)
          if (gc + e < cols) gview_w(q)[e] = f2bf(v[e]);
    } else {
      float* q = (float*)d.Out + o;
      if (whole && ((uintptr_t)d.Out % 16 == 0) && d.ldo % 4 == 0) store16(q, v);
      else
#pragma unroll
        for (int e = 0; e < 16; ++e)
          if (gc + e < cols) gview_w(q)[e] = v[e];
    }
  }
  if (d.W) {
    const float keep = 1.0f - args.mlr * args.mwd;
    const bool rounded = args.tail >= 0 && d.Out && d.out_bf16;
    const size_t o = (size_t)gr * d.ldw + gc;
    const bool vec = whole && ((uintptr_t)d.W % 16 == 0) && d.ldw % (d.w_bf16 ? 8 : 4) == 0;
    float w[16];
    if (vec) {
      if (d.w_bf16) load16((const uint16_t*)d.W + o, w);
      else load16((const float*)d.W + o, w);
    } else {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        w[e] = 0.0f;
        if (gc + e < cols) w[e] = d.w_bf16 ? bf2f(gview((const uint16_t*)d.W)[o + e]) : gview((const float*)d.W)[o + e];
      }
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) w[e] = __builtin_fmaf(-args.mlr, rounded ? bf2f(f2bf(v[e])) : v[e], keep * w[e]);
    if (vec) {
      if (d.w_bf16) store16((uint16_t*)d.W + o, w);
      else store16((float*)d.W + o, w);
    } else {
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if (gc + e < cols) {
          if (d.w_bf16) gview_w((uint16_t*)d.W)[o + e] = f2bf(w[e]);
          else gview_w((float*)d.W)[o + e] = w[e];
        }
    }
  }
}

// Planes of a fast-iteration buffer.  P lives only between a segment's Gram
// matrix and its update, while the other copy of X (L >= s: at least as large)
// holds nothing.
__device__ __forceinline__ uint16_t* fb_planes(const KArgs& args, CDesc& d, int k) {
  return k == kFbP ? xb_next(args, d) : d.fbp[k];
}

// A at a chunk: its bf16 copy, or FP32
template <int PL>
__device__ __forceinline__ void load_a(CDesc& d, size_t o, float (&v)[16]) {
  if constexpr (PL == 1) load16((const uint16_t*)d.As + o, v);
  else load16(d.Af + o, v);
}

// -------------------------------------------------------------- kernels
template <int KIND, typename C>
__global__ __launch_bounds__((C::NT), (C::LDS + kSmallTail <= 80 * 1024 ? 2 : 1)) void small_gemm_kernel(KArgs args) {
  constexpr int BT = C::BT;
  constexpr bool UPD = KIND == KIND_UPD || KIND == KIND_UPD_LAST || KIND == KIND_UPD0 || KIND == KIND_UPDI;
  __shared__ __attribute__((aligned(16))) char smem[C::LDS + kSmallTail];
  float* cs = (float*)smem;
  float* red = (float*)(smem + C::LDS);
  for (int slot = blockIdx.x; slot < args.total; slot += gridDim.x) {
    constexpr int PER = 256 / BT;  // tiles of a 256 tile (an update's last tiles): PER x PER
    int item = xcd_item(slot, args.total), part = 0;
    if (UPD && C::PL == 1 && args.tail >= 0) {
      part = item % (PER * PER);
      item = args.tail + item / (PER * PER);
    }
    const int pos = find_mat(args.offs, args.count, item);
    CDesc& d = const_desc(args, args.ord ? const_i32(args.ord, pos) : pos);
    if (skip_matrix(args, d)) continue;
    const bool past = past_schedule(args, d);
    if (past && KIND != KIND_UPD_LAST) continue;
    const int local = item - const_i32(args.offs, pos);
    const size_t sp = d.sp, Lp = d.Lp;
    if (slot != (int)blockIdx.x) __syncthreads();  // the previous tile's readers are done
    if constexpr (UPD) {
      int tm, tn;
      banded_decode(local, d.nb, d.nbL, &tm, &tn);
      if (C::PL == 1 && args.tail >= 0) {
        tm = PER * tm + part / PER;
        tn = PER * tn + part % PER;
      }
      // the tile of X_t in FP32 and the step's scalars
      float xr[C::NCH][16];
      float a, b, c, alpha = 1.0f, palpha = 1.0f;
      auto inputs = [&]() {
#pragma unroll
        for (int p = 0; p < C::NCH; ++p) {
          const size_t o = (size_t)(tm * BT + C::row(p)) * Lp + tn * BT + C::col();
          if (KIND == KIND_UPD0 || (KIND == KIND_UPDI && args.x0b)) load16(xb_cur(args, d) + o, xr[p]);
          else if constexpr (C::PL == 1) load16_halves(xb_at(d, past ? schedule_steps(args, d) : args.t) + o, d.Xl + o, xr[p]);
          else load16(d.Xf + o, xr[p]);
        }
        step_coef(args, d, &a, &b, &c);
        if (!args.fast && !past) a += d.scal[kScBeta];
        const float sigma = args.t == 0 ? matrix_sigma(args, d) : 1.0f;
        alpha = sigma;
        // fp32 path: the product is of scaled planes, X_0 itself is not scaled yet
        if constexpr (C::PL > 1) {
          a *= alpha;
          palpha = args.init_step ? args.deq / d.scal[kScInitQ] : args.deq;
          if (args.t == 0) palpha *= x0_rest(sigma);
          alpha = 1.0f;
        }
      };
      const uint16_t* Bop = (const uint16_t*)d.Bs;
      if (C::PL > 1 && args.fast) Bop = fb_planes(args, d, args.fp_);
      // a matrix past its schedule: no product, X is copied (a = 1)
      if constexpr (C::PL == 0) {
        inputs();
        tiny_product<true>(args.fast ? d.fb[args.fp_] : (const float*)d.Bs, d.Xf, sp, Lp, tn * BT, 0, past ? 0 : d.sp, d.s, smem);
      } else {
        small_product<C, true, KIND == KIND_UPDI>(Bop, xb_cur(args, d), sp, Lp, sp * sp, sp * Lp, tm * BT, tn * BT, 0,
                                                  past ? 0 : d.sp, smem, inputs, (const uint16_t*)d.As);
      }
      float amax = 0.0f;
#pragma unroll
      for (int p = 0; p < C::NCH; ++p) {
        const int row = C::row(p), col = C::col();
        float x[16];
        small_gather<C>(smem, p, x);
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          x[e] = C::PL > 1 ? __builtin_fmaf(a, xr[p][e], palpha * x[e]) : alpha * (a * xr[p][e] + x[e]);
          amax = fmaxf(amax, fabsf(x[e]));
        }
        if constexpr (KIND == KIND_UPD_LAST) {
          if (d.trans) cs_store<BT>(cs, row, col, x);
          else store_result(args, d, tm * BT + row, tn * BT + col, d.s, d.L, x);
        } else {
          const size_t o = (size_t)(tm * BT + row) * Lp + tn * BT + col;
          if constexpr (C::PL == 1) {
            store16_halves(xb_next(args, d) + o, d.Xl + o, x);
          } else {
            store16(d.Xf + o, x);
            if constexpr (C::PL > 1) store16_planes<C::PL>(xb_next(args, d) + o, sp * Lp, args.oscale, x);
          }
        }
      }
      if constexpr (KIND == KIND_UPD_LAST) {
        if (d.trans) {
          __syncthreads();
#pragma unroll
          for (int p = 0; p < C::NCH; ++p) {
            const int row = C::row(p), col = C::col();
            float v[16];
            cs_load_t<BT>(cs, col, row, v);
            store_result(args, d, tn * BT + row, tm * BT + col, d.L, d.s, v);
          }
        }
      } else if (args.fp8_next) {
        wave_amax_atomic(amax, d.scal + kScAmaxX + args.t + 1);
      }
    } else {
      const int split = KIND == KIND_GRAM ? d.gram_split : d.a2_split;
      const int tile = local / split, ksp = local % split;
      int ti, tj;
      tri_decode_banded(tile, d.nbs, &ti, &tj);
      const uint16_t* Op = KIND == KIND_GRAM ? xb_cur(args, d) : a_operand<C::PL>(args, d);
      const int K = KIND == KIND_GRAM ? d.Lp : d.sp;
      int k0, k1;
      split_range(K, split, ksp, 64, &k0, &k1);
      // a degree-3 step (c = 0 in the fixed schedule) needs no A^2: the
      // epilogue forms B = b A - beta I from an empty product
      if (KIND == KIND_A2 && !args.sel_coef && args.c == 0.0f) k1 = k0;
      float ar[C::NCH][16], x[C::NCH][16];
      float a = 0.0f, b = 0.0f, c = 0.0f, beta = 0.0f, sigma = 1.0f;
      auto inputs = [&]() {
        if (KIND == KIND_GRAM && args.t == 0 && split == 1) sigma = matrix_sigma(args, d);
        if (KIND == KIND_A2 && split == 1) {
#pragma unroll
          for (int p = 0; p < C::NCH; ++p)
            load_a<C::PL>(d, (size_t)(ti * BT + C::row(p)) * sp + tj * BT + C::col(), ar[p]);
          if (!args.raw_a2) {
            step_coef(args, d, &a, &b, &c);
            beta = shift_beta(d, b, c);
            if (tile == 0 && threadIdx.x == 0) d.scal[kScBeta] = beta;
          }
        }
      };
      const size_t pl = sp * (size_t)K;
      if constexpr (C::PL == 0) {
        inputs();
        const float* F = KIND == KIND_GRAM ? d.Xf : d.Af;
        tiny_product<false>(F, F, K, K, 0, k0, k1, d.s, smem);
      } else {
        small_product<C, false>(Op, Op, K, K, pl, pl, ti * BT, tj * BT, k0, k1, smem, inputs);
      }
#pragma unroll
      for (int p = 0; p < C::NCH; ++p) small_gather<C>(smem, p, x[p]);
      if (split == 1) {
        small_epi_syrk<C, KIND>(args, d, ti, tj, sigma, beta, b, c, x, ar, cs, red);
      } else {
        // partial tiles, row-major
        float* part = d.part + (size_t)(tile * split + ksp) * BT * BT;
#pragma unroll
        for (int p = 0; p < C::NCH; ++p) store16(part + C::row(p) * BT + C::col(), x[p]);
      }
    }
  }
}

// Sums the split-K partial tiles in split order and runs the same epilogue.
template <int KIND, int BT, int PL>
__global__ __launch_bounds__(kThreads) void small_reduce_kernel(KArgs args) {
  typedef SmallTile<BT, BT == 64 ? 4 : 1, 2, PL> C;  // 256 threads
  __shared__ __attribute__((aligned(16))) char smem[C::CB + kSmallTail];
  for (int item = blockIdx.x; item < args.total; item += gridDim.x) {
    const int mi = find_mat(args.offs, args.count, item);
    CDesc& d = const_desc(args, mi);
    if (skip_matrix(args, d) || past_schedule(args, d)) continue;
    const int tile = item - const_i32(args.offs, mi);
    const int split = KIND == KIND_GRAM ? d.gram_split : d.a2_split;
    int ti, tj;
    tri_decode_banded(tile, d.nbs, &ti, &tj);
    if (item != (int)blockIdx.x) __syncthreads();  // the previous tile's readers are done
    float ar[C::NCH][16], x[C::NCH][16];
    float a = 0.0f, b = 0.0f, c = 0.0f, beta = 0.0f;
    const float sigma = KIND == KIND_GRAM && args.t == 0 ? matrix_sigma(args, d) : 1.0f;
    if (KIND == KIND_A2) {
#pragma unroll
      for (int p = 0; p < C::NCH; ++p)
        load_a<C::PL>(d, (size_t)(ti * BT + C::row(p)) * d.sp + tj * BT + C::col(), ar[p]);
      if (!args.raw_a2) {
        step_coef(args, d, &a, &b, &c);
        beta = shift_beta(d, b, c);
        if (tile == 0 && threadIdx.x == 0) d.scal[kScBeta] = beta;
      }
    }
    const float* part = d.part + (size_t)tile * split * BT * BT;
#pragma unroll
    for (int p = 0; p < C::NCH; ++p) {
#pragma unroll
      for (int e = 0; e < 16; ++e) x[p][e] = 0.0f;
      for (int k = 0; k < split; ++k) {
        float y[16];
        load16(part + (size_t)k * BT * BT + C::row(p) * BT + C::col(), y);
#pragma unroll
        for (int e = 0; e < 16; ++e) x[p][e] = k == 0 ? y[e] : x[p][e] + y[e];
      }
    }
    small_epi_syrk<C, KIND>(args, d, ti, tj, sigma, beta, b, c, x, ar, (float*)smem, (float*)(smem + C::CB));
  }
}

// ------------------------------------------------ fast rectangular iteration
// Appendix G, Algorithm 4, restarted every k steps, on the fp32 path's operand
// planes.  Within a segment the library carries Q_t = (prod a) I + D_t and
// R_t = Y Q_{t-1}^2 as polynomials in the segment's Gram matrix Y (all
// symmetric and commuting), so every product is a symmetric s x s product
// computed on upper-triangle tiles and mirrored:
//   B_t = b R_t + c R_t^2                       (SYRK of R_t)
//   D_t = a_t D_{t-1} + q_{t-1} B_t + D_{t-1} B_t   (D_1 = B_1, q_t = prod a)
//   P   = R_t B_t,  R_{t+1} = a_t^2 R_t + 2 a_t P + P B_t   (= R_t h_t(R_t)^2)
// and the segment ends with X <- q X + D X (the update kernel with a = q and
// D as its B operand).  KIND_GRAM: Y = X X^T; KIND_A2: a symmetric product
// fb[fp_] fb[fq_].  One epilogue serves every product:
//   out = cacc * acc + c1 * E1 + c2 * E2 + cdiag * I   (cdiag on the real rows)
// stored in FP32 and as planes.  E1 and E2 are read by the block that writes
// the same tile, so R and D, whose old values are E1, are replaced in place;
// D's planes are an operand of its own product and alternate, R's are not.
// The FP32 values below the diagonal tiles are never read and not stored (s =
// 4096: 32 MB of the 128 a product stores; a call's products all split their
// tiles alike, quarters included).
template <int KIND, typename C>
__global__ __launch_bounds__((C::NT), (C::LDS + kSmallTail <= 80 * 1024 ? 2 : 1)) void small_fast_kernel(KArgs args) {
  constexpr int BT = C::BT;
  __shared__ __attribute__((aligned(16))) char smem[C::LDS + kSmallTail];
  float* cs = (float*)smem;
  for (int slot = blockIdx.x; slot < args.total; slot += gridDim.x) {
    int item = xcd_item(slot, args.total), quarter = 0;
    if (BT == 64 && args.tail >= 0) {
      quarter = item & 3;
      item = args.tail + (item >> 2);
    }
    const int pos = find_mat(args.offs, args.count, item);
    CDesc& d = const_desc(args, pos);
    int ti, tj;
    tri_decode_banded(item - const_i32(args.offs, pos), d.nbs, &ti, &tj);
    if (BT == 64 && args.tail >= 0) {
      ti = 2 * ti + (quarter >> 1);
      tj = 2 * tj + (quarter & 1);
      if (ti > tj) continue;  // the lower quarter of a diagonal tile is a mirror
    }
    const size_t sp = d.sp, Lp = d.Lp;
    if (slot != (int)blockIdx.x) __syncthreads();  // the previous tile's readers are done
    const float* E1 = args.fe1 >= 0 ? d.fb[args.fe1] : nullptr;
    const float* E2 = args.fe2 >= 0 ? d.fb[args.fe2] : nullptr;
    if constexpr (C::PL == 0) {
      const float *F = KIND == KIND_GRAM ? d.Xf : d.fb[args.fp_], *H = KIND == KIND_GRAM ? d.Xf : d.fb[args.fq_];
      const int K = KIND == KIND_GRAM ? d.Lp : d.sp;
      tiny_product<false>(F, H, K, K, 0, 0, K, d.s, smem);
    } else if constexpr (KIND == KIND_GRAM) {
      const uint16_t* X = xb_cur(args, d);
      small_product<C, false>(X, X, Lp, Lp, sp * Lp, sp * Lp, ti * BT, tj * BT, 0, d.Lp, smem, []() {});
    } else {
      small_product<C, false>(fb_planes(args, d, args.fp_), fb_planes(args, d, args.fq_), sp, sp, sp * sp, sp * sp, ti * BT, tj * BT,
                              0, d.sp, smem, []() {});
    }
    float* out = d.fb[args.fout];
    uint16_t* outp = fb_planes(args, d, args.fout);
    float ca = args.cacc * args.deq;
    if (KIND == KIND_GRAM && args.t == 0) {
      const float sigma = matrix_sigma(args, d), sg = C::PL > 1 ? x0_rest(sigma) : sigma;
      ca *= sg * sg;
    }
#pragma unroll
    for (int p = 0; p < C::NCH; ++p) {
      const int row = C::row(p), col = C::col(), i = ti * BT + row;
      const size_t o = (size_t)i * sp + tj * BT + col;
      float x[16], e1[16], e2[16];
      if (E1) load16(E1 + o, e1);
      if (E2) load16(E2 + o, e2);
      small_gather<C>(smem, p, x);
      const int dd = ti == tj ? row - col : -1;
      const float cd = i < d.s ? args.cdiag : 0.0f;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        float v = ca * x[e];
        if (E1) v = __builtin_fmaf(args.c1, e1[e], v);
        if (E2) v = __builtin_fmaf(args.c2, e2[e], v);
        x[e] = v + (dd == e ? cd : 0.0f);
      }
      store16(out + o, x);
      store16_planes<C::PL>(outp + o, sp * sp, args.oscale, x);
      if (ti != tj) cs_store<BT>(cs, row, col, x);
    }
    if (ti != tj) {
      __syncthreads();
#pragma unroll
      for (int p = 0; p < C::NCH; ++p) {
        const int row = C::row(p), col = C::col();
        float v[16];
        cs_load_t<BT>(cs, col, row, v);
        const size_t o = (size_t)(tj * BT + row) * sp + ti * BT + col;
        store16_planes<C::PL>(outp + o, sp * sp, args.oscale, v);
      }
    }
  }
}

// Planes of X_0 on the fp32 path, once the norm is known, from the unscaled
// FP32 copy.  One item is 16384 elements.
__global__ __launch_bounds__(kThreads) void planes_kernel(KArgs args) {
  for (int item = blockIdx.x; item < args.total; item += gridDim.x) {
    const int mi = find_mat(args.offs, args.count, item);
    CDesc& d = const_desc(args, mi);
    if (skip_matrix(args, d)) continue;
    const size_t n = (size_t)d.sp * d.Lp, base = (size_t)(item - const_i32(args.offs, mi)) * 16384;
    const float q = pow2_part(matrix_sigma(args, d)) * args.oscale;
    float v[4][16];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const size_t o = base + (size_t)(k * kThreads + threadIdx.x) * 16;
      if (o < n) load16(d.Xf + o, v[k]);
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const size_t o = base + (size_t)(k * kThreads + threadIdx.x) * 16;
      if (o < n) store16_planes<2>((uint16_t*)d.Xb + o, n, q, v[k]);
    }
  }
}

// ------------------------------------------------------------- launchers
// Ring depth: the deep rings (up to 135 KB, one block per CU) when the launch
// has no more tiles than the device has CUs, so that each tile's loads are in
// flight together; the shallow ones with two blocks per CU otherwise, where
// one block's loads and epilogue run beside the other's products.  Stages are
// 64 deep but for the deep ring of the fp32 path's 64 tile, where two stages of
// 32 fit in the place of one of 64 and a short K feeds twice the waves (64 x 64:
// 86 us per call against 101, 768 x 768 226 against 239).  The deep rings of the
// 128 tile belong to two groups of waves that share out k, another order of the
// sums: not where results may not depend on the call (KArgs::alike).
template <int KIND, typename C>
static void launch_small_c(const KArgs& a, int cap, hipStream_t st) {
  hipLaunchKernelGGL((small_gemm_kernel<KIND, C>), dim3(a.total < cap ? a.total : cap), dim3(C::NT), 0, st, a);
}
template <int KIND>
static void launch_small_k(int prec, int bt, const KArgs& a, hipStream_t st) {
  const bool deep = a.total <= 256 && (bt == kTileTiny || !a.alike);
  if (prec == kTiny) {
    if constexpr (KIND != KIND_UPD0 && KIND != KIND_UPDI) launch_small_c<KIND, SmallTile<64, 4, 1, 0>>(a, 256, st);
  } else if (prec == kF32) {
    if constexpr (KIND != KIND_UPD0 && KIND != KIND_UPDI) {
      if (bt == kTileTiny) {
        if (deep) launch_small_c<KIND, SmallTile<64, 4, 2, 2, 32>>(a, 256, st);
        else launch_small_c<KIND, SmallTile<64, 4, 1, 2, 32>>(a, 512, st);
      } else {
        if (deep) launch_small_c<KIND, SmallTile<128, 2, 1, 2>>(a, 256, st);
        else launch_small_c<KIND, SmallTile<128, 1, 1, 2>>(a, 512, st);
      }
    }
  } else if (bt == kTileTiny) {
    if (deep) launch_small_c<KIND, SmallTile<64, 4, 2>>(a, 256, st);
    else launch_small_c<KIND, SmallTile<64, 4, 1>>(a, 512, st);
  } else {
    if (deep) launch_small_c<KIND, SmallTile<128, 2, 2>>(a, 256, st);
    else launch_small_c<KIND, SmallTile<128, 1, 2>>(a, 512, st);
  }
}

hipError_t launch_small_gemm(int prec, int bt, int kind, const KArgs& a, hipStream_t st) {
  if (a.total <= 0) return hipSuccess;
  if (kind == KIND_GRAM) launch_small_k<KIND_GRAM>(prec, bt, a, st);
  else if (kind == KIND_A2) launch_small_k<KIND_A2>(prec, bt, a, st);
  else if (a.last) launch_small_k<KIND_UPD_LAST>(prec, bt, a, st);
  else if (a.init_step && prec == kBF16) launch_small_k<KIND_UPDI>(prec, bt, a, st);
  else if (a.x0b && prec == kBF16) launch_small_k<KIND_UPD0>(prec, bt, a, st);
  else launch_small_k<KIND_UPD>(prec, bt, a, st);
  return hipGetLastError();
}

// The last tiles of a 256-tile update (a.tail.., a.total of them): quarters of
// 128, or sixteenths of 64 where those still fit one per CU (16 of the 1296
// tiles of 48 GPT-small matrices: 17 us against 12).
hipError_t launch_update_tail(KArgs a, hipStream_t st) {
  if (a.total <= 0) return hipSuccess;
  const int bt = a.total <= 16 ? kTileTiny : kTileSmall, per = 256 / bt;
  a.total *= per * per;
  if (a.last) launch_small_k<KIND_UPD_LAST>(kBF16, bt, a, st);
  else if (a.init_step) launch_small_k<KIND_UPDI>(kBF16, bt, a, st);
  else if (a.x0b) launch_small_k<KIND_UPD0>(kBF16, bt, a, st);
  else launch_small_k<KIND_UPD>(kBF16, bt, a, st);
  return hipGetLastError();
}

template <int BT, int PL>
static void launch_reduce_t(int kind, const KArgs& a, hipStream_t st) {
  const dim3 g(a.total < 1024 ? a.total : 1024), b(kThreads);
  if (kind == KIND_GRAM) hipLaunchKernelGGL((small_reduce_kernel<KIND_GRAM, BT, PL>), g, b, 0, st, a);
  else hipLaunchKernelGGL((small_reduce_kernel<KIND_A2, BT, PL>), g, b, 0, st, a);
}

hipError_t launch_small_reduce(int prec, int bt, int kind, const KArgs& a, hipStream_t st) {
  if (a.total <= 0) return hipSuccess;
  if (prec == kTiny) {
    launch_reduce_t<64, 0>(kind, a, st);
  } else if (prec == kF32) {
    if (bt == kTileTiny) launch_reduce_t<64, 2>(kind, a, st);
    else launch_reduce_t<128, 2>(kind, a, st);
  } else {
    if (bt == kTileTiny) launch_reduce_t<64, 1>(kind, a, st);
    else launch_reduce_t<128, 1>(kind, a, st);
  }
  return hipGetLastError();
}

// 128 tiles fill the 256 CUs two at a time.  A last round of few tiles would
// take as long as a full one (s = 4096: 528 tiles, 16 of them in a second
// round: 0.31 ms per product against 0.18), so those tiles run as quarters of 64
// in a launch of their own, up to a fourth of a round.
template <int KIND>
static hipError_t launch_fast_t(int prec, int bt, KArgs a, hipStream_t st) {
  a.tail = -1;
  if (prec == kTiny) {
    typedef SmallTile<64, 4, 1, 0> C;
    hipLaunchKernelGGL((small_fast_kernel<KIND, C>), dim3(a.total < 256 ? a.total : 256), dim3(C::NT), 0, st, a);
    return hipGetLastError();
  }
  typedef SmallTile<64, 4, 1, 2, 64> Q;
  if (bt == kTileTiny) {
    hipLaunchKernelGGL((small_fast_kernel<KIND, Q>), dim3(a.total < 256 ? a.total : 256), dim3(Q::NT), 0, st, a);
    return hipGetLastError();
  }
  typedef SmallTile<128, 1, 1, 2> C;
  constexpr int kRound = 512;
  const int rest = !a.alike && a.total > kRound && a.total % kRound <= kRound / 4 ? a.total % kRound : 0;
  a.total -= rest;
  hipLaunchKernelGGL((small_fast_kernel<KIND, C>), dim3(a.total < kRound ? a.total : kRound), dim3(C::NT), 0, st, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || !rest) return e;
  a.tail = a.total;
  a.total = 4 * rest;
  hipLaunchKernelGGL((small_fast_kernel<KIND, Q>), dim3(a.total < 256 ? a.total : 256), dim3(Q::NT), 0, st, a);
  return hipGetLastError();
}

hipError_t launch_fast(int prec, int bt, int kind, const KArgs& a, hipStream_t st) {
  if (a.total <= 0) return hipSuccess;
  return kind == KIND_GRAM ? launch_fast_t<KIND_GRAM>(prec, bt, a, st) : launch_fast_t<KIND_A2>(prec, bt, a, st);
}

hipError_t launch_planes(const KArgs& a, hipStream_t st) {
  if (a.total <= 0) return hipSuccess;
  hipLaunchKernelGGL(planes_kernel, dim3(a.total < 2048 ? a.total : 2048), dim3(kThreads), 0, st, a);
  return hipGetLastError();
}

}  // namespace pe
