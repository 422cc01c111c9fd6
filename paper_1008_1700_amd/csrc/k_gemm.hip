// Grouped GEMM on CDNA4 matrix cores: D = C0 +/- op(A) op(B) over a list of
// independent problems (one launch covers every block of the partition).
//
// k_gemm_dma: f64 / f32 MFMA 16x16x4, operands copied from global memory
// straight into LDS.  k_gemm_std: the same products with element loads, for
// operands that are not 16-byte aligned.  k_gemm_bf16 (bf16 MFMA on FP32
// operands staged through registers), k_gemm_dl (the same bf16 products with
// the operands copied straight into LDS, split as they are read) and
// k_gemm_x3 (256 x 256 tiles, split as they are staged); all three give the
// same bits.  Operands are column-major (LAPACK layout); M and N need only be
// multiples of 64 (a larger tile on the edge is masked).  Triangular operands are exploited twice: the K range of
// each output tile is clipped to where both operands can be nonzero, and
// masks read the unit-lower / upper / lower halves of the packed tiles.
//
// The MFMA is fed with B^T as its first and A^T as its second operand, so it
// accumulates D^T: the 16 lanes of a lane group hold 16 consecutive rows of
// one column of D, and the stores to the column-major D are 64-128-byte
// segments.
#include "ddps_internal.h"
#include "mma_device.h"

#include <type_traits>

namespace ddps {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// The problem records hold generic pointers; loads through them compile to
// flat loads, which also count against the LDS wait counter, so every wait
// for LDS would wait for them too.  Casting to the global address space gives
// global loads and stores with their own counter.
template <typename T> using gptr = const __attribute__((address_space(1))) T*;
template <typename T> using gmut = __attribute__((address_space(1))) T*;
__device__ __forceinline__ float4 gload4(const float* p) {
  const f32x4 v = *(gptr<f32x4>)p;
  return make_float4(v[0], v[1], v[2], v[3]);
}

// Logical workgroup index such that each XCD (hardware dispatches workgroups
// round-robin over the 8 XCDs) receives one contiguous range of tiles: tiles
// of the same block then share that XCD's L2.
__device__ __forceinline__ int xcd_swizzle(int bid, int n) {
  const int xcd = bid & 7, idx = bid >> 3;
  const int per = n >> 3, rem = n & 7;
  return xcd * per + min(xcd, rem) + idx;
}

__device__ __forceinline__ int find_prob(const GemmProb* __restrict__ probs, int nprob, int wg) {
  int lo = 0, hi = nprob - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (probs[mid].tile0 <= wg) lo = mid; else hi = mid - 1;
  }
  return lo;
}

// Value of op(X)(r, c) given the stored value v: masks of the packed
// triangles (unit lower, upper, lower with its diagonal) and zero outside the
// problem (rows >= rmax or columns >= cmax).  A select, so whatever the other
// triangle of a packed tile holds never reaches a product.
template <typename T>
__device__ __forceinline__ T select_op(T v, int r, int c, bool lu, bool up, bool lo, int rmax, int cmax) {
  if (lu) v = r > c ? v : (r == c ? T(1) : T(0));
  if (up) v = r <= c ? v : T(0);
  if (lo) v = r >= c ? v : T(0);
  return (r < rmax && c < cmax) ? v : T(0);
}

// Output mask of the epilogue: G_D_UP stores only entries on or above the
// diagonal, G_D_LO only entries on or below it (the two halves of a packed
// pair of triangles); the other half of the destination is left untouched.
__device__ __forceinline__ bool store_ok(int fl, int r, int c) {
  if ((fl & G_D_UP) && r > c) return false;
  if ((fl & G_D_LO) && r < c) return false;
  return true;
}

struct TileCoord {
  int I0, J0, kb, ke;
};

template <int BM, int BN>
__device__ __forceinline__ TileCoord tile_of(const GemmProb& P, int wg) {
  const int tiles_m = (P.M + BM - 1) / BM;
  const int local = wg - P.tile0;
  TileCoord t;
  t.I0 = (local % tiles_m) * BM;
  t.J0 = (local / tiles_m) * BN;
  const int fl = P.flags;
  t.kb = 0;
  t.ke = P.K;
  if (fl & G_A_UP) t.kb = max(t.kb, t.I0);
  if (fl & G_B_LO) t.kb = max(t.kb, t.J0);
  if (fl & G_A_LO) t.ke = min(t.ke, t.I0 + BM);
  if (fl & G_B_UP) t.ke = min(t.ke, t.J0 + BN);
  return t;
}

// ------------------------------------------------------------------------
// f64 / f32 with element loads (any alignment): 256 threads = 4 waves in a
// 2 x 2 arrangement, each wave a 32 x 32 sub-tile of 16 x 16 MFMA blocks; K advances in chunks of 16 staged through LDS, with the next
// chunk's global loads in flight while the current chunk is multiplied.
// ------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256, 2) void k_gemm_std(const GemmProb* __restrict__ probs, int nprob,
                                                     const int32_t* __restrict__ order) {
  constexpr int BM = 64, BN = 64, BK = 16, PADL = 4;
  constexpr int MB = BM / 32, NB = BN / 32;          // 16x16 blocks per wave
  constexpr int AE = BM * BK / 256, BE = BN * BK / 256;  // elements per thread
  __shared__ T As[2][BK][BM + PADL];
  __shared__ T Bs[2][BK][BN + PADL];
  using acc_t = typename Mma<T>::acc;

  const int wg = order ? order[xcd_swizzle(blockIdx.x, gridDim.x)] : xcd_swizzle(blockIdx.x, gridDim.x);
  const GemmProb P = probs[find_prob(probs, nprob, wg)];
  const TileCoord tc = tile_of<BM, BN>(P, wg);
  const int I0 = tc.I0, J0 = tc.J0, kb = tc.kb, ke = tc.ke;
  const int fl = P.flags;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave & 1, wn = wave >> 1;
  gptr<T> A = (gptr<T>)P.A;
  gptr<T> B = (gptr<T>)P.B;
  const bool a_lu = fl & G_A_MLU, a_up = fl & G_A_MUP, b_lu = fl & G_B_MLU, b_up = fl & G_B_MUP;
  const bool a_lo = fl & G_A_MLO, b_lo = fl & G_B_MLO;

  acc_t acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[i][j] = acc_t{0, 0, 0, 0};

  // A chunk BM x 16: thread -> row m = tid % BM, k = tid / BM + (256/BM) i
  // B chunk 16 x BN: thread -> col n = tid % BN, k = (tid / BN) * BE + i  (BE consecutive k)
  constexpr int ASTEP = 256 / BM;
  static_assert(AE * ASTEP == BK, "A chunk mapping");
  const int am = tid % BM, ak = tid / BM;
  const int bn = tid % BN, bk0 = (tid / BN) * BE;
  const int arow = min(I0 + am, P.M - 1);
  const int bcol = min(J0 + bn, P.N - 1);
  T ra[AE], rb[BE];
  auto load = [&](int k0) {
#pragma unroll
    for (int i = 0; i < AE; ++i) {
      const int c = k0 + ak + ASTEP * i;
      ra[i] = select_op(A[(int64_t)c * P.lda + arow], I0 + am, c, a_lu, a_up, a_lo, P.M, 1 << 30);
    }
    gptr<T> bp = B + (int64_t)bcol * P.ldb + k0 + bk0;
#pragma unroll
    for (int i = 0; i < BE; ++i) rb[i] = select_op(bp[i], k0 + bk0 + i, J0 + bn, b_lu, b_up, b_lo, 1 << 30, P.N);
  };
  auto store = [&](int buf) {
#pragma unroll
    for (int i = 0; i < AE; ++i) As[buf][ak + ASTEP * i][am] = ra[i];
#pragma unroll
    for (int i = 0; i < BE; ++i) Bs[buf][bk0 + i][bn] = rb[i];
  };

  if (kb < ke) {
    load(kb);
    store(0);
    __syncthreads();
    int cur = 0;
    for (int k0 = kb; k0 < ke; k0 += BK) {
      const bool more = (k0 + BK) < ke;
      if (more) load(k0 + BK);
#pragma unroll
      for (int k4 = 0; k4 < BK / 4; ++k4) {
        const int kk = k4 * 4 + (lane >> 4);
        T xa[NB], xb[MB];
#pragma unroll
        for (int ni = 0; ni < NB; ++ni) xa[ni] = Bs[cur][kk][wn * (BN / 2) + ni * 16 + (lane & 15)];
#pragma unroll
        for (int mi = 0; mi < MB; ++mi) xb[mi] = As[cur][kk][wm * (BM / 2) + mi * 16 + (lane & 15)];
#pragma unroll
        for (int mi = 0; mi < MB; ++mi)
#pragma unroll
          for (int ni = 0; ni < NB; ++ni) acc[mi][ni] = Mma<T>::run(xa[ni], xb[mi], acc[mi][ni]);
      }
      if (more) store(cur ^ 1);
      __syncthreads();
      cur ^= 1;
    }
  }

  // Epilogue: lane holds D[row = .. + (lane&15)][col = .. + Mma::row(lane, v)].
  // Whole tiles load their C0 values in one batch per 16 x 16 block.
  gptr<T> C0 = (gptr<T>)P.C0;
  gmut<T> D = (gmut<T>)P.D;
  const bool has_c0 = fl & G_C0;
  const T sg = (fl & G_NEG) ? T(-1) : T(1);
  if (I0 + BM <= P.M && J0 + BN <= P.N && !(fl & (G_D_UP | G_D_LO))) {
#pragma unroll
    for (int mi = 0; mi < MB; ++mi)
#pragma unroll
      for (int ni = 0; ni < NB; ++ni) {
        const int r = I0 + wm * (BM / 2) + mi * 16 + (lane & 15);
        const int c = J0 + wn * (BN / 2) + ni * 16;
        if (has_c0) {
          T cv[4];
#pragma unroll
          for (int v = 0; v < 4; ++v) cv[v] = C0[(int64_t)(c + Mma<T>::row(lane, v)) * P.ldc0 + r];
#pragma unroll
          for (int v = 0; v < 4; ++v) D[(int64_t)(c + Mma<T>::row(lane, v)) * P.ldd + r] = sg * acc[mi][ni][v] + cv[v];
        } else {
#pragma unroll
          for (int v = 0; v < 4; ++v) D[(int64_t)(c + Mma<T>::row(lane, v)) * P.ldd + r] = sg * acc[mi][ni][v];
        }
      }
    return;
  }
#pragma unroll
  for (int mi = 0; mi < MB; ++mi)
#pragma unroll
    for (int ni = 0; ni < NB; ++ni)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = I0 + wm * (BM / 2) + mi * 16 + (lane & 15);
        const int c = J0 + wn * (BN / 2) + ni * 16 + Mma<T>::row(lane, v);
        if (r < P.M && c < P.N && store_ok(fl, r, c)) {
          T val = sg * acc[mi][ni][v];
          if (has_c0) val += C0[(int64_t)c * P.ldc0 + r];
          D[(int64_t)c * P.ldd + r] = val;
        }
      }
}

// ------------------------------------------------------------------------
// bf16 MFMA (32x32x16, FP32 accumulation) on FP32-stored operands.  With
// SPLIT each FP32 operand x is written as hi + lo, hi = bf16(x),
// lo = bf16(x - hi), and the product is hi*hi + hi*lo + lo*hi (the lo*lo
// term lies below the FP32 rounding of the result).  The split is done once
// per element while the chunk is staged into LDS, in layout [row][k] with k
// contiguous, so each MFMA operand is one 16-byte LDS read.
//
// MFMA 32x32x16 bf16 lane layout (measured): operand X (32 x 16) lane l
// holds X[l%32][8(l/32) .. +8), operand Y (16 x 32) lane l holds
// Y[8(l/32) .. +8)[l%32]; accumulator register v of lane l is element
// (8(v/4) + 4(l/32) + v%4, l%32).
// ------------------------------------------------------------------------
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Where a block of rows [r, r + nr) and columns [c, c + nc) lies: 0 nothing of
// it is stored (outside the problem, whose sides are multiples of the block's,
// or on the other side of a D_UP / D_LO diagonal), 1 all of it, 2 the
// diagonal crosses it.
__device__ __forceinline__ int store_block(const GemmProb& P, int r, int c, int nr, int nc) {
  if (r >= P.M || c >= P.N) return 0;
  if (P.flags & G_D_UP) return r > c + nc - 1 ? 0 : r + nr - 1 <= c ? 1 : 2;
  if (P.flags & G_D_LO) return r + nr - 1 < c ? 0 : r >= c + nc - 1 ? 1 : 2;
  return 1;
}

// Epilogue of MB x NB accumulator blocks of 32 x 32, RS rows and CS columns
// apart: register v of lane l in block (mi, ni) is D(r0 + RS (mi ^ flip) +
// l % 32, c0 + CS ni + 8 (v / 4) + 4 (l / 32) + v % 4), and D = C0 -/+ acc.
// C0 is loaded one row block (NB blocks) at a time before the first store: C0
// and D may be the same entries, so the loads cannot move above stores by
// themselves, and one by one each waits for the memory's latency.  Addresses
// are a wave-uniform part and one 32-bit lane offset.
template <int MB, int NB, int RS = 32, int CS = 32>
__device__ __forceinline__ void store_tile32(const GemmProb& P, const f32x16 (&acc)[MB][NB], int r0, int c0,
                                             int lane, int flip = 0) {
  gptr<float> C0 = (gptr<float>)P.C0;
  gmut<float> D = (gmut<float>)P.D;
  const bool has_c0 = P.flags & G_C0;
  const float sg = (P.flags & G_NEG) ? -1.f : 1.f;
  const uint32_t lc = (4u * (lane >> 5) * (uint32_t)P.ldc0 + (lane & 31)) * 4u;
  const uint32_t ld = (4u * (lane >> 5) * (uint32_t)P.ldd + (lane & 31)) * 4u;
  auto at = [&](int mi, int ni, int v, int ldx) -> int64_t {
    return (int64_t)(c0 + CS * ni + 8 * (v >> 2) + (v & 3)) * ldx + r0 + RS * (mi ^ flip);
  };
#pragma unroll
  for (int mi = 0; mi < MB; ++mi) {
    const int r = r0 + RS * (mi ^ flip);
    int how[NB];
    bool whole = true;
#pragma unroll
    for (int ni = 0; ni < NB; ++ni) {
      how[ni] = store_block(P, r, c0 + CS * ni, 32, 32);
      whole = whole && how[ni] == 1;
    }
    if (whole) {
      if (has_c0) {
        float cv[NB][16];
#pragma unroll
        for (int ni = 0; ni < NB; ++ni)
#pragma unroll
          for (int v = 0; v < 16; ++v) cv[ni][v] = *(gptr<float>)((gptr<char>)(C0 + at(mi, ni, v, P.ldc0)) + lc);
#pragma unroll
        for (int ni = 0; ni < NB; ++ni)
#pragma unroll
          for (int v = 0; v < 16; ++v)
            *(gmut<float>)((gmut<char>)(D + at(mi, ni, v, P.ldd)) + ld) = sg * acc[mi][ni][v] + cv[ni][v];
      } else {
#pragma unroll
        for (int ni = 0; ni < NB; ++ni)
#pragma unroll
          for (int v = 0; v < 16; ++v)
            *(gmut<float>)((gmut<char>)(D + at(mi, ni, v, P.ldd)) + ld) = sg * acc[mi][ni][v];
      }
      continue;
    }
#pragma unroll
    for (int ni = 0; ni < NB; ++ni) {
      if (how[ni] == 0) continue;
      auto ok = [&](int v) {
        return store_ok(P.flags, r + (lane & 31), c0 + CS * ni + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3));
      };
      float cv[16];
      if (has_c0) {
#pragma unroll
        for (int v = 0; v < 16; ++v)
          cv[v] = ok(v) ? *(gptr<float>)((gptr<char>)(C0 + at(mi, ni, v, P.ldc0)) + lc) : 0.f;
      }
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (ok(v)) {
          const float val = sg * acc[mi][ni][v];
          *(gmut<float>)((gmut<char>)(D + at(mi, ni, v, P.ldd)) + ld) = has_c0 ? val + cv[v] : val;
        }
    }
  }
}

template <bool SPLIT, int BM, int BN, int OCC = 1, int ST = 1, int BK = 32, int NW = 4>
__global__ __launch_bounds__(64 * NW, OCC) void k_gemm_bf16(const GemmProb* __restrict__ probs, int nprob,
                                                 const int32_t* __restrict__ order) {
  // NW waves in a 2 x NW/2 arrangement, wave tile BM/2 x 2BN/NW of 32 x 32 blocks
  constexpr int NT = 64 * NW;
  constexpr int LDK = BK + 8;
  constexpr int MB = BM / 64, NB = BN / (16 * NW);
  constexpr int NS = SPLIT ? 2 : 1;
  __shared__ __attribute__((aligned(16))) __bf16 As[ST][NS][BM][LDK];
  __shared__ __attribute__((aligned(16))) __bf16 Bs[ST][NS][BN][LDK];

  const int wg = order ? order[xcd_swizzle(blockIdx.x, gridDim.x)] : xcd_swizzle(blockIdx.x, gridDim.x);
  const GemmProb P = probs[find_prob(probs, nprob, wg)];
  const TileCoord tc = tile_of<BM, BN>(P, wg);
  const int I0 = tc.I0, J0 = tc.J0, kb = tc.kb, ke = tc.ke;
  const int fl = P.flags;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave & 1, wn = wave >> 1;
  const float* __restrict__ A = (const float*)P.A;
  const float* __restrict__ B = (const float*)P.B;
  const bool a_lu = fl & G_A_MLU, a_up = fl & G_A_MUP, b_lu = fl & G_B_MLU, b_up = fl & G_B_MUP;
  const bool a_lo = fl & G_A_MLO, b_lo = fl & G_B_MLO;
  const bool a_edge = I0 + BM > P.M, b_edge = J0 + BN > P.N;

  f32x16 acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  // A chunk BM x BK: thread -> 4 consecutive rows (a float4 per k) x AK k
  // (float4 loads along the contiguous row index).
  // B chunk BK x BN: thread -> one column, BKT consecutive k (float4 loads,
  // 16-byte LDS stores).
  constexpr int AROWG = BM / 4;
  constexpr int AK = BK * AROWG / NT;
  constexpr int BKT = BK * BN / NT;
  static_assert(AK >= 1 && BKT % 8 == 0, "chunk split");
  const int arg = tid % AROWG, akg = tid / AROWG;
  const int ar = I0 + 4 * arg;
  const int bn = tid % BN, bkg = tid / BN;
  const int bc = J0 + bn;
  const int arow_ld = min(ar, P.M - 4);
  const int bcol_ld = min(bc, P.N - 1);
  float4 ra[AK];
  float4 rb[BKT / 4];
  auto load = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < AK; ++i)
      ra[i] = gload4(A + (int64_t)(k0 + akg * AK + i) * P.lda + arow_ld);
    const float* bp = B + (int64_t)bcol_ld * P.ldb + k0 + bkg * BKT;
#pragma unroll
    for (int i = 0; i < BKT / 4; ++i) rb[i] = gload4(bp + 4 * i);
  };
  typedef __bf16 bfa __attribute__((ext_vector_type(AK)));
  // Stage one chunk into LDS as bf16 (hi, and lo = x - hi when split).  The
  // masked form applies the packed-triangle and edge masks; it is taken only
  // for chunks that cross a packed triangle's diagonal or the problem edge.
  auto store_chunk = [&](int st, int k0, bool am, bool bm) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int r = ar + q;
      bfa h, l;
#pragma unroll
      for (int i = 0; i < AK; ++i) {
        float x = ra[i][q];
        if (am) x = select_op(x, r, k0 + akg * AK + i, a_lu, a_up, a_lo, P.M, 1 << 30);
        h[i] = (__bf16)x;
        if (SPLIT) l[i] = (__bf16)(x - (float)h[i]);
      }
      *(bfa*)&As[st][0][4 * arg + q][akg * AK] = h;
      if (SPLIT) *(bfa*)&As[st][NS - 1][4 * arg + q][akg * AK] = l;
    }
#pragma unroll
    for (int j = 0; j < BKT / 8; ++j) {
      bf16x8 h, l;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        float x = rb[2 * j + e / 4][e % 4];
        if (bm) x = select_op(x, k0 + bkg * BKT + 8 * j + e, bc, b_lu, b_up, b_lo, 1 << 30, P.N);
        h[e] = (__bf16)x;
        if (SPLIT) l[e] = (__bf16)(x - (float)h[e]);
      }
      *(bf16x8*)&Bs[st][0][bn][bkg * BKT + 8 * j] = h;
      if (SPLIT) *(bf16x8*)&Bs[st][NS - 1][bn][bkg * BKT + 8 * j] = l;
    }
  };
  auto stage = [&](int st, int k0) __attribute__((always_inline)) {
    const bool am = a_edge || ((a_lu || a_up || a_lo) && k0 + BK > I0 && k0 < I0 + BM);
    const bool bm = b_edge || ((b_lu || b_up || b_lo) && k0 + BK > J0 && k0 < J0 + BN);
    if (am || bm) store_chunk(st, k0, am, bm);
    else store_chunk(st, k0, false, false);
  };
  auto compute = [&](int st) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) {
      const int kk = ks * 16 + 8 * (lane >> 5);
      bf16x8 xh[NB], xl[NB], yh[MB], yl[MB];
#pragma unroll
      for (int ni = 0; ni < NB; ++ni) {
        const int n = wn * (2 * BN / NW) + ni * 32 + (lane & 31);
        xh[ni] = *(const bf16x8*)&Bs[st][0][n][kk];
        if (SPLIT) xl[ni] = *(const bf16x8*)&Bs[st][NS - 1][n][kk];
      }
#pragma unroll
      for (int mi = 0; mi < MB; ++mi) {
        const int m = wm * (BM / 2) + mi * 32 + (lane & 31);
        yh[mi] = *(const bf16x8*)&As[st][0][m][kk];
        if (SPLIT) yl[mi] = *(const bf16x8*)&As[st][NS - 1][m][kk];
      }
      // one term over every block before the next, so consecutive MFMAs
      // write different accumulators (small terms first)
      if (SPLIT) {
#pragma unroll
        for (int mi = 0; mi < MB; ++mi)
#pragma unroll
          for (int ni = 0; ni < NB; ++ni)
            acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xl[ni], yh[mi], acc[mi][ni], 0, 0, 0);
#pragma unroll
        for (int mi = 0; mi < MB; ++mi)
#pragma unroll
          for (int ni = 0; ni < NB; ++ni)
            acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xh[ni], yl[mi], acc[mi][ni], 0, 0, 0);
      }
#pragma unroll
      for (int mi = 0; mi < MB; ++mi)
#pragma unroll
        for (int ni = 0; ni < NB; ++ni)
          acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xh[ni], yh[mi], acc[mi][ni], 0, 0, 0);
    }
  };

  if (kb < ke) {
    if (ST == 2) {
      // two LDS stages: the next chunk is loaded before and staged after the
      // current chunk's products, one barrier per chunk
      load(kb);
      stage(0, kb);
      __syncthreads();
      int st = 0;
      for (int kcur = kb; kcur < ke; kcur += BK) {
        const bool more = kcur + BK < ke;
        if (more) load(kcur + BK);
        compute(st);
        if (more) stage(st ^ 1, kcur + BK);
        __syncthreads();
        st ^= 1;
      }
    } else {
      load(kb);
      for (int kcur = kb; kcur < ke; kcur += BK) {
        __syncthreads();             // previous chunk's LDS reads are done
        stage(0, kcur);
        __syncthreads();
        if (kcur + BK < ke) load(kcur + BK);
        compute(0);
      }
    }
  }

  store_tile32<MB, NB>(P, acc, I0 + wm * (BM / 2), J0 + wn * (2 * BN / NW), lane);
}


// ------------------------------------------------------------------------
// bf16 MFMA with the operands copied from global memory straight into LDS
// (global_load_lds_dwordx4: each lane's 16 bytes land at lane * 16 of the
// wave's 1 KiB destination), FP32 in LDS, split into hi/lo in registers as
// the fragments are read.  No VGPRs hold operands in flight and no staging
// pass stands between the loads and the products.
//
// LDS, two stages of a 32-deep K chunk:
//   A as [k][m] (m contiguous, as in global memory): one wave instruction
//     fills 2 rows of k; a fragment (8 consecutive k of one row) is
//     eight 4-byte reads.
//   B as [n][k] (k contiguous): one wave instruction fills 8 columns; the
//     eight 16-byte slots of column n hold k pieces slot ^ (n & 7), so that
//     the 16-byte fragment reads of 8 consecutive columns hit distinct banks.
// Per chunk: one barrier (the chunk has landed, the other stage is free), the
// first 16-deep step's LDS reads, the DMA of the next chunk into the other
// stage, then the products.  Chunks crossing a packed triangle's diagonal get
// their masks applied in LDS first (one more barrier).  Rows beyond M and
// column groups beyond N load clamped in-range data: they only feed outputs
// that are not stored.  Same split and the same MFMA order per 16-deep step
// as k_gemm_bf16, so the results are bitwise the same.
// ------------------------------------------------------------------------
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef const __attribute__((address_space(1))) void* dma_src_t;
typedef __attribute__((address_space(3))) void* dma_dst_t;

// hi = bf16(x), lo = bf16(x - hi) for 8 values, converted two at a time
template <bool SPLIT>
__device__ __forceinline__ void split8(const float (&x)[8], bf16x8& h, bf16x8& l) {
#pragma unroll
  for (int e = 0; e < 8; e += 2) {
    const f32x2 v = {x[e], x[e + 1]};
    const bf16x2 hv = __builtin_convertvector(v, bf16x2);
    h[e] = hv[0];
    h[e + 1] = hv[1];
    if (SPLIT) {
      const f32x2 r = {x[e] - (float)hv[0], x[e + 1] - (float)hv[1]};
      const bf16x2 lv = __builtin_convertvector(r, bf16x2);
      l[e] = lv[0];
      l[e + 1] = lv[1];
    }
  }
}

constexpr int kDlTile = 128, kDlBK = 32;
constexpr int kDlInstr = kDlBK * kDlTile / 256 / 4;   // instructions per wave, operand and chunk

// One K chunk of k_gemm_dl.  The LDS pointers are restrict: the compiler then
// sees that the reads of the current stage (ca, cb) do not alias the DMA into
// the next stage (na, nb), and does not make them wait for it.
template <bool SPLIT>
__device__ __forceinline__ void dl_chunk(const float* __restrict__ ca, const float* __restrict__ cb,
                                         float* __restrict__ na, float* __restrict__ nb,
                                         const char* __restrict__ ga, const char* __restrict__ gb,
                                         const int64_t (&goff)[2 * kDlInstr], bool issue_next, int lane, int wm, int wn,
                                         f32x16 (&acc)[2][2]) {
  constexpr int BM = kDlTile, BN = kDlTile, BK = kDlBK, MB = 2, NB = 2, NA = kDlInstr, NBI = kDlInstr;
  auto read = [&](int ks, float (&xb)[NB][8], float (&xa)[MB][8]) __attribute__((always_inline)) {
    const int kk = ks * 16 + 8 * (lane >> 5);
#pragma unroll
    for (int ni = 0; ni < NB; ++ni) {
      const int n = wn * (BN / 2) + ni * 32 + (lane & 31);
      const int s0 = (kk >> 2) ^ (n & 7), s1 = ((kk >> 2) + 1) ^ (n & 7);
      const f32x4 v0 = *(const f32x4*)&cb[n * BK + 4 * s0];
      const f32x4 v1 = *(const f32x4*)&cb[n * BK + 4 * s1];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        xb[ni][e] = v0[e];
        xb[ni][e + 4] = v1[e];
      }
    }
#pragma unroll
    for (int mi = 0; mi < MB; ++mi) {
      const int m = wm * (BM / 2) + mi * 32 + (lane & 31);
#pragma unroll
      for (int e = 0; e < 8; ++e) xa[mi][e] = ca[(kk + e) * BM + m];
    }
  };
  auto mult = [&](const float (&xb)[NB][8], const float (&xa)[MB][8]) __attribute__((always_inline)) {
    bf16x8 xh[NB], xl[NB];
#pragma unroll
    for (int ni = 0; ni < NB; ++ni) split8<SPLIT>(xb[ni], xh[ni], xl[ni]);
#pragma unroll
    for (int mi = 0; mi < MB; ++mi) {
      bf16x8 yh, yl;
      split8<SPLIT>(xa[mi], yh, yl);
      if (SPLIT) {
#pragma unroll
        for (int ni = 0; ni < NB; ++ni)
          acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xl[ni], yh, acc[mi][ni], 0, 0, 0);
#pragma unroll
        for (int ni = 0; ni < NB; ++ni)
          acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xh[ni], yl, acc[mi][ni], 0, 0, 0);
      }
#pragma unroll
      for (int ni = 0; ni < NB; ++ni)
        acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(xh[ni], yh, acc[mi][ni], 0, 0, 0);
    }
  };
  float xb[NB][8], xa[MB][8];
  read(0, xb, xa);
  __builtin_amdgcn_sched_barrier(0);
  if (issue_next) {
#pragma unroll
    for (int q = 0; q < NA; ++q)
      __builtin_amdgcn_global_load_lds((dma_src_t)(ga + goff[q]), (dma_dst_t)(na + q * 256), 16, 0, 0);
#pragma unroll
    for (int q = 0; q < NBI; ++q)
      __builtin_amdgcn_global_load_lds((dma_src_t)(gb + goff[NA + q]), (dma_dst_t)(nb + q * 256), 16, 0, 0);
  }
  __builtin_amdgcn_sched_barrier(0);
  mult(xb, xa);
#pragma unroll
  for (int ks = 1; ks < BK / 16; ++ks) {
    __builtin_amdgcn_sched_barrier(0);
    read(ks, xb, xa);
    mult(xb, xa);
  }
}

template <bool SPLIT>
__global__ __launch_bounds__(256, 2) void k_gemm_dl(const GemmProb* __restrict__ probs, int nprob,
                                                    const int32_t* __restrict__ order) {
  constexpr int BM = kDlTile, BN = kDlTile, BK = kDlBK, MB = 2, NB = 2, NA = kDlInstr, NBI = kDlInstr;
  constexpr int KPI = 256 / BM;   // k rows per A instruction
  __shared__ __attribute__((aligned(16))) float As[2][BK * BM];
  __shared__ __attribute__((aligned(16))) float Bs[2][BN * BK];

  const int wg = order ? order[xcd_swizzle(blockIdx.x, gridDim.x)] : xcd_swizzle(blockIdx.x, gridDim.x);
  const GemmProb P = probs[find_prob(probs, nprob, wg)];
  const TileCoord tc = tile_of<BM, BN>(P, wg);
  const int I0 = tc.I0, J0 = tc.J0, kb = tc.kb, ke = tc.ke;
  const int fl = P.flags;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave & 1, wn = wave >> 1;
  const char* A = (const char*)P.A;
  const char* B = (const char*)P.B;
  const bool a_lu = fl & G_A_MLU, a_up = fl & G_A_MUP, b_lu = fl & G_B_MLU, b_up = fl & G_B_MUP;
  const bool a_lo = fl & G_A_MLO, b_lo = fl & G_B_MLO;

  f32x16 acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  // byte offsets of this lane's 16-byte pieces: a wave-uniform part per
  // instruction and one per-lane part for A and one for B
  const int64_t a_lane =
      ((int64_t)((lane * 4) / BM) * P.lda + min(I0 + (lane * 4) % BM, P.M - 4)) * 4;
  const int64_t b_lane = ((int64_t)(lane >> 3) * P.ldb + 4 * ((lane & 7) ^ ((lane >> 3) & 7))) * 4;
  auto a_off = [&](int k, int q) __attribute__((always_inline)) {
    return (int64_t)(k + (wave * NA + q) * KPI) * P.lda * 4 + a_lane;
  };
  auto b_off = [&](int k, int q) __attribute__((always_inline)) {
    return ((int64_t)min(J0 + 8 * (wave * NBI + q), P.N - 8) * P.ldb + k) * 4 + b_lane;
  };

  if (kb < ke) {
#pragma unroll
    for (int q = 0; q < NA; ++q)
      __builtin_amdgcn_global_load_lds((dma_src_t)(A + a_off(kb, q)), (dma_dst_t)&As[0][(wave * NA + q) * 256], 16,
                                       0, 0);
#pragma unroll
    for (int q = 0; q < NBI; ++q)
      __builtin_amdgcn_global_load_lds((dma_src_t)(B + b_off(kb, q)), (dma_dst_t)&Bs[0][(wave * NBI + q) * 256], 16,
                                       0, 0);
    int st = 0;
    for (int k0 = kb; k0 < ke; k0 += BK) {
      __syncthreads();   // chunk k0 has landed; every wave is done with the other stage
      const bool am = (a_lu || a_up || a_lo) && k0 + BK > I0 && k0 < I0 + BM;
      const bool bm = (b_lu || b_up || b_lo) && k0 + BK > J0 && k0 < J0 + BN;
      if (am || bm) {
        if (am)
          for (int i = tid; i < BK * BM; i += 256) {
            const int k = i / BM, m = i % BM;
            As[st][i] = select_op(As[st][i], I0 + m, k0 + k, a_lu, a_up, a_lo, 1 << 30, 1 << 30);
          }
        if (bm)
          for (int i = tid; i < BN * BK; i += 256) {
            const int n = i / BK, k = 4 * (((i % BK) >> 2) ^ (n & 7)) + (i & 3);
            Bs[st][i] = select_op(Bs[st][i], k0 + k, J0 + n, b_lu, b_up, b_lo, 1 << 30, 1 << 30);
          }
        __syncthreads();
      }
      const int k1 = k0 + BK;
      int64_t goff[NA + NBI];
#pragma unroll
      for (int q = 0; q < NA; ++q) goff[q] = a_off(k1, q);
#pragma unroll
      for (int q = 0; q < NBI; ++q) goff[NA + q] = b_off(k1, q);
      dl_chunk<SPLIT>(As[st], Bs[st], &As[st ^ 1][wave * NA * 256], &Bs[st ^ 1][wave * NBI * 256], A, B, goff, k1 < ke,
                      lane, wm, wn, acc);
      st ^= 1;
    }
  }
  store_tile32<MB, NB>(P, acc, I0 + wm * (BM / 2), J0 + wn * (BN / 2), lane);
}

// ------------------------------------------------------------------------
// f64 / f32 with the operands copied from global memory straight into LDS
// (global_load_lds_dwordx4) and no vector instruction between them and the
// products.  Workgroup tile BM x BN (128 x 128 or 64 x 64), 4 waves 2 x 2; a
// K chunk is 128 bytes deep (16 doubles, 32 floats), two LDS stages.
//   A as [k][m]: one wave instruction fills 1 KiB (1, 2 or 4 rows of k), the
//     next one starts kPadA bytes later, so that the two k rows of a 32-lane
//     read pass lie in different banks;
//   B as [n][k]: one wave instruction fills 8 columns of 128 bytes; slot s of
//     column n holds the 16-byte k piece s ^ (n >> 1 & 7).
// Lane group g = lane / 16 takes the chunk's k in [g kq, (g + 1) kq), one per
// product (kq = 4 doubles, 8 floats), so its B entries are two 16-byte reads,
// and the lane's two rows of A are adjacent: an accumulator pair holds rows
// 2i, 2i + 1 and is stored as one vector.  Wave (wm, wn) owns rows 64 h +
// 32 wm + [0, 32) and columns 64 h + 32 wn + [0, 32), h < BM / 64: a tile
// with only 64 rows or columns inside the problem does half the products on
// every wave.
//
// Bound: the matrix pipe (64 cycles per f64 MFMA, 32 per f32; a loop of
// products alone runs at 74.5 / 154 TF/s).  Element loads spent a quarter of
// the time on addresses, masks and register staging that the pipe waited
// for.  32 problems, TF/s before -> now: dense 1600^3 f64 48 -> 68, f32 93 ->
// 127; upper triangle times 1600 x 3200 f64 45 -> 60, f32 95 -> 117; rank-256
// update of 1344^2 f64 40 -> 57, f32 76 -> 100.
// ------------------------------------------------------------------------
template <typename T, int BM, int BN>
struct DmaTile {
  static constexpr int VE = 16 / (int)sizeof(T);            // entries per 16 bytes
  static constexpr int BK = 128 / (int)sizeof(T);
  static constexpr int KQ = BK / 4;                         // k per lane group
  static constexpr int RPI = 1024 / (BM * (int)sizeof(T));  // k rows per A instruction
  static constexpr int kPadA = sizeof(T) == 8 ? 0 : (BM == 128 ? 32 : 64);
  static constexpr int kRowGroup = 1024 + kPadA;
  static constexpr int kBytesA = BK / RPI * kRowGroup;
  static constexpr int kBytesB = BN * 128;
  static constexpr int NA = BK / RPI / 4, NB = BN / 32;     // instructions per wave and chunk
  static constexpr int H = BM / 64, HN = BN / 64;
  static __device__ __forceinline__ int a_row(int k) {
    return k / RPI * kRowGroup + (k % RPI) * (BM * (int)sizeof(T));
  }
};

// One chunk: the products of the stage cur, the DMA of the next chunk into
// nxt.  The two are restrict so that the reads do not wait for the DMA.  HM,
// HN: 64-row and 64-column groups inside the problem.
template <typename T, int BM, int BN, int HM, int HN>
__device__ __forceinline__ void dma_chunk(const char* __restrict__ cur, char* __restrict__ nxt,
                                          const char* __restrict__ ga, const char* __restrict__ gb,
                                          const int64_t (&offa)[DmaTile<T, BM, BN>::NA],
                                          const int64_t (&offb)[DmaTile<T, BM, BN>::NB], bool issue_next, int wa, int wb,
                                          int fa, const int (&fb)[2],
                                          typename Mma<T>::acc (&acc)[BM / 64][2][BN / 32]) {
  using D = DmaTile<T, BM, BN>;
  typedef T vec2 __attribute__((ext_vector_type(2)));
  typedef T vecb __attribute__((ext_vector_type(D::VE)));
  if (issue_next) {
#pragma unroll
    for (int q = 0; q < D::NA; ++q)
      __builtin_amdgcn_global_load_lds((dma_src_t)(ga + offa[q]), (dma_dst_t)(nxt + wa + q * D::kRowGroup), 16, 0, 0);
#pragma unroll
    for (int q = 0; q < D::NB; ++q)
      __builtin_amdgcn_global_load_lds((dma_src_t)(gb + offb[q]), (dma_dst_t)(nxt + wb + q * 1024), 16, 0, 0);
  }
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    vecb b[2 * HN];
#pragma unroll
    for (int n = 0; n < 2 * HN; ++n) b[n] = *(const vecb*)(cur + fb[p] + (n >> 1) * 8192 + (n & 1) * 2048);
#pragma unroll
    for (int e = 0; e < D::VE; ++e) {
      vec2 a[HM];
#pragma unroll
      for (int h = 0; h < HM; ++h)
        a[h] = *(const vec2*)(cur + fa + D::a_row(D::VE * p + e) + h * 64 * (int)sizeof(T));
#pragma unroll
      for (int h = 0; h < HM; ++h)
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
          for (int n = 0; n < 2 * HN; ++n) acc[h][q][n] = Mma<T>::run(b[n][e], a[h][q], acc[h][q][n]);
    }
  }
}

template <typename T, int BM, int BN, int OCC>
__global__ __launch_bounds__(256, OCC) void k_gemm_dma(const GemmProb* __restrict__ probs, int nprob,
                                                       const int32_t* __restrict__ order) {
  using D = DmaTile<T, BM, BN>;
  using acc_t = typename Mma<T>::acc;
  typedef T vec2 __attribute__((ext_vector_type(2)));
  __shared__ __attribute__((aligned(1024))) char lds[2][D::kBytesA + D::kBytesB];
  const int wg = order ? order[xcd_swizzle(blockIdx.x, gridDim.x)] : xcd_swizzle(blockIdx.x, gridDim.x);
  const GemmProb P = probs[find_prob(probs, nprob, wg)];
  const TileCoord tc = tile_of<BM, BN>(P, wg);
  const int I0 = tc.I0, J0 = tc.J0, kb = tc.kb, ke = tc.ke;
  const int fl = P.flags;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave & 1, wn = wave >> 1;
  const int li = lane & 15, g = lane >> 4;
  acc_t acc[D::H][2][2 * D::HN];
#pragma unroll
  for (int h = 0; h < D::H; ++h)
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int n = 0; n < 2 * D::HN; ++n) acc[h][q][n] = acc_t{0, 0, 0, 0};

  // 64: the two 64-row groups are taken in reverse order (lower triangular A)
  const int flip = D::H == 2 && (fl & G_A_LO) && I0 + BM <= P.M ? 64 : 0;
  if (kb < ke) {
    const bool a_lu = fl & G_A_MLU, a_up = fl & G_A_MUP, b_lu = fl & G_B_MLU, b_up = fl & G_B_MUP;
    const bool a_lo = fl & G_A_MLO, b_lo = fl & G_B_MLO;
    // byte offsets of the lane's 16-byte pieces from the chunk's first row of
    // k (A) and first k (B); rows and columns past the problem re-read its
    // last ones (they only feed outputs that are not stored)
    int64_t offa[D::NA], offb[D::NB];
    const int64_t lda8 = (int64_t)P.lda * (int)sizeof(T), ldb8 = (int64_t)P.ldb * (int)sizeof(T);
    const int am = ((lane * D::VE) % BM) ^ flip, ak = (lane * D::VE) / BM;
#pragma unroll
    for (int q = 0; q < D::NA; ++q)
      offa[q] = ((wave * D::NA + q) * D::RPI + ak) * lda8 + (int64_t)min(I0 + am, P.M - D::VE) * (int)sizeof(T);
#pragma unroll
    for (int q = 0; q < D::NB; ++q) {
      const int n = 8 * (wave * D::NB + q) + (lane >> 3);
      offb[q] = min(J0 + n, P.N - 1) * ldb8 + 16 * ((lane & 7) ^ ((n >> 1) & 7));
    }
    const char* A = (const char*)P.A + kb * lda8;
    const char* B = (const char*)P.B + (int64_t)kb * (int)sizeof(T);
    // fragment addresses
    const int fa = D::a_row(D::KQ * g) + (32 * wm + 2 * li) * (int)sizeof(T);
    const int nb = 32 * wn + li;
    const int fb[2] = {D::kBytesA + nb * 128 + (((2 * g) ^ ((nb >> 1) & 7)) << 4),
                       D::kBytesA + nb * 128 + (((2 * g + 1) ^ ((nb >> 1) & 7)) << 4)};
    const int wa = wave * D::NA * D::kRowGroup, wb = D::kBytesA + wave * D::NB * 1024;
#pragma unroll
    for (int q = 0; q < D::NA; ++q)
      __builtin_amdgcn_global_load_lds((dma_src_t)(A + offa[q]), (dma_dst_t)(lds[0] + wa + q * D::kRowGroup), 16, 0, 0);
#pragma unroll
    for (int q = 0; q < D::NB; ++q)
      __builtin_amdgcn_global_load_lds((dma_src_t)(B + offb[q]), (dma_dst_t)(lds[0] + wb + q * 1024), 16, 0, 0);
    // chunks [k0, kend) with the first 64 HM rows and 64 HN columns
    int st = 0, k0 = kb;
    auto steps = [&](auto hm, auto hn, int kend) __attribute__((always_inline)) {
      for (; k0 < kend; k0 += D::BK) {
        __syncthreads();   // chunk k0 has landed; every wave is done with the other stage
        const bool ma = (a_lu || a_up || a_lo) && k0 + D::BK > I0 && k0 < I0 + BM;
        const bool mb = (b_lu || b_up || b_lo) && k0 + D::BK > J0 && k0 < J0 + BN;
        if (ma || mb) {
          if (ma)
            for (int i = tid; i < D::BK * BM; i += 256) {
              const int k = i / BM, m = i % BM;
              T* e = (T*)(lds[st] + D::a_row(k) + m * (int)sizeof(T));
              *e = select_op(*e, I0 + (m ^ flip), k0 + k, a_lu, a_up, a_lo, 1 << 30, 1 << 30);
            }
          if (mb)
            for (int i = tid; i < BN * D::BK; i += 256) {
              const int n = i / D::BK, k = i % D::BK;
              T* e = (T*)(lds[st] + D::kBytesA + n * 128 + (((k / D::VE) ^ ((n >> 1) & 7)) << 4)) + k % D::VE;
              *e = select_op(*e, k0 + k, J0 + n, b_lu, b_up, b_lo, 1 << 30, 1 << 30);
            }
          __syncthreads();
        }
        A += D::BK * lda8;
        B += 128;
        dma_chunk<T, BM, BN, decltype(hm)::value, decltype(hn)::value>(lds[st], lds[st ^ 1], A, B, offa, offb,
                                                                       k0 + D::BK < ke, wa, wb, fa, fb, acc);
        st ^= 1;
      }
    };
    using I1 = std::integral_constant<int, 1>;
    using I2 = std::integral_constant<int, D::H>;
    if constexpr (D::H == 2 && D::HN == 2) {
      // the second group takes part where it is inside the problem and, with
      // an upper A, from the k on that reaches its rows; with a lower A it
      // holds the tile's first rows and leaves when k has passed them
      const int k1 = I0 + 64 >= P.M ? ke : (fl & G_A_UP) ? min(ke, I0 + 64) : kb;
      const int k2 = flip ? min(ke, I0 + 64) : ke;
      if (J0 + 64 < P.N) {
        steps(I1{}, I2{}, k1);
        steps(I2{}, I2{}, k2);
        steps(I1{}, I2{}, ke);
      } else {
        steps(I1{}, I1{}, k1);
        steps(I2{}, I1{}, k2);
        steps(I1{}, I1{}, ke);
      }
    } else {
      steps(I2{}, I2{}, ke);
    }
  }

  // lane: rows r, r + 1 of the columns c + Mma::row(lane, v)
  gptr<T> C0 = (gptr<T>)P.C0;
  gmut<T> Dp = (gmut<T>)P.D;
  const bool has_c0 = fl & G_C0;
  const T sg = (fl & G_NEG) ? T(-1) : T(1);
  // whole pairs in one access where the addresses allow it
  const uintptr_t al = (uintptr_t)P.D | (uintptr_t)P.ldd * sizeof(T) |
                       (has_c0 ? (uintptr_t)P.C0 | (uintptr_t)P.ldc0 * sizeof(T) : 0);
  const bool vec = (al & (2 * sizeof(T) - 1)) == 0;
#pragma unroll
  for (int h = 0; h < D::H; ++h) {
    const int r = I0 + ((64 * h) ^ flip) + 32 * wm + 2 * li;
#pragma unroll
    for (int n = 0; n < 2 * D::HN; ++n) {
      const int c = J0 + 64 * (n >> 1) + 32 * wn + 16 * (n & 1);
      const int how = store_block(P, r - 2 * li, c, 32, 16);
      if (how == 0) continue;
      if (vec && how == 1) {
        vec2 cv[4];
        if (has_c0) {
#pragma unroll
          for (int v = 0; v < 4; ++v) cv[v] = *(gptr<vec2>)(C0 + (int64_t)(c + Mma<T>::row(lane, v)) * P.ldc0 + r);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          vec2 o = {sg * acc[h][0][n][v], sg * acc[h][1][n][v]};
          if (has_c0) o = vec2{o[0] + cv[v][0], o[1] + cv[v][1]};
          *(gmut<vec2>)(Dp + (int64_t)(c + Mma<T>::row(lane, v)) * P.ldd + r) = o;
        }
      } else {
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
          for (int q = 0; q < 2; ++q) {
            const int cc = c + Mma<T>::row(lane, v);
            if (!store_ok(fl, r + q, cc)) continue;
            T val = sg * acc[h][q][n][v];
            if (has_c0) val += C0[(int64_t)cc * P.ldc0 + r + q];
            Dp[(int64_t)cc * P.ldd + r + q] = val;
          }
      }
    }
  }
}

// ------------------------------------------------------------------------
// k_gemm_x3: the bf16 products on 256 x 256 tiles, one workgroup of 8 waves
// (2 x 4) per CU, each FP32 operand entry split once per tile.
//
// K advances in steps of 16.  Waves 0-3 stage A, waves 4-7 B: 16 entries per
// thread loaded into registers three steps ahead, split into hi and lo while
// the current step multiplies (two pairs of entries under each three
// products, so that both waves of a SIMD keep the matrix pipe busy), and
// written to the other of two LDS stages as bf16 in the fragments' layout,
// so that a fragment is one 16-byte read.  One barrier per step, placed
// before the last row block: the products of that block cover the reads of
// the next step's first fragments.  Wave (wm, wn) owns the 32-row blocks 64
// mi + 32 wm and the 32-column blocks 128 ni + 32 wn: a tile at the edge of
// the problem, or crossing the diagonal of a triangular A, does only the
// products of the 64-row groups that have any, on all eight waves alike.
//
// Bound: the matrix pipe, at the clock that the card holds under it.  32 dense
// products of 2048^2 x 4096 take 2.9 ms with the pipe busy for 76% of the cycles
// (about 2020 per 16-deep step, of which the products are 1536) at 1.43 GHz, or
// 1.57 GHz when they run for seconds (2.6 ms); the f64 and f32 kernels run at 2.38
// GHz.  That the clock falls points to power, which could not be read.  32
// problems, TF/s of FP32 products, the kernel that split every fragment it read
// (256 x 256 tiles) -> this one: dense 1600^3 225 -> 277, 2048^2 x 1024 325 -> 383,
// upper triangle times 1600 x 3200 230 -> 285, rank-256 update of 1344^2 104 -> 161.
// ------------------------------------------------------------------------
// LDS image of one 16-deep K step of one operand: row (column) r holds four
// 16-byte units, the hi halves of k 0-7 and 8-15, then the lo halves; four
// rows share 256 bytes, in which unit (r & 3) * 4 + u is stored at that index
// XOR ((r >> 2) & 3 | (r >> 4 & 1) << 2).  With it the fragment reads (32
// consecutive rows, one unit) and both operands' writes touch every bank of
// a 256-byte pass once.
__device__ __forceinline__ int x3_addr(int r, int u) {
  const int g = ((r >> 2) & 3) | (((r >> 4) & 1) << 2);
  return (r >> 2) * 256 + ((((r & 3) * 4 + u) ^ g) << 4);
}

struct X3Tile {
  int fl, I0, J0, kb, ke, M, N;
  int flip;   // 3: the tile's four 64-row groups are taken in reverse order (lower triangular A), else 0
};

__device__ __forceinline__ int x3_flip(const GemmProb& P, int I0) {
  return (P.flags & G_A_LO) && I0 + 256 <= P.M ? 3 : 0;
}

// State of one wave in the K loop.  ISA: the wave stages A (waves 0-3), else B.
template <bool SPLIT, bool ISA>
struct X3Wave {
  static constexpr int kStage = 32768, kB = 16384;
  typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
  const X3Tile& T;
  const float* X;
  int64_t ldx;
  char* lds;
  // Staging: a thread holds 16 entries of one operand's step.
  //   A (rows contiguous in memory): rows R, R + 1 at 8 consecutive k (8
  //     eight-byte loads; a wave load covers 512 contiguous bytes of one k);
  //   B (k contiguous): 4 consecutive k of 4 columns 16 apart (4 sixteen-byte
  //     loads; 4 lanes cover the 64 bytes of one column).
  int r0, q0;        // A: row R, first k;  B: first column, first k
  uint32_t ld4;
  uint32_t off[4];   // byte offsets of the lane's loads from the step's first element
  int wa[2];         // LDS write addresses
  int fa, fb;        // LDS fragment addresses (hi; lo at ^ 32)
  uint32_t hq[8], lq[8];
  bf16x8 ah[2], al[2], bh[2], bl[2];   // A of the current and the next 32-row block (slots mi & 1), both B blocks

  __device__ __forceinline__ X3Wave(const X3Tile& T_, const float* X_, int64_t ldx_, char* lds_, int lane, int w4, int wm,
                                    int wn)
      : T(T_), X(X_), ldx(ldx_), lds(lds_) {
    const int li = lane & 31, half = lane >> 5;
    ld4 = (uint32_t)ldx * 4u;
    // rows and columns past the problem re-read its last ones (they only feed
    // outputs that are not stored)
    if (ISA) {
      const int oct = w4 & 1, R = 128 * (w4 >> 1) + 2 * lane;
      r0 = T.I0 + R;
      q0 = 8 * oct;
      wa[0] = x3_addr(R, oct) ^ (T.flip << 12);   // 64 rows are 4 KiB
      wa[1] = x3_addr(R + 1, oct) ^ (T.flip << 12);
      off[0] = (uint32_t)(min(r0, T.M - 2) - T.I0) * 4u + 8u * oct * ld4;
    } else {
      const int nq = lane >> 2, kq = lane & 3;
      const int cb = 64 * w4 + ((nq & 3) | (((nq >> 3) & 1) << 2) | (((nq >> 2) & 1) << 3));
      r0 = T.J0 + cb;
      q0 = 4 * kq;
      wa[0] = kB + x3_addr(cb, kq >> 1) + (kq & 1) * 8;
      wa[1] = kB + x3_addr(cb + 16, kq >> 1) + (kq & 1) * 8;
#pragma unroll
      for (int i = 0; i < 4; ++i) off[i] = (uint32_t)(min(r0 + 16 * i, T.N - 1) - T.J0) * ld4 + 16u * kq;
    }
    fa = x3_addr(32 * wm + li, half);
    fb = kB + x3_addr(32 * wn + li, half);
  }
  // half j of a step's entries (A: 4 of the 8 k of both rows; B: 2 of the 4 columns)
  __device__ __forceinline__ void load(float (&s)[16], int k, int j) {
    const auto rs = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(ISA ? X + (int64_t)k * ldx + T.I0 : X + (int64_t)T.J0 * ldx + k), 0, 0xffffffffu, 0x00027000);
    if (ISA) {
#pragma unroll
      for (int i = 4 * j; i < 4 * j + 4; ++i) {
        const f32x2 v = __builtin_bit_cast(f32x2, __builtin_amdgcn_raw_buffer_load_b64(rs, off[0], i * ld4, 0));
        s[2 * i] = v[0];
        s[2 * i + 1] = v[1];
      }
    } else {
#pragma unroll
      for (int i = 2 * j; i < 2 * j + 2; ++i) {
        const f32x4 v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rs, off[i], 0, 0));
#pragma unroll
        for (int e = 0; e < 4; ++e) s[4 * i + e] = v[e];
      }
    }
  }
  // packed-triangle masks on the staged entries of step k (where it crosses the diagonal)
  __device__ __forceinline__ void mask(float (&s)[16], int k) {
    const int fl = T.fl;
    const bool lu = fl & (ISA ? G_A_MLU : G_B_MLU), up = fl & (ISA ? G_A_MUP : G_B_MUP),
               lo = fl & (ISA ? G_A_MLO : G_B_MLO);
    const int d0 = ISA ? T.I0 : T.J0;
    if (!(lu || up || lo) || k + 16 <= d0 || k >= d0 + 256) return;
    if (ISA) {
#pragma unroll
      for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          s[2 * i + j] = select_op(s[2 * i + j], r0 + j, k + q0 + i, lu, up, lo, 1 << 30, 1 << 30);
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          s[4 * i + e] = select_op(s[4 * i + e], k + q0 + e, r0 + 16 * i, lu, up, lo, 1 << 30, 1 << 30);
    }
  }
  // pair q (0 .. 7) of the staged entries split: hi and lo packed in hq[q], lq[q]
  __device__ __forceinline__ void split2(const float (&s)[16], int q) {
    // A: pair q = k 2(q & 3), + 1 of row q >> 2;  B: k 2(q & 1), + 1 of column q >> 1
    const float x0 = ISA ? s[4 * (q & 3) + (q >> 2)] : s[2 * q], x1 = ISA ? s[4 * (q & 3) + 2 + (q >> 2)] : s[2 * q + 1];
    const bf16x2 hv = __builtin_convertvector((f32x2{x0, x1}), bf16x2);
    hq[q] = __builtin_bit_cast(uint32_t, hv);
    if (SPLIT) {
      const bf16x2 lv = __builtin_convertvector((f32x2{x0 - (float)hv[0], x1 - (float)hv[1]}), bf16x2);
      lq[q] = __builtin_bit_cast(uint32_t, lv);
    }
  }
  // writes of the split entries: A row j, B columns j and j + 2 ... (pairs 4j .. 4j + 3)
  __device__ __forceinline__ void put(int st, int j) {
    char* base = lds + st * kStage;
    if (ISA) {
      *(u32x4*)(base + wa[j]) = u32x4{hq[4 * j], hq[4 * j + 1], hq[4 * j + 2], hq[4 * j + 3]};
      if (SPLIT) *(u32x4*)(base + (wa[j] ^ 32)) = u32x4{lq[4 * j], lq[4 * j + 1], lq[4 * j + 2], lq[4 * j + 3]};
    } else {
#pragma unroll
      for (int i = 2 * j; i < 2 * j + 2; ++i) {
        *(u32x2*)(base + wa[i & 1] + (i >> 1) * 2048) = u32x2{hq[2 * i], hq[2 * i + 1]};
        if (SPLIT) *(u32x2*)(base + (wa[i & 1] ^ 32) + (i >> 1) * 2048) = u32x2{lq[2 * i], lq[2 * i + 1]};
      }
    }
  }
  __device__ __forceinline__ void read_a(int mi, int st) {
    ah[mi & 1] = *(const bf16x8*)(lds + st * kStage + mi * 4096 + fa);
    if (SPLIT) al[mi & 1] = *(const bf16x8*)(lds + st * kStage + mi * 4096 + (fa ^ 32));
  }
  __device__ __forceinline__ void read_b(int ni, int st) {
    bh[ni] = *(const bf16x8*)(lds + st * kStage + ni * 8192 + fb);
    if (SPLIT) bl[ni] = *(const bf16x8*)(lds + st * kStage + ni * 8192 + (fb ^ 32));
  }
  __device__ __forceinline__ void sync() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  }
  // Body of step k (fragments in stage st): its products by 32-row block,
  // with step k + 16 split and staged into stage st ^ 1 under the first ones
  // (free: every wave waited for its last reads of it before the last
  // barrier), step k + 48 then loaded into the same registers, and after the
  // barrier before the last row block the first fragments of step k + 16
  // read.  MB x NB: the tile's 64-row and 128-column groups inside the
  // problem.
  template <int MB, int NB>
  __device__ __forceinline__ void body(int k, int klast, int st, float (&s)[16], f32x16 (&acc)[4][2]) {
    constexpr int H = MB > 1 ? MB / 2 : 1;   // row blocks that carry the split
    mask(s, k + 16);
#pragma unroll
    for (int mi = 0; mi < MB; ++mi) {
      if (mi == MB - 1 && MB > 1) {
        if (MB <= 2) {
          put(st ^ 1, 0);
          put(st ^ 1, 1);
        }
        sync();
        if ((MB & 1) == 0) read_a(0, st ^ 1);
      }
      if (mi + 1 < MB) read_a(mi + 1, st);
      if (mi < H) {
#pragma unroll
        for (int q = 8 * mi / H; q < 8 * (mi + 1) / H; ++q) split2(s, ISA ? (q >> 1) + 4 * (q & 1) : q);
      }
      if (MB == 1 || (mi == H && MB > 2)) {
        put(st ^ 1, 0);
        put(st ^ 1, 1);
      }
      if (mi == H || MB == 1) {
        load(s, min(k + 48, klast), 0);
        load(s, min(k + 48, klast), 1);
      }
      const bf16x8 yh = ah[mi & 1], yl = al[mi & 1];
      if (SPLIT) {
#pragma unroll
        for (int ni = 0; ni < NB; ++ni)
          acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bl[ni], yh, acc[mi][ni], 0, 0, 0);
#pragma unroll
        for (int ni = 0; ni < NB; ++ni)
          acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bh[ni], yl, acc[mi][ni], 0, 0, 0);
      }
#pragma unroll
      for (int ni = 0; ni < NB; ++ni)
        acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bh[ni], yh, acc[mi][ni], 0, 0, 0);
      if (mi < H) {
#pragma unroll
        for (int q = 0; q < 3 * NB; ++q) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 16 / H / NB, 0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    if (MB == 1) sync();
#pragma unroll
    for (int ni = 0; ni < NB; ++ni) read_b(ni, st ^ 1);
    if (MB & 1) read_a(0, st ^ 1);
  }
  // K steps [k, kend) with the first 64 MB rows
  template <int MB, int NB>
  __device__ __forceinline__ void steps(int& k, int kend, float (&s0)[16], float (&s1)[16], f32x16 (&acc)[4][2]) {
    const int klast = T.ke - 16;
    for (; k < kend; k += 32) {
      body<MB, NB>(k, klast, 0, s1, acc);
      body<MB, NB>(k + 16, klast, 1, s0, acc);
    }
  }
  template <int NB>
  __device__ __forceinline__ void run(f32x16 (&acc)[4][2]) {
    float s0[16], s1[16];
    // the first three steps on the way, the first staged, its first fragments read
    load(s0, T.kb, 0);
    load(s0, T.kb, 1);
    load(s1, T.kb + 16, 0);
    load(s1, T.kb + 16, 1);
    mask(s0, T.kb);
#pragma unroll
    for (int q = 0; q < 8; ++q) split2(s0, q);
    put(0, 0);
    put(0, 1);
    load(s0, T.kb + 32, 0);
    load(s0, T.kb + 32, 1);
    sync();
    read_a(0, 0);
#pragma unroll
    for (int ni = 0; ni < NB; ++ni) read_b(ni, 0);
    // 64-row groups inside the problem; with an upper A a group joins when k
    // reaches its rows, with a lower A (groups in reverse order) the last
    // one leaves when k passes them
    const int mb = (min(T.M - T.I0, 256) + 63) >> 6;
    const int up = T.fl & G_A_UP ? T.I0 : -256;
    int k = T.kb;
    steps<1, NB>(k, min(T.ke, mb > 1 ? up + 64 : T.ke), s0, s1, acc);
    steps<2, NB>(k, min(T.ke, mb > 2 ? up + 128 : T.ke), s0, s1, acc);
    steps<3, NB>(k, min(T.ke, mb > 3 ? up + 192 : T.ke), s0, s1, acc);
    steps<4, NB>(k, T.flip ? min(T.ke, T.I0 + 64) : T.ke, s0, s1, acc);
    steps<3, NB>(k, min(T.ke, T.I0 + 128), s0, s1, acc);
    steps<2, NB>(k, min(T.ke, T.I0 + 192), s0, s1, acc);
    steps<1, NB>(k, T.ke, s0, s1, acc);
  }
  __device__ __forceinline__ void tile(f32x16 (&acc)[4][2]) {
    if (T.N - T.J0 > 128) run<2>(acc);
    else run<1>(acc);
  }
};

template <bool SPLIT>
__global__ __launch_bounds__(512, 2) void k_gemm_x3(const GemmProb* __restrict__ probs, int nprob,
                                                    const int32_t* __restrict__ order) {
  __shared__ __attribute__((aligned(256))) char lds[2 * X3Wave<SPLIT, true>::kStage];
  const int wg = order ? order[xcd_swizzle(blockIdx.x, gridDim.x)] : xcd_swizzle(blockIdx.x, gridDim.x);
  int pi = find_prob(probs, nprob, wg);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;
  f32x16 acc[4][2];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;
  {
    const GemmProb& P = probs[pi];
    const TileCoord tc = tile_of<256, 256>(P, wg);
    if (tc.kb < tc.ke) {
      const X3Tile T{P.flags, tc.I0, tc.J0, tc.kb, tc.ke, P.M, P.N, x3_flip(P, tc.I0)};
      if (wave < 4) {
        X3Wave<SPLIT, true> W(T, (const float*)P.A, P.lda, lds, lane, wave, wm, wn);
        W.tile(acc);
      } else {
        X3Wave<SPLIT, false> W(T, (const float*)P.B, P.ldb, lds, lane, wave - 4, wm, wn);
        W.tile(acc);
      }
    }
  }
  // the record is read again for the epilogue instead of being held in
  // scalar registers through the K loop
  asm volatile("" : "+s"(pi));
  const GemmProb P = probs[pi];
  const TileCoord tc = tile_of<256, 256>(P, wg);
  store_tile32<4, 2, 64, 128>(P, acc, tc.I0 + 32 * wm, tc.J0 + 32 * wn, lane, x3_flip(P, tc.I0));
}

// mode: 0 = 64 x 64 tiles, 1 = 128 x 128 tiles, 2 = 256 x 128 tiles (bf16 only),
// 3 = 128 x 128 tiles with direct LDS loads (bf16 only; otherwise as 1),
// 4 = 256 x 256 tiles on 8 waves (bf16 only; otherwise as 1),
// -1 = f64 / f32 operands that are not 16-byte aligned (64 x 64 tiles, element loads)
void launch_gemm(int dtype, int mode, const GemmProb* probs, int nprob, int nwg, hipStream_t s,
                 const int32_t* order) {
  if (nwg <= 0 || nprob <= 0) return;
  const dim3 g(nwg), b(256);
  if (dtype <= 1) {
    if (mode < 0) {
      if (dtype == 0) hipLaunchKernelGGL(k_gemm_std<double>, g, b, 0, s, probs, nprob, order);
      else hipLaunchKernelGGL(k_gemm_std<float>, g, b, 0, s, probs, nprob, order);
    } else if (mode >= 1) {
      if (dtype == 0) hipLaunchKernelGGL((k_gemm_dma<double, 128, 128, 2>), g, b, 0, s, probs, nprob, order);
      else hipLaunchKernelGGL((k_gemm_dma<float, 128, 128, 2>), g, b, 0, s, probs, nprob, order);
    } else {
      if (dtype == 0) hipLaunchKernelGGL((k_gemm_dma<double, 64, 64, 2>), g, b, 0, s, probs, nprob, order);
      else hipLaunchKernelGGL((k_gemm_dma<float, 64, 64, 2>), g, b, 0, s, probs, nprob, order);
    }
    return;
  }
  const bool split = dtype == 2;
  switch (mode) {
    case 4:
      if (split) hipLaunchKernelGGL((k_gemm_x3<true>), g, dim3(512), 0, s, probs, nprob, order);
      else hipLaunchKernelGGL((k_gemm_x3<false>), g, dim3(512), 0, s, probs, nprob, order);
      break;
    case 3:
      if (split) hipLaunchKernelGGL(k_gemm_dl<true>, g, b, 0, s, probs, nprob, order);
      else hipLaunchKernelGGL(k_gemm_dl<false>, g, b, 0, s, probs, nprob, order);
      break;
    case 2:
      if (split) hipLaunchKernelGGL((k_gemm_bf16<true, 256, 128, 1, 2>), g, b, 0, s, probs, nprob, order);
      else hipLaunchKernelGGL((k_gemm_bf16<false, 256, 128, 1, 2>), g, b, 0, s, probs, nprob, order);
      break;
    case 1:
      if (split) hipLaunchKernelGGL((k_gemm_bf16<true, 128, 128, 2>), g, b, 0, s, probs, nprob, order);
      else hipLaunchKernelGGL((k_gemm_bf16<false, 128, 128, 2>), g, b, 0, s, probs, nprob, order);
      break;
    default:
      if (split) hipLaunchKernelGGL((k_gemm_bf16<true, 64, 64, 2>), g, b, 0, s, probs, nprob, order);
      else hipLaunchKernelGGL((k_gemm_bf16<false, 64, 64, 2>), g, b, 0, s, probs, nprob, order);
      break;
  }
}

// tile edge (rows, columns) of a launch mode
void gemm_tile_shape(int dtype, int mode, int* bm, int* bn) {
  if (mode == 4 && dtype >= 2) { *bm = 256; *bn = 256; }
  else if (mode == 2 && dtype >= 2) { *bm = 256; *bn = 128; }
  else if (mode >= 1) { *bm = 128; *bn = 128; }
  else { *bm = 64; *bn = 64; }
}

}  // namespace ddps
