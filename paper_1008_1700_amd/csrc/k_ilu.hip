// Incomplete block factors (Section 3: D~ built from L~_i U~_i), read as
// ILU(0): L~_i unit lower and U~_i upper with the sparsity pattern of A_ii,
// so that (L~_i U~_i)(r, j) = a_rj wherever A_ii stores an entry.
//
// Storage.  The factor values sit at A's own CSR positions (fv, double):
// for global row r of block i, positions [lo[r], dg[r]) hold the strictly
// lower entries of L~ (unit diagonal implied), dg[r] the pivot and
// (dg[r], hi[r]) the rest of U~'s row (columns sorted; the positions outside
// [lo, hi) are coupling entries and are not touched).
//
// Order.  Both the factorisation and the forward solve need, for row r, the
// finished rows of its lower pattern; the backward solve the finished rows
// of its upper pattern.  The host groups each block's rows into levels
// (level of r = 1 + the largest level of the rows it refers to), so the rows
// of a level are independent; one workgroup runs one block level by level.
//
// Spikes.  G_i = D~_i^{-1} R~_i has 2t dense columns per block; one thread
// owns one column and runs both triangular solves down and up the block in
// row order (no barriers between waves: the columns are independent), in a
// row-major workspace so that a wave's 64 columns of one row are one coalesced
// access.  Only the spike tips (first and last t rows) are kept, transposed
// into the column-major tip store by an LDS-tiled copy.
#include "ddps_internal.h"

namespace ddps {
namespace {

constexpr int kIluThreads = 256;

// ILU(0) of every diagonal block, one workgroup per block.  IKJ form per
// row: for each k < r of its pattern, in increasing order, l_rk = a_rk / u_kk,
// then a_rj -= l_rk u_kj for every j > k stored in both row r and row k (the
// two sorted column lists are merged).  A pivot at or below the row's
// threshold is reported through `bad` (block << 40 | row, smallest wins).
__global__ __launch_bounds__(kIluThreads) void k_ilu0(const IluBlock* __restrict__ blocks,
                                                        const int32_t* __restrict__ lrows,
                                                        const int64_t* __restrict__ lptr,
                                                        const int64_t* __restrict__ lo, const int64_t* __restrict__ dg,
                                                        const int64_t* __restrict__ hi,
                                                        const int32_t* __restrict__ col,
                                                        const double* __restrict__ val, double* fv,
                                                        const double* __restrict__ thresh,
                                                        unsigned long long* __restrict__ bad) {
  const int bi = blockIdx.x;
  const IluBlock B = blocks[bi];
  for (int64_t r = B.s + threadIdx.x; r < B.s + B.n; r += blockDim.x)
    for (int64_t q = lo[r]; q < hi[r]; ++q) fv[q] = val[q];
  __syncthreads();
  for (int64_t lv = 0; lv < B.lnum; ++lv) {
    const int64_t a = lptr[B.lbeg + lv], e = lptr[B.lbeg + lv + 1];
    for (int64_t idx = a + threadIdx.x; idx < e; idx += blockDim.x) {
      const int64_t r = lrows[idx];
      const int64_t rdg = dg[r], rhi = hi[r];
      for (int64_t q = lo[r]; q < rdg; ++q) {
        const int64_t k = col[q];
        const int64_t kdg = dg[k], khi = hi[k];
        const double l = fv[q] / fv[kdg];
        fv[q] = l;
        int64_t w = q + 1;
        for (int64_t u = kdg + 1; u < khi && w < rhi; ++u) {
          const int32_t j = col[u];
          while (w < rhi && col[w] < j) ++w;
          if (w < rhi && col[w] == j) fv[w] -= l * fv[u];
        }
      }
      const double piv = fv[rdg];
      if (!(fabs(piv) > thresh[B.vbase + (r - B.s)]))
        atomicMin(bad, ((unsigned long long)bi << 40) | (unsigned long long)r);
    }
    __syncthreads();
  }
}

// Spike columns of a batch of blocks: workgroup (x = position in the batch,
// y = chunk of 64 columns), one wave, a lane per column.  Column c < t is the
// left coupling column c (right-hand side C_i(:, c) on the block's first t
// rows, upper triangular: rows <= c), column c >= t the right coupling column
// c - t (B_i(:, c - t) on the last t rows, lower triangular: rows >= c - t).
// The right-hand sides come from the compact coupling store, one t x (t+1)
// pair per block (C_i at offset t, B_i at offset 0, leading dimension t).
//
// The rows of a column are a serial chain; what a row needs besides the row
// just finished is brought up before it.  The factor's rows are copied to LDS
// kChunk at a time (a lane per row), each row's entries split by their distance:
// entries up to kNear rows away are read from a ring of the last kNear rows in
// LDS a row early, the row just finished from a register, farther ones from the
// workspace kAhead rows early.  Rows with more than kNearMax or kFarMax of them
// are read in place.  Values are always taken as stored (rounded to T), and each
// row's entries in their stored order.
//
// Bound: one wave's instruction rate (a row is some 150 instructions), so the
// waves are made small and many; up to 16 share a CU's LDS.  2048 columns of 32
// blocks of 8192 rows take 5.9 ms, 24.1 ms with a load of every entry in the
// chain; of 512 blocks 47 and 77 ms.  Rows read in place, all of them in a
// 27-point stencil (13 entries a side), still gain from the smaller waves: a whole
// factorisation of 20 blocks of 3200 rows 20.0 ms, with every row in place and
// large waves 27.0, of 32 blocks of 8192 55.3 and 79.8 ms.
constexpr int kNear = 16, kAhead = 8, kNearMax = 2, kFarMax = 4, kChunk = 32;

template <typename T>
struct IluRows {
  int fk[2 * kChunk][kFarMax], nk[2 * kChunk][kNearMax], meta[2 * kChunk];
  double fv[2 * kChunk][kFarMax], nv[2 * kChunk][kNearMax], piv[2 * kChunk];
  T ring[kNear][64];
};

// One sweep over the rows row(s) = UP ? r1 - 1 - s : r0 + s, s < r1 - r0.
// SRC: what a row starts from, 0: zero, 1: the right-hand side src (column
// entry of row r at src[r]), rows with r < lo_ok or r > hi_ok zero, 2: the
// workspace row itself.  last: the value of the row finished before.
template <bool UP, int SRC, typename T>
__device__ __forceinline__ void ilu_column_sweep(IluRows<T>& L, int r0, int r1, int kmin,
                                                 const IluBlock& B, const int64_t* __restrict__ lo,
                                                 const int64_t* __restrict__ dg, const int64_t* __restrict__ hi,
                                                 const int32_t* __restrict__ col, const double* __restrict__ fv,
                                                 const T* __restrict__ src, int lo_ok, int hi_ok, T* W, unsigned t2,
                                                 T& last) {
  const int lane = threadIdx.x;
  const int len = r1 - r0;
  if (len <= 0) return;
  auto row = [&](int s) __attribute__((always_inline)) { return UP ? r1 - 1 - s : r0 + s; };
  // rows s .. s + kChunk - 1 to LDS, one per lane, from their entry ranges
  // [qa, qe) loaded before (those of the next rows are loaded here); more than
  // kWide entries: read in place
  constexpr int kWide = 8;
  int64_t qa = 0, qe = 0;
  auto range = [&](int s) __attribute__((always_inline)) {
    const int64_t R = B.s + row(min(s + (lane & (kChunk - 1)), len - 1));
    qa = UP ? dg[R] : lo[R];
    qe = UP ? hi[R] : dg[R];
  };
  auto stage = [&](int s) __attribute__((always_inline)) {
    int k[kWide];
    double v[kWide];
    const int64_t q0 = qa + (UP ? 1 : 0);
    const int cnt = (int)min(qe - q0, (int64_t)kWide + 1);
    const double pivot = UP ? fv[qa] : 0.0;
#pragma unroll
    for (int u = 0; u < kWide; ++u) {
      const int64_t q = u < cnt ? q0 + u : qa;   // qa: the pivot or an entry before it
      k[u] = col[q] - (int)B.s;
      v[u] = fv[q];
    }
    range(s + kChunk);
    __syncthreads();
    if (lane < kChunk && s + lane < len) {
      const int i = (s + lane) & (2 * kChunk - 1);
      const int r = row(s + lane);
      int nf = 0, nn = 0;
      bool slow = cnt > kWide;
#pragma unroll
      for (int u = 0; u < kWide; ++u) {
        if (u >= cnt || k[u] < kmin) continue;
        if ((UP ? k[u] - r : r - k[u]) <= kNear) {
          if (nn < kNearMax) {
            L.nk[i][nn] = k[u];
            L.nv[i][nn] = v[u];
          } else slow = true;
          ++nn;
        } else {
          if (nf < kFarMax) {
            L.fk[i][nf] = k[u];
            L.fv[i][nf] = v[u];
          } else slow = true;
          ++nf;
        }
      }
      for (int u = min(nf, kFarMax); u < kFarMax; ++u) L.fk[i][u] = r, L.fv[i][u] = 0.0;
      for (int u = min(nn, kNearMax); u < kNearMax; ++u) L.nk[i][u] = UP ? r + 1 : r - 1, L.nv[i][u] = 0.0;
      L.meta[i] = slow ? kFarMax + 1 : nf | nn << 8;
      if (UP) L.piv[i] = pivot;
    }
    __syncthreads();
  };
  struct Far {
    T w[kFarMax], src;
  };
  typedef int i32x4_t __attribute__((ext_vector_type(4)));
  static_assert(kFarMax == 4, "far rows are read as one piece");
  i32x4_t fk;   // far rows of the next fetch
  auto far_rows = [&](int s) __attribute__((always_inline)) {
    fk = *(const i32x4_t*)L.fk[min(s, len - 1) & (2 * kChunk - 1)];
  };
  auto fetch = [&](Far& F, int s) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < kFarMax; ++u) F.w[u] = W[(uint64_t)(unsigned)__builtin_amdgcn_readfirstlane(fk[u]) * t2 + lane];
    const int r = row(min(s, len - 1));
    if (SRC == 1) F.src = src[r];
    if (SRC == 2) F.src = W[(uint64_t)(unsigned)r * t2 + lane];
  };
  struct Rec {
    int nk[kNearMax], meta;
    double fv[kFarMax], nv[kNearMax], piv;
  };
  auto record = [&](Rec& C, int s) __attribute__((always_inline)) {
    const int i = min(s, len - 1) & (2 * kChunk - 1);
#pragma unroll
    for (int u = 0; u < kNearMax; ++u) C.nk[u] = L.nk[i][u], C.nv[u] = L.nv[i][u];
#pragma unroll
    for (int u = 0; u < kFarMax; ++u) C.fv[u] = L.fv[i][u];
    C.meta = L.meta[i];
    if (UP) C.piv = L.piv[i];
  };
  T near[2][kNearMax];   // ring values of the current row and the next
  auto read_near = [&](const Rec& C, T* w) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < kNearMax; ++u) w[u] = L.ring[C.nk[u] & (kNear - 1)][lane];
  };
  auto solve = [&](const Far& F, const Rec& C, const T* w, int s) __attribute__((always_inline)) {
    const int r = row(s);
    const int meta = __builtin_amdgcn_readfirstlane(C.meta), nf = meta & 255, nn = meta >> 8;
    const double b = SRC == 0 || (SRC == 1 && (r < lo_ok || r > hi_ok)) ? 0.0 : (double)F.src;
    double acc = b;
    auto far = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < kFarMax; ++u) acc -= C.fv[u] * (double)(u < nf ? F.w[u] : T(0));
    };
    if (!UP) far();
#pragma unroll
    for (int u = 0; u < kNearMax; ++u) acc -= C.nv[u] * (double)(u >= nn ? T(0) : C.nk[u] == (UP ? r + 1 : r - 1) ? last : w[u]);
    if (UP) far();
    if (nf > kFarMax) {
      const int64_t R = B.s + r, d = dg[R], q1 = UP ? hi[R] : d;
      acc = b;
#pragma unroll 1
      for (int64_t q = UP ? d + 1 : lo[R]; q < q1; ++q) {
        const int k = col[q] - (int)B.s;
        if (k >= kmin) acc -= fv[q] * (double)W[(uint64_t)(unsigned)k * t2 + lane];
      }
    }
    last = (T)(UP ? acc / C.piv : acc);
    W[(uint64_t)(unsigned)r * t2 + lane] = last;
    L.ring[r & (kNear - 1)][lane] = last;
  };
  range(0);
  stage(0);
  stage(kChunk);
  Far F[kAhead];
  Rec C[4];
#pragma unroll
  for (int u = 0; u < kAhead; ++u) {
    far_rows(u);
    fetch(F[u], u);
  }
  record(C[0], 0);
  record(C[1], 1);
  read_near(C[0], near[0]);
#pragma unroll 1
  for (int s = 0; s < len; s += kAhead) {
    if ((s & (kChunk - 1)) == 0 && s > 0) stage(s + kChunk);
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      record(C[(u + 2) % 4], s + u + 2);
      read_near(C[(u + 1) % 4], near[(u + 1) % 2]);
      far_rows(s + u + kAhead);
      if (s + u < len) solve(F[u], C[u % 4], near[u % 2], s + u);
      fetch(F[u], s + u + kAhead);
    }
  }
}

template <typename T>
__global__ __launch_bounds__(64) void k_ilu_spikes(const IluBlock* __restrict__ blocks,
                                                     const int32_t* __restrict__ batch, int t,
                                                     const T* __restrict__ rhs, const int64_t* __restrict__ lo,
                                                     const int64_t* __restrict__ dg,
                                                     const int64_t* __restrict__ hi,
                                                     const int32_t* __restrict__ col,
                                                     const double* __restrict__ fv, T* ws, int64_t slot_elems) {
  __shared__ __attribute__((aligned(16))) IluRows<T> L;
  const int c0 = blockIdx.y * 64;
  const int t2 = 2 * t;
  const int bi = batch[blockIdx.x];
  const IluBlock B = blocks[bi];
  const bool left = c0 < t;
  if (left ? !B.left : !B.right) return;
  T* W = ws + (int64_t)blockIdx.x * slot_elems + c0;
  const int64_t pt = (int64_t)t * t + t;
  const int n = (int)B.n;
  const int r0 = left ? 0 : n - t;   // rows above r0 stay zero in the forward solve
  const int j = (left ? c0 : c0 - t) + (int)threadIdx.x;
  // entry of row r in this lane's column: rows r0 .. r0 + t - 1
  const T* __restrict__ P = rhs + (int64_t)bi * pt + (left ? t : 0) + (int64_t)j * t - r0;
  T last = T(0);
  ilu_column_sweep<false, 1>(L, r0, r0 + t, r0, B, lo, dg, hi, col, fv, P, left ? r0 : r0 + j, left ? r0 + j : n, W,
                             t2, last);
  if (left) ilu_column_sweep<false, 0>(L, t, n, r0, B, lo, dg, hi, col, fv, P, 0, 0, W, t2, last);
  last = T(0);
  ilu_column_sweep<true, 2>(L, r0, n, 0, B, lo, dg, hi, col, fv, P, 0, 0, W, t2, last);
  if (!left) ilu_column_sweep<true, 0>(L, 0, r0, 0, B, lo, dg, hi, col, fv, P, 0, 0, W, t2, last);
}

// Tips of a batch: rows [0, t) of block i's spikes into tip part 2i - 1 and
// rows [n - t, n) into part 2i, each part t x 2t column-major (leading
// dimension t).  64 x 64 tiles through LDS: read along the workspace rows,
// written along the part's columns.  Columns of a coupling the block does
// not have (left of block 0, right of block p-1) are written as zeros.
template <typename T>
__global__ __launch_bounds__(kIluThreads) void k_ilu_tips(const IluBlock* __restrict__ blocks,
                                                            const int32_t* __restrict__ batch, int p, int t,
                                                            const T* __restrict__ ws, int64_t slot_elems,
                                                            T* __restrict__ tips) {
  __shared__ T tile[64][65];
  const int bi = batch[blockIdx.x];
  const IluBlock B = blocks[bi];
  const int part = blockIdx.y;   // 0: top rows, 1: bottom rows
  if (part == 0 ? bi == 0 : bi == p - 1) return;
  const int t2 = 2 * t;
  const int ct = t2 / 64;
  const int tr = blockIdx.z / ct, tc = blockIdx.z % ct;   // tile row (of t / 64), tile column
  const T* __restrict__ W = ws + (int64_t)blockIdx.x * slot_elems;
  const int64_t rbase = part == 0 ? 0 : B.n - t;
  const int64_t q = part == 0 ? 2 * (int64_t)bi - 1 : 2 * (int64_t)bi;
  T* __restrict__ D = tips + q * (int64_t)t2 * t;
  const int lx = threadIdx.x & 63, ly = threadIdx.x >> 6;   // 64 x 4 threads
  for (int rr = ly; rr < 64; rr += 4) {
    const int64_t r = rbase + (int64_t)tr * 64 + rr;
    const int c = tc * 64 + lx;
    const bool have = c < t ? B.left : B.right;
    tile[rr][lx] = have ? W[r * t2 + c] : T(0);
  }
  __syncthreads();
  for (int cc = ly; cc < 64; cc += 4) {
    const int c = tc * 64 + cc;
    const int64_t r = (int64_t)tr * 64 + lx;
    D[(int64_t)c * t + r] = tile[lx][cc];
  }
}

// D~^{-1} y for every block, in place on the padded vector (R columns,
// column stride ldy), for blocks that k_ilu_solve_lds cannot take: one
// workgroup of kSolveThreads per block, forward solve with L~ level by level,
// then backward with U~.  The solve is bound by the latency of its dependent
// loads (level list -> row -> entries -> vector), so each level-ordered slot
// carries its row's entry range (lq: [lo, dg) of the forward order, uq: [dg + 1,
// hi) of the backward one, pivot at uq.x - 1), read together with the row
// number, and a workgroup runs 16 waves; the R lanes of one row are adjacent.
// Entries are taken four at a time with their loads issued together (columns
// and values, then the vector entries), so a row costs three dependent loads,
// not two per entry.
constexpr int kSolveThreads = 1024;
constexpr int64_t kIluLds = 160 * 1024;   // LDS of a workgroup

// acc - sum over q in [q0, q1) of fv[q] * Yc[(col[q] - s) * R]
__device__ __forceinline__ double row_dot(double acc, int64_t q0, int64_t q1, const int32_t* __restrict__ col,
                                          const double* __restrict__ fv, const double* Yc, int64_t s, int R) {
  for (int64_t q = q0; q < q1; q += 4) {
    int64_t c[4];
    double v[4], x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool ok = q + u < q1;
      c[u] = ok ? ((int64_t)col[q + u] - s) * R : 0;
      v[u] = ok ? fv[q + u] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) x[u] = q + u < q1 ? Yc[c[u]] : 0.0;
#pragma unroll
    for (int u = 0; u < 4; ++u) acc -= v[u] * x[u];
  }
  return acc;
}
__global__ __launch_bounds__(kSolveThreads) void k_ilu_solve(const IluBlock* __restrict__ blocks,
                                                               const int32_t* __restrict__ lrows,
                                                               const int64_t* __restrict__ lptr,
                                                               const longlong2* __restrict__ lq,
                                                               const int32_t* __restrict__ urows,
                                                               const int64_t* __restrict__ uptr,
                                                               const longlong2* __restrict__ uq,
                                                               const int32_t* __restrict__ col,
                                                               const double* __restrict__ fv, double* y,
                                                               int64_t ldy, int R, double* __restrict__ yt) {
  const IluBlock B = blocks[blockIdx.x];
  // y: entry of global row r in column j at y[j * ldy + vbase + (r - s)].
  // The solves run on a row-major copy (yt + vbase * R, R entries per row),
  // so that the R lanes of a row read one stretch of R doubles.
  double* __restrict__ Yt = yt + B.vbase * R;
  const int64_t nR = B.n * R;
  for (int64_t w = threadIdx.x; w < nR; w += blockDim.x) {
    const int64_t r = w % B.n, j = w / B.n;
    Yt[r * R + j] = y[j * ldy + B.vbase + r];
  }
  __syncthreads();
  for (int64_t lv = 0; lv < B.lnum; ++lv) {
    const int64_t a = lptr[B.lbeg + lv], e = lptr[B.lbeg + lv + 1];
    for (int64_t w = threadIdx.x; w < (e - a) * R; w += blockDim.x) {
      const int64_t j = a + w / R;
      const int64_t r = lrows[j];
      const longlong2 qr = lq[j];
      double* __restrict__ Yc = Yt + (w % R);
      Yc[(r - B.s) * R] = row_dot(Yc[(r - B.s) * R], qr.x, qr.y, col, fv, Yc, B.s, R);
    }
    __syncthreads();
  }
  for (int64_t lv = 0; lv < B.unum; ++lv) {
    const int64_t a = uptr[B.ubeg + lv], e = uptr[B.ubeg + lv + 1];
    for (int64_t w = threadIdx.x; w < (e - a) * R; w += blockDim.x) {
      const int64_t j = a + w / R;
      const int64_t r = urows[j];
      const longlong2 qr = uq[j];
      double* __restrict__ Yc = Yt + (w % R);
      const double piv = fv[qr.x - 1];
      Yc[(r - B.s) * R] = row_dot(Yc[(r - B.s) * R], qr.x, qr.y, col, fv, Yc, B.s, R) / piv;
    }
    __syncthreads();
  }
  for (int64_t w = threadIdx.x; w < nR; w += blockDim.x) {
    const int64_t r = w % B.n, j = w / B.n;
    y[j * ldy + B.vbase + r] = Yt[r * R + j];
  }
}

// The same solves with one workgroup per block and right-hand side, for blocks
// whose vector fits in LDS.  A level is then a few LDS reads, the rows'
// arithmetic and a barrier.  What it reads from memory does not depend on the
// solution and is loaded D levels ahead into registers; it is stored in level
// order for that (k_ilu_pack), so that a wave reads consecutive pieces: read at
// the CSR positions, a level of 200 rows moves some 1500 cache lines to one CU
// and takes 1.07 us, packed 0.35 us.  Per slot of the level order
//   pat: the block-local columns of the first four entries (n, where the LDS
//        vector holds a zero, for entries the row does not have), the row, the
//        entry count, 16 bits each
//   val: two entries at slot j and two at slot n_all + j, then (backward) the
//        pivots
// Rows beyond the first NT of a level are loaded when they are due (from the CSR
// positions two loads more, which made levels of 2000 to 5000 rows slower than
// k_ilu_solve for one column: 93 and 88 us a solve, from here 79); entries beyond
// the fourth of a row are read in place.  Every row's sum is taken in the order of
// k_ilu_solve, so that both give the same bits.
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
typedef double f64x2_t __attribute__((ext_vector_type(2)));

__global__ __launch_bounds__(kIluThreads) void k_ilu_pack(const IluBlock* __restrict__ blocks, int64_t n_all,
                                                            const int32_t* __restrict__ lrows,
                                                            const longlong2* __restrict__ lq,
                                                            const int32_t* __restrict__ urows,
                                                            const longlong2* __restrict__ uq,
                                                            const int32_t* __restrict__ col,
                                                            const double* __restrict__ fv, IluPacked P) {
  const IluBlock B = blocks[blockIdx.y];
  const int64_t i = (int64_t)blockIdx.x * kIluThreads + threadIdx.x;
  if (i >= B.n) return;
  const int64_t j = B.s + i;
#pragma unroll
  for (int up = 0; up < 2; ++up) {
    const longlong2 q = up ? uq[j] : lq[j];
    const int64_t row = (up ? urows[j] : lrows[j]) - B.s, cnt = q.y - q.x;
    unsigned c[4];
    double v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      c[u] = u < cnt ? (unsigned)(col[q.x + u] - B.s) : (unsigned)B.n;
      v[u] = u < cnt ? fv[q.x + u] : 0.0;
    }
    u32x4_t* pat = (u32x4_t*)(up ? P.upat : P.lpat);
    f64x2_t* val = (f64x2_t*)(up ? P.uval : P.lval);
    pat[j] = u32x4_t{c[0] | c[1] << 16, c[2] | c[3] << 16, (unsigned)row | (unsigned)(cnt < 65535 ? cnt : 65535) << 16, 0u};
    val[j] = f64x2_t{v[0], v[1]};
    val[n_all + j] = f64x2_t{v[2], v[3]};
    if (up) P.piv[j] = fv[q.x - 1];
  }
}

template <bool UP, int NT>
__device__ __forceinline__ void ilu_sweep(double* Y, int64_t s, int n, int64_t n_all, int64_t num,
                                          const int64_t* __restrict__ ptr, const longlong2* __restrict__ rq,
                                          const int32_t* __restrict__ col, const double* __restrict__ fv,
                                          const u32x4_t* __restrict__ pat,
                                          const f64x2_t* __restrict__ val, const double* __restrict__ piv) {
  constexpr int D = 8;   // levels between loads and use
  struct Row {
    u32x4_t p;
    f64x2_t v[2];
    double piv;
  };
  const int tid = threadIdx.x, lane = tid & 63;
  rq += s;
  pat += s;
  val += s;
  piv += s;
  // the level pointers of 128 levels from l0 on sit in two registers of a wave
  auto offs = [&](int64_t l) __attribute__((always_inline)) { return (int)ptr[l < num ? l : num]; };
  int cur = offs(lane), nxt = offs(64 + lane);
  // first slot of level l0 + k, k < 128
  auto at = [&](int k) __attribute__((always_inline)) {
    const int a = __builtin_amdgcn_readlane(cur, k & 63), b = __builtin_amdgcn_readlane(nxt, k & 63);
    return (k < 64 ? a : b) - (int)s;
  };
  auto load = [&](Row& F, int j) __attribute__((always_inline)) {
    F.p = pat[j];
    F.v[0] = val[j];
    F.v[1] = val[n_all + j];
    if (UP) F.piv = piv[j];
  };
  auto fetch = [&](Row& F, int k) __attribute__((always_inline)) { load(F, min(at(k) + tid, n - 1)); };
  auto solve = [&](const Row& F, int j) __attribute__((always_inline)) {
    const int y = F.p.z & 0xffff, cnt = F.p.z >> 16;
    double acc = Y[y];
    const double x0 = Y[F.p.x & 0xffff], x1 = Y[F.p.x >> 16], x2 = Y[F.p.y & 0xffff], x3 = Y[F.p.y >> 16];
    acc -= F.v[0].x * x0;
    acc -= F.v[0].y * x1;
    acc -= F.v[1].x * x2;
    acc -= F.v[1].y * x3;
    if (cnt > 4) {
      const longlong2 q = rq[j];
#pragma unroll 1
      for (int64_t i = q.x + 4; i < q.y; ++i) acc -= fv[i] * Y[col[i] - s];
    }
    Y[y] = UP ? acc / F.piv : acc;
  };
  auto compute = [&](const Row& F, int k) __attribute__((always_inline)) {
    const int e = at(k + 1);
    int j = at(k) + tid;
    if (j < e) {
      solve(F, j);
#pragma unroll 1
      for (j += NT; j < e; j += NT) {
        Row G;
        load(G, j);
        solve(G, j);
      }
    }
  };
  Row F[D];
#pragma unroll
  for (int u = 0; u < D; ++u) fetch(F[u], u);
  int64_t l0 = 0;
#pragma unroll 1
  for (int64_t lv = 0; lv < num; lv += D) {
    if (lv - l0 == 64) {
      l0 = lv;
      cur = nxt;
      nxt = offs(l0 + 64 + lane);
    }
    const int k = (int)(lv - l0);
#pragma unroll
    for (int u = 0; u < D; ++u) {
      compute(F[u], k + u);
      fetch(F[u], k + u + D);
      // LDS writes done, then every wave; loads from memory stay in flight
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    }
  }
}

template <int NT>
__global__ __launch_bounds__(NT) void k_ilu_solve_lds(const IluBlock* __restrict__ blocks, int p, int64_t n_all,
                                                      const int64_t* __restrict__ lptr,
                                                      const longlong2* __restrict__ lq,
                                                      const int64_t* __restrict__ uptr,
                                                      const longlong2* __restrict__ uq,
                                                      const int32_t* __restrict__ col,
                                                      const double* __restrict__ fv, IluPacked P, double* y,
                                                      int64_t ldy) {
  extern __shared__ __attribute__((aligned(16))) double Y[];
  const IluBlock B = blocks[blockIdx.x % p];
  double* __restrict__ yc = y + (int64_t)(blockIdx.x / p) * ldy + B.vbase;
  const int n = (int)B.n;
  for (int r = threadIdx.x; r < n; r += NT) Y[r] = yc[r];
  if (threadIdx.x == 0) Y[n] = 0.0;
  __syncthreads();
  ilu_sweep<false, NT>(Y, B.s, n, n_all, B.lnum, lptr + B.lbeg, lq, col, fv, (const u32x4_t*)P.lpat,
                       (const f64x2_t*)P.lval, P.piv);
  ilu_sweep<true, NT>(Y, B.s, n, n_all, B.unum, uptr + B.ubeg, uq, col, fv, (const u32x4_t*)P.upat,
                      (const f64x2_t*)P.uval, P.piv);
  __syncthreads();
  for (int r = threadIdx.x; r < n; r += NT) yc[r] = Y[r];
}

}  // namespace

void ilu_factor(int p, const IluBlock* blocks, const int32_t* lrows, const int64_t* lptr, const int64_t* lo,
                const int64_t* dg, const int64_t* hi, const int32_t* col, const double* val, double* fv,
                const double* thresh, unsigned long long* bad, hipStream_t s) {
  hipLaunchKernelGGL(k_ilu0, dim3(p), dim3(kIluThreads), 0, s, blocks, lrows, lptr, lo, dg, hi, col, val, fv, thresh,
                     bad);
}

void ilu_spikes(int dtype, int nb, const IluBlock* blocks, const int32_t* batch, int p, int t, const void* rhs,
                const int64_t* lo, const int64_t* dg, const int64_t* hi, const int32_t* col, const double* fv,
                void* ws, int64_t slot_elems, void* tips, hipStream_t s) {
  if (nb <= 0) return;
  const dim3 g1((unsigned)nb, (unsigned)(2 * t / 64));
  const dim3 g2((unsigned)nb, 2u, (unsigned)((t / 64) * (2 * t / 64)));
  if (dtype == 0) {
    hipLaunchKernelGGL(k_ilu_spikes<double>, g1, dim3(64), 0, s, blocks, batch, t, (const double*)rhs, lo, dg,
                       hi, col, fv, (double*)ws, slot_elems);
    hipLaunchKernelGGL(k_ilu_tips<double>, g2, dim3(kIluThreads), 0, s, blocks, batch, p, t, (const double*)ws,
                       slot_elems, (double*)tips);
  } else {
    hipLaunchKernelGGL(k_ilu_spikes<float>, g1, dim3(64), 0, s, blocks, batch, t, (const float*)rhs, lo, dg,
                       hi, col, fv, (float*)ws, slot_elems);
    hipLaunchKernelGGL(k_ilu_tips<float>, g2, dim3(kIluThreads), 0, s, blocks, batch, p, t, (const float*)ws,
                       slot_elems, (float*)tips);
  }
}

int64_t ilu_packed_bytes(int64_t n_all) { return n_all * (2 * 16 + 4 * 16 + 8); }

IluPacked ilu_packed(void* buf, int64_t n_all) {
  char* c = (char*)buf;
  return {c, c + 16 * n_all, c + 32 * n_all, c + 64 * n_all, (double*)(c + 96 * n_all)};
}

bool ilu_packs(int64_t nmax) { return (nmax + 1) * (int64_t)sizeof(double) <= kIluLds; }

void ilu_pack(int p, int64_t nmax, int64_t n_all, const IluBlock* blocks, const int32_t* lrows, const void* lq,
              const int32_t* urows, const void* uq, const int32_t* col, const double* fv, IluPacked P,
              hipStream_t s) {
  hipLaunchKernelGGL(k_ilu_pack, dim3((unsigned)((nmax + kIluThreads - 1) / kIluThreads), (unsigned)p),
                     dim3(kIluThreads), 0, s, blocks, n_all, lrows, (const longlong2*)lq, urows,
                     (const longlong2*)uq, col, fv, P);
}

void ilu_solve_packed(int p, int64_t nmax, int64_t n_all, int wmax, const IluBlock* blocks, const int64_t* lptr,
                      const void* lq, const int64_t* uptr, const void* uq, const int32_t* col, const double* fv,
                      IluPacked P, double* y, int64_t ldy, int R, hipStream_t s) {
  const size_t lds = (size_t)(nmax + 1) * sizeof(double);
#define DDPS_ILU_LDS(NT)                                                                                              \
  hipLaunchKernelGGL(k_ilu_solve_lds<NT>, dim3((unsigned)(p * R)), dim3(NT), lds, s, blocks, p, n_all, lptr,        \
                     (const longlong2*)lq, uptr, (const longlong2*)uq, col, fv, P, y, ldy)
  if (wmax <= 64) DDPS_ILU_LDS(64);
  else if (wmax <= 256) DDPS_ILU_LDS(256);
  else DDPS_ILU_LDS(512);
#undef DDPS_ILU_LDS
}

void ilu_solve(int p, const IluBlock* blocks, const int32_t* lrows, const int64_t* lptr, const void* lq,
               const int32_t* urows, const int64_t* uptr, const void* uq, const int32_t* col, const double* fv,
               double* y, int64_t ldy, int R, double* yt, hipStream_t s) {
  hipLaunchKernelGGL(k_ilu_solve, dim3(p), dim3(kSolveThreads), 0, s, blocks, lrows, lptr, (const longlong2*)lq, urows,
                     uptr, (const longlong2*)uq, col, fv, y, ldy, R, yt);
}

}  // namespace ddps
