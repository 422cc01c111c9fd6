// Grouped tile GEMV for 1..8 right-hand sides: y_out = y_in +/- A x.
//
// Used by every HBM-bound stream of the solve phase: the block sweeps of
// step 6.1 (triangular inverse tiles and coupling tiles), the reduced-matrix
// product of 6.3 (spike-tip rows, masked to the index set c) and the
// retrieval z = g - G z^ of 6.5.  Each workgroup owns 64 consecutive output
// rows of one problem; its 4 waves take interleaved columns, so one wave
// load reads 64 consecutive rows of one column (512 B for f64 matrices), and
// the vector entries are wave-uniform (scalar loads).  Triangular problems
// clip the column range per 64-row slab and mask the diagonal slab.
#include "ddps_internal.h"
#include "krylov_device.h"

namespace ddps {

template <typename T>
using gptr = const T __attribute__((address_space(1)))*;

// Problem of workgroup wg of nwg (an argument: gridDim would bring 256 bytes of
// hidden ones with each launch, 0.5 to 1 us of host time in a chain of short
// ones).  Most launches hold problems of equal size, where the proportional guess
// is right and the dependent loads of a search (a microsecond or more of a short
// kernel) are saved.
__device__ __forceinline__ int find_gemv(const GemvProb* __restrict__ probs, int nprob, int wg, int nwg) {
  const int gs = min((int)(((float)wg + 0.5f) * ((float)nprob * __builtin_amdgcn_rcpf((float)nwg))), nprob - 1);
  const int b0 = probs[gs].wg0, b1 = gs + 1 < nprob ? probs[gs + 1].wg0 : nwg;
  if (b0 <= wg && wg < b1) return gs;
  int lo = 0, hi = nprob - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (probs[mid].wg0 <= wg) lo = mid; else hi = mid - 1;
  }
  return lo;
}

template <typename T, int R>
__global__ __launch_bounds__(256) void k_gemv(const GemvProb* __restrict__ probs, int nprob, int nwg,
                                              int64_t ldx, int64_t ldy,
                                              const double* __restrict__ dotv,
                                              double* __restrict__ partial,
                                              const int32_t* __restrict__ stop) {
  __shared__ double red[4][64][R];
  if (stop) {
    bool all = true;
#pragma unroll
    for (int j = 0; j < R; ++j) all &= stop[j] != KS_RUNNING;
    if (all) return;
  }
  const int wg = blockIdx.x;
  const GemvProb& Pg = probs[find_gemv(probs, nprob, wg, nwg)];
  const GemvProb P = Pg;
  const int r0 = (wg - P.wg0) * 64;
  int cb = P.cb, ce = P.ce;
  if (P.tri == 1) ce = min(ce, r0 + 64);
  if (P.tri == 2) cb = max(cb, r0);
  const int tid = threadIdx.x, lane = tid & 63;
  const int g = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r = r0 + lane;
  const int fl = P.flags;
  const bool mlu = fl & V_A_MLU, mup = fl & V_A_MUP, mlo = fl & V_A_MLO;
  const T* __restrict__ A = (const T*)P.A + r;
  const int64_t lda = P.lda;
  const int split = P.split;

  double acc[R];
#pragma unroll
  for (int j = 0; j < R; ++j) acc[j] = 0.0;

  auto xval = [&](int c, int j) -> double {
    return c < split ? P.x1[c + j * ldx] : P.x2[(c - split) + j * ldx];
  };
  int c = cb + g;
  // four independent columns per step for memory-level parallelism
  for (; c + 12 < ce; c += 16) {
    T a[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) a[u] = A[(int64_t)(c + 4 * u) * lda];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int cc = c + 4 * u;
      double av = (double)a[u];
      if (mlu) av = r > cc ? av : (r == cc ? 1.0 : 0.0);
      if (mup) av = r <= cc ? av : 0.0;
      if (mlo) av = r >= cc ? av : 0.0;
#pragma unroll
      for (int j = 0; j < R; ++j) acc[j] += av * xval(cc, j);
    }
  }
  for (; c < ce; c += 4) {
    double av = (double)A[(int64_t)c * lda];
    if (mlu) av = r > c ? av : (r == c ? 1.0 : 0.0);
    if (mup) av = r <= c ? av : 0.0;
    if (mlo) av = r >= c ? av : 0.0;
#pragma unroll
    for (int j = 0; j < R; ++j) acc[j] += av * xval(c, j);
  }
#pragma unroll
  for (int j = 0; j < R; ++j) red[g][lane][j] = acc[j];
  __syncthreads();
  if (tid < 64) {
    double dot[R], dd[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
      double s = red[0][lane][j] + red[1][lane][j] + red[2][lane][j] + red[3][lane][j];
      if (fl & V_MASK) s *= P.mask[r];
      if (fl & V_NEG) s = -s;
      if (fl & V_YIN) s += P.yin[r + j * ldy];
      if (r >= P.row_skip) P.yout[r + j * ldy] = s;
      dot[j] = (fl & V_DOT) ? dotv[P.dot_off + r + j * ldy] * s : 0.0;
      dd[j] = (fl & V_DOT2) ? s * s : 0.0;
    }
    if (fl & V_DOT) {
#pragma unroll
      for (int j = 0; j < R; ++j) {
        double v = dot[j], w = dd[j];
        for (int off = 32; off > 0; off >>= 1) {
          v += __shfl_xor(v, off, 64);
          w += __shfl_xor(w, off, 64);
        }
        if (lane == 0) {
          partial[((int64_t)wg * R + j) * 2 + 0] = v;
          partial[((int64_t)wg * R + j) * 2 + 1] = w;
        }
      }
    }
  }
}

// ------------------------------------------------------------------------
// Wide-load form of k_gemv for 16-byte aligned problems and many right-hand
// sides: a lane reads VEC
// consecutive rows of one column in one 16-byte load, so one wave load
// covers 64 rows of VEC columns (1 KB) instead of 64 rows of one column.
// The VEC column slots of a wave are summed by lane shuffles, the 4 waves
// through LDS; epilogue, flags and partial sums as in k_gemv.  U loads are in
// flight per lane.
// ------------------------------------------------------------------------
template <typename T, int R, int U>
__global__ __launch_bounds__(256) void k_gemv_w(const GemvProb* __restrict__ probs, int nprob, int nwg,
                                                int64_t ldx, int64_t ldy,
                                                const double* __restrict__ dotv,
                                                double* __restrict__ partial,
                                                const int32_t* __restrict__ stop) {
  constexpr int VEC = 16 / sizeof(T);   // rows per lane
  constexpr int LPC = 64 / VEC;         // lanes per column
  constexpr int STEP = 4 * VEC;         // columns per round of the workgroup
  typedef T vec_t __attribute__((ext_vector_type(VEC)));
  __shared__ double red[4][64][R];
  if (stop) {
    bool all = true;
#pragma unroll
    for (int j = 0; j < R; ++j) all &= stop[j] != KS_RUNNING;
    if (all) return;
  }
  const int wg = blockIdx.x;
  const GemvProb& Pg = probs[find_gemv(probs, nprob, wg, nwg)];
  const GemvProb P = Pg;
  const int r0 = (wg - P.wg0) * 64;
  int cb = P.cb, ce = P.ce;
  if (P.tri == 1) ce = min(ce, r0 + 64);
  if (P.tri == 2) cb = max(cb, r0);
  const int tid = threadIdx.x, lane = tid & 63;
  const int g = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = lane / LPC;             // column slot of this lane
  const int rl = (lane % LPC) * VEC;    // first local row of this lane
  const int fl = P.flags;
  const bool mlu = fl & V_A_MLU, mup = fl & V_A_MUP, mlo = fl & V_A_MLO;
  const T* __restrict__ A = (const T*)P.A + r0 + rl;
  const int64_t lda = P.lda;
  const int split = P.split;

  double acc[VEC][R];
#pragma unroll
  for (int e = 0; e < VEC; ++e)
#pragma unroll
    for (int j = 0; j < R; ++j) acc[e][j] = 0.0;

  // many right-hand sides: the vector entries of each round of U STEP
  // columns are staged once per workgroup in LDS (double-buffered), so a
  // lane reads its columns' R entries as 16-byte LDS reads instead of R
  // separate global loads
  constexpr int RC = U * STEP;   // columns per round
  __shared__ __attribute__((aligned(16))) double xs[2][RC][R];
  int buf = 0;
  for (int c0 = cb; c0 < ce; c0 += RC) {
    for (int i = tid; i < RC * R; i += 256) {
      const int cc = c0 + i / R, j = i % R;
      xs[buf][i / R][j] = cc < ce ? (cc < split ? P.x1[cc + j * ldx] : P.x2[(cc - split) + j * ldx]) : 0.0;
    }
    __syncthreads();
    vec_t a[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int cc = c0 + g * VEC + q + u * STEP;
      a[u] = cc < ce ? *(const vec_t*)(A + (int64_t)cc * lda) : vec_t{};
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int cl = g * VEC + q + u * STEP, cc = c0 + cl;
      double xv[R];
#pragma unroll
      for (int j = 0; j < R; ++j) xv[j] = xs[buf][cl][j];
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        const int rr = r0 + rl + e;
        double av = (double)a[u][e];
        if (mlu) av = rr > cc ? av : (rr == cc ? 1.0 : 0.0);
        if (mup) av = rr <= cc ? av : 0.0;
        if (mlo) av = rr >= cc ? av : 0.0;
#pragma unroll
        for (int j = 0; j < R; ++j) acc[e][j] += av * xv[j];
      }
    }
    buf ^= 1;
  }
  // sum the column slots of the wave (lanes with equal lane % LPC)
#pragma unroll
  for (int e = 0; e < VEC; ++e)
#pragma unroll
    for (int j = 0; j < R; ++j)
      for (int off = LPC; off < 64; off <<= 1) acc[e][j] += __shfl_xor(acc[e][j], off, 64);
  if (lane < LPC) {
#pragma unroll
    for (int e = 0; e < VEC; ++e)
#pragma unroll
      for (int j = 0; j < R; ++j) red[g][rl + e][j] = acc[e][j];
  }
  __syncthreads();
  if (tid < 64) {
    const int r = r0 + lane;
    double dot[R], dd[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
      double s = red[0][lane][j] + red[1][lane][j] + red[2][lane][j] + red[3][lane][j];
      if (fl & V_MASK) s *= P.mask[r];
      if (fl & V_NEG) s = -s;
      if (fl & V_YIN) s += P.yin[r + j * ldy];
      if (r >= P.row_skip) P.yout[r + j * ldy] = s;
      dot[j] = (fl & V_DOT) ? dotv[P.dot_off + r + j * ldy] * s : 0.0;
      dd[j] = (fl & V_DOT2) ? s * s : 0.0;
    }
    if (fl & V_DOT) {
#pragma unroll
      for (int j = 0; j < R; ++j) {
        double v = dot[j], w = dd[j];
        for (int off = 32; off > 0; off >>= 1) {
          v += __shfl_xor(v, off, 64);
          w += __shfl_xor(w, off, 64);
        }
        if (lane == 0) {
          partial[((int64_t)wg * R + j) * 2 + 0] = v;
          partial[((int64_t)wg * R + j) * 2 + 1] = w;
        }
      }
    }
  }
}

// ------------------------------------------------------------------------
// One or two right-hand sides, 16-byte aligned problems: the column range's
// vector entries are staged in LDS once per workgroup (CH columns at a time), and
// the NW waves take interleaved groups of columns, U loads of 1 KiB each in flight
// per wave (a lane reads VEC consecutive rows of one column, a wave load 64 rows
// of VEC columns).  SHORT: ranges of at most U loads per wave, without the stage:
// a lane loads the vector entries of its columns itself, and the masks are applied
// to the batch at once.  Epilogue, flags and partial sums as in k_gemv.
//
// Bound: HBM for long launches; the sweeps are chains of short launches, so
// latency: with four loads in flight on four waves and the vector entries
// loaded beside every matrix entry, a 1024-wide triangle took 59 us (f32, 64
// blocks) and a 512-wide f64 one of 16 blocks 20.1 us; this form takes 31 us,
// and 7 us with sixteen waves.
// ------------------------------------------------------------------------
template <typename T, int R, int NW, int U, bool SHORT>
__global__ __launch_bounds__(64 * NW) void k_gemv_n(const GemvProb* __restrict__ probs, int nprob, int nwg,
                                                    int64_t ldx, int64_t ldy,
                                                    const double* __restrict__ dotv,
                                                    double* __restrict__ partial,
                                                    const int32_t* __restrict__ stop) {
  constexpr int VEC = 16 / sizeof(T);   // rows per lane
  constexpr int LPC = 64 / VEC;         // lanes per column
  constexpr int CH = SHORT ? U * NW * VEC : 2048 / R;   // columns at a time
  typedef T vec_t __attribute__((ext_vector_type(VEC)));
  // the vector entries, then the waves' sums
  constexpr int XS = SHORT ? 0 : CH * R;
  __shared__ __attribute__((aligned(16))) double xs[XS > NW * 64 * R ? XS : NW * 64 * R];
  double (*red)[64][R] = (double (*)[64][R])xs;
  if (stop) {
    bool all = true;
#pragma unroll
    for (int j = 0; j < R; ++j) all &= stop[j] != KS_RUNNING;
    if (all) return;
  }
  const int wg = blockIdx.x;
  const GemvProb P = probs[find_gemv(probs, nprob, wg, nwg)];
  const int r0 = (wg - P.wg0) * 64;
  int cb = P.cb, ce = P.ce;
  if (P.tri == 1) ce = min(ce, r0 + 64);
  if (P.tri == 2) cb = max(cb, r0);
  const int tid = threadIdx.x, lane = tid & 63;
  const int g = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q = lane / LPC;             // column slot of this lane
  const int rl = (lane % LPC) * VEC;    // first local row of this lane
  const int fl = P.flags;
  const bool mlu = fl & V_A_MLU, mup = fl & V_A_MUP, mlo = fl & V_A_MLO;
  const bool masked = mlu || mup || mlo;
  // global pointers: a generic one would be loaded from through the LDS path too
  gptr<T> A = (gptr<T>)P.A + r0 + rl;
  gptr<double> x1 = (gptr<double>)P.x1, x2 = (gptr<double>)P.x2;
  const int64_t lda = P.lda;
  const int split = P.split;
  double acc[VEC][R];
#pragma unroll
  for (int e = 0; e < VEC; ++e)
#pragma unroll
    for (int j = 0; j < R; ++j) acc[e][j] = 0.0;
  auto xval = [&](int cc, int j) __attribute__((always_inline)) {
    gptr<double> xp = cc < split ? x1 + cc : x2 + (cc - split);
    return xp[j * ldx];
  };
  auto fetch = [&](vec_t (&a)[U], int c, int c1) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int cc = c + u * NW * VEC;
      a[u] = cc < c1 ? *(gptr<vec_t>)(A + (int64_t)cc * lda) : vec_t{};
    }
  };
  // the packed-triangle masks change only the columns [r0, r0 + 64) of a slab
  auto mask = [&](vec_t& a, int cc) __attribute__((always_inline)) {
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      const int rr = r0 + rl + e;
      if (mlu) a[e] = rr > cc ? a[e] : (rr == cc ? T(1) : T(0));
      if (mup) a[e] = rr <= cc ? a[e] : T(0);
      if (mlo) a[e] = rr >= cc ? a[e] : T(0);
    }
  };
  // wave g takes the column groups c0 + VEC (g + NW s), s = 0, 1, ...
  if constexpr (SHORT) {
    // a range may begin and end at any column (the parts of a direct reduced solve
    // do); one of CH columns goes without the tests
    const int c = cb + g * VEC;
    auto batch = [&](auto all) __attribute__((always_inline)) {
      vec_t a[U] = {};
      double xv[U][R] = {};
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int cu = c + u * NW * VEC;
        if (!decltype(all)::value && cu + q >= ce) continue;
        a[u] = *(gptr<vec_t>)(A + (int64_t)(cu + q) * lda);
#pragma unroll
        for (int j = 0; j < R; ++j) xv[u][j] = xval(cu + q, j);
      }
      // the masks hold for every column of a clipped range: one test for the batch
      auto select = [&](auto in) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int e = 0; e < VEC; ++e) a[u][e] = in(a[u][e], r0 + rl + e, c + u * NW * VEC + q);
      };
      if (mlu) select([](T v, int r, int cc) { return r > cc ? v : (r == cc ? T(1) : T(0)); });
      if (mup) select([](T v, int r, int cc) { return r <= cc ? v : T(0); });
      if (mlo) select([](T v, int r, int cc) { return r >= cc ? v : T(0); });
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int j = 0; j < R; ++j)
#pragma unroll
          for (int e = 0; e < VEC; ++e) acc[e][j] += (double)a[u][e] * xv[u][j];
    };
    if (ce - cb == CH) batch(std::true_type{});
    else batch(std::false_type{});
  } else {
    for (int c0 = cb; c0 < ce; c0 += CH) {
      const int c1 = min(ce, c0 + CH);
      if (c0 > cb) __syncthreads();   // every wave is done with the previous columns
      for (int i = tid; i < (c1 - c0) * R; i += 64 * NW) {
        const int cc = c0 + i % (c1 - c0), j = i / (c1 - c0);
        xs[(cc - c0) * R + j] = xval(cc, j);
      }
      __syncthreads();
      for (int c = c0 + g * VEC + q; c - q < c1; c += U * NW * VEC) {
        vec_t a[U];
        fetch(a, c, c1);
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int cc = c + u * NW * VEC;
          if (cc >= c1) continue;
          if (masked && cc >= r0 && cc < r0 + 64) mask(a[u], cc);
#pragma unroll
          for (int j = 0; j < R; ++j) {
            const double xv = xs[(cc - c0) * R + j];
#pragma unroll
            for (int e = 0; e < VEC; ++e) acc[e][j] += (double)a[u][e] * xv;
          }
        }
      }
    }
  }
  // sum the column slots of the wave (lanes with equal lane % LPC)
#pragma unroll
  for (int e = 0; e < VEC; ++e)
#pragma unroll
    for (int j = 0; j < R; ++j)
      for (int off = LPC; off < 64; off <<= 1) acc[e][j] += __shfl_xor(acc[e][j], off, 64);
  if (!SHORT) __syncthreads();   // every wave is done with the vector entries
  if (lane < LPC) {
#pragma unroll
    for (int e = 0; e < VEC; ++e)
#pragma unroll
      for (int j = 0; j < R; ++j) red[g][rl + e][j] = acc[e][j];
  }
  __syncthreads();
  if (tid < 64) {
    const int r = r0 + lane;
    double dot[R], dd[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
      double s = 0.0;
#pragma unroll
      for (int w = 0; w < NW; ++w) s += red[w][lane][j];
      if (fl & V_MASK) s *= P.mask[r];
      if (fl & V_NEG) s = -s;
      if (fl & V_YIN) s += P.yin[r + j * ldy];
      if (r >= P.row_skip) P.yout[r + j * ldy] = s;
      dot[j] = (fl & V_DOT) ? dotv[P.dot_off + r + j * ldy] * s : 0.0;
      dd[j] = (fl & V_DOT2) ? s * s : 0.0;
    }
    if (fl & V_DOT) {
#pragma unroll
      for (int j = 0; j < R; ++j) {
        double v = dot[j], w = dd[j];
        for (int off = 32; off > 0; off >>= 1) {
          v += __shfl_xor(v, off, 64);
          w += __shfl_xor(w, off, 64);
        }
        if (lane == 0) {
          partial[((int64_t)wg * R + j) * 2 + 0] = v;
          partial[((int64_t)wg * R + j) * 2 + 1] = w;
        }
      }
    }
  }
}

// ------------------------------------------------------------------------
// Reduced-matrix product on packed spike tips.  The rows of G^ are the
// first and last t rows of each spike G_i (2t columns each), which inside
// the column-major spikes are 4t-byte column pieces N_i apart.  After every
// factorisation they are packed row-major (k_pack_tips), and the product
// streams each row as one contiguous run: a wave takes four rows at a time,
// its lanes read consecutive 16-byte pieces of them, the right-hand-side
// entries (2t values shared by every row of the part) come from LDS, once
// for the four rows, and the four row sums are reduced over the wave
// together.  Lane 16 i of a group of four rows ends with row i's sum; one
// epilogue per wave serves its RPW rows.  Same problem records, flags and
// partial-sum layout as k_gemv (A = first packed row, lda = row length 2t),
// a workgroup of 4 RPW rows and one partial per workgroup.
//
// Bound: HBM (2.1 GB of f64 tips in 355 us, 6.0 TB/s; splitting the columns
// over the waves as k_tipmv_c does takes 398 us); launches of a few workgroups:
// latency, so RPW is 4 instead of 16 where 64-row workgroups would leave CUs
// idle.  With one row at a time and the vector entries in registers, reloaded by
// every wave, six workgroups of 128-entry rows took 8.7 us, now 4.2 us.
// ------------------------------------------------------------------------
template <typename T, int R, int RPW, bool STEP>
__global__ __launch_bounds__(256) void k_tipmv(const GemvProb* __restrict__ probs, int nprob, int nwg,
                                               int64_t ldx, int64_t ldy,
                                               const double* __restrict__ dotv,
                                               double* __restrict__ partial,
                                               const int32_t* __restrict__ stop, TipStep F) {
  constexpr int VEC = 16 / sizeof(T);
  constexpr int SB = 16 / RPW;                  // workgroups per 64 rows
  typedef T vec_t __attribute__((ext_vector_type(VEC)));
  extern __shared__ __attribute__((aligned(16))) double xs[];   // [columns][R]
  constexpr int NS = STEP ? 3 : 2;              // sums per workgroup and column
  __shared__ double red[4][R][NS];
  if (stop) {
    bool all = true;
#pragma unroll
    for (int j = 0; j < R; ++j) all &= stop[j] != KS_RUNNING;
    if (all) return;
  }
  // the step's alpha, as k_bicg_s takes it
  double al[R];
  bool run[R];
  if (STEP) {
    __shared__ double sh[4][1][2];
    bool any = false;
#pragma unroll
    for (int j = 0; j < R; ++j) {
      double v1[2];
      take_sums(F.s1.W, R, j, F.s1.part, F.s1.sums, v1, sh);
      run[j] = s_ok(F.st, F.it, j, v1[0], al[j]);
      any |= run[j];
    }
    if (!any) return;   // no column goes on: nothing reads s, the product or their sums
  }
  const int wg = blockIdx.x / SB;
  const GemvProb& P = probs[find_gemv(probs, nprob, wg, nwg)];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int fl = P.flags;
  const int cb = P.cb, ce = P.ce, split = P.split, nc = ce - cb;
  const int rbase = (wg - P.wg0) * 64 + (blockIdx.x % SB) * (64 / SB) + wave * RPW;
  for (int i = tid; i < nc * R; i += 256) {
    const int c = cb + i % nc, j = i / nc;
    const double* xp = (c < split ? P.x1 + c : P.x2 + (c - split)) + j * ldx;
    if (STEP) {
      const int64_t o = xp - F.s;
      xs[(c - cb) * R + j] = run[j] ? F.r[o] - al[j] * F.v[o] : 0.0;
    } else {
      xs[(c - cb) * R + j] = *xp;
    }
  }
  __syncthreads();
  const T* __restrict__ A0 = (const T*)P.A + cb;
  const int64_t lda = P.lda;
  double mine[R];   // lane rr < RPW: the sum of the wave's row rr
#pragma unroll
  for (int j = 0; j < R; ++j) mine[j] = 0.0;
#pragma unroll 1
  for (int rr = 0; rr < RPW; rr += 4) {
    const T* __restrict__ Arow = A0 + (int64_t)(rbase + rr) * lda;
    double acc[4][R];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < R; ++j) acc[i][j] = 0.0;
    // 2t and the column range are multiples of 64, so a lane's piece lies
    // inside the row or outside it
    for (int c0 = lane * VEC; c0 < nc; c0 += 2 * 64 * VEC) {
      vec_t a[2][4];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int c = c0 + h * 64 * VEC;
#pragma unroll
        for (int i = 0; i < 4; ++i) a[h][i] = c < nc ? *(const vec_t*)(Arow + i * lda + c) : vec_t{};
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int c = c0 + h * 64 * VEC;
        if (c >= nc) continue;
#pragma unroll
        for (int e = 0; e < VEC; ++e)
#pragma unroll
          for (int j = 0; j < R; ++j) {
            const double xv = xs[(c + e) * R + j];
#pragma unroll
            for (int i = 0; i < 4; ++i) acc[i][j] += (double)a[h][i][e] * xv;
          }
      }
    }
    // four sums at once: lanes with bit 5 set continue with rows 2 and 3,
    // then lanes with bit 4 set with the odd row of the pair
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const bool h5 = lane & 32, h4 = lane & 16;
      const double s0 = (h5 ? acc[2][j] : acc[0][j]) + __shfl_xor(h5 ? acc[0][j] : acc[2][j], 32, 64);
      const double s1 = (h5 ? acc[3][j] : acc[1][j]) + __shfl_xor(h5 ? acc[1][j] : acc[3][j], 32, 64);
      double v = (h4 ? s1 : s0) + __shfl_xor(h4 ? s0 : s1, 16, 64);
      for (int off = 8; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
      // row i's sum is in lanes 16 i .. 16 i + 15
      const double w = __shfl(v, (lane & 3) * 16, 64);
      mine[j] = (lane >= rr && lane < rr + 4) ? w : mine[j];
    }
  }
  double dot[R], dd[R], ss[R];
#pragma unroll
  for (int j = 0; j < R; ++j) dot[j] = dd[j] = ss[j] = 0.0;
  if (lane < RPW) {
    const int r = rbase + lane;
#pragma unroll
    for (int j = 0; j < R; ++j) {
      double v = mine[j];
      if (fl & V_MASK) v *= P.mask[r];
      if (fl & V_NEG) v = -v;
      if (STEP) {
        // y_in and the vector of the dot product are s
        const int64_t o = P.yin + r + j * ldy - F.s;
        const double sv = run[j] ? F.r[o] - al[j] * F.v[o] : 0.0;
        if (run[j]) F.s[o] = sv;
        ss[j] = sv * sv;
        v += sv;
        P.yout[r + j * ldy] = v;
        dot[j] = sv * v;
      } else {
        if (fl & V_YIN) v += P.yin[r + j * ldy];
        P.yout[r + j * ldy] = v;
        if (fl & V_DOT) dot[j] = dotv[P.dot_off + r + j * ldy] * v;
      }
      if (fl & V_DOT2) dd[j] = v * v;
    }
  }
  if (fl & (V_DOT | V_DOT2)) {
#pragma unroll
    for (int j = 0; j < R; ++j)
      for (int off = RPW / 2; off > 0; off >>= 1) {
        dot[j] += __shfl_xor(dot[j], off, 64);
        dd[j] += __shfl_xor(dd[j], off, 64);
        if (STEP) ss[j] += __shfl_xor(ss[j], off, 64);
      }
    if (lane == 0)
#pragma unroll
      for (int j = 0; j < R; ++j) {
        red[wave][j][0] = dot[j];
        red[wave][j][1] = dd[j];
        if (STEP) red[wave][j][NS - 1] = ss[j];
      }
    __syncthreads();
    if (tid < R) {
      const int j = tid;
      partial[((int64_t)blockIdx.x * R + j) * 2 + 0] = (red[0][j][0] + red[1][j][0]) + (red[2][j][0] + red[3][j][0]);
      partial[((int64_t)blockIdx.x * R + j) * 2 + 1] = (red[0][j][1] + red[1][j][1]) + (red[2][j][1] + red[3][j][1]);
      if (STEP) {
        F.ss[((int64_t)blockIdx.x * R + j) * 2 + 0] =
            (red[0][j][NS - 1] + red[1][j][NS - 1]) + (red[2][j][NS - 1] + red[3][j][NS - 1]);
        F.ss[((int64_t)blockIdx.x * R + j) * 2 + 1] = 0.0;
      }
    }
  }
}

// The same product for launches that fill the GPU: the four waves of a
// workgroup split the columns instead of the rows, so that the workgroup
// streams its 64 rows one after another as one contiguous run, and a wave's
// vector entries (NS pieces of 64 VEC columns) stay in registers.  A wave
// reduces its part of eight rows at a time; the four parts of a row are added
// in LDS.  1.06 GB of f32 tips take 177 us (6.0 TB/s; by rows 189 us).
template <typename T, int R, int NS>
__global__ __launch_bounds__(256) void k_tipmv_c(const GemvProb* __restrict__ probs, int nprob, int nwg,
                                                 int64_t ldx, int64_t ldy,
                                                 const double* __restrict__ dotv,
                                                 double* __restrict__ partial,
                                                 const int32_t* __restrict__ stop) {
  constexpr int VEC = 16 / sizeof(T);
  constexpr int RB = NS * R <= 2 ? 8 : 4;       // rows in flight
  typedef T vec_t __attribute__((ext_vector_type(VEC)));
  __shared__ double red[4][64][R];
  if (stop) {
    bool all = true;
#pragma unroll
    for (int j = 0; j < R; ++j) all &= stop[j] != KS_RUNNING;
    if (all) return;
  }
  const int wg = blockIdx.x;
  const GemvProb& P = probs[find_gemv(probs, nprob, wg, nwg)];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cb = P.cb, split = P.split, nc = P.ce - cb;
  const int r0 = (wg - P.wg0) * 64;
  const int64_t lda = P.lda;
  // this lane's columns: piece s starts at (4 s + wave) * 64 VEC + lane VEC
  int c[NS];
  double x[NS][VEC][R];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    c[s] = ((4 * s + wave) * 64 + lane) * VEC;
#pragma unroll
    for (int e = 0; e < VEC; ++e)
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const int cc = cb + c[s] + e;
        x[s][e][j] = c[s] < nc ? (cc < split ? P.x1[cc + j * ldx] : P.x2[(cc - split) + j * ldx]) : 0.0;
      }
    // bytes from a row's start; past the row: out of the buffer's range, where a
    // load gives zero
    c[s] = c[s] < nc ? c[s] * (int)sizeof(T) : (int)0x80000000;
  }
  const auto A0 = __builtin_amdgcn_make_buffer_rsrc((void*)((const T*)P.A + (int64_t)r0 * lda + cb), 0, 0x7fffffff,
                                                    0x00027000);
#pragma unroll 1
  for (int rr = 0; rr < 64; rr += RB) {
    vec_t a[RB][NS];
#pragma unroll
    for (int i = 0; i < RB; ++i)
#pragma unroll
      for (int s = 0; s < NS; ++s)
        a[i][s] = __builtin_bit_cast(
            vec_t, __builtin_amdgcn_raw_buffer_load_b128(A0, c[s], (int)((rr + i) * lda * (int)sizeof(T)), 0));
#pragma unroll
    for (int j = 0; j < R; ++j) {
      double v[RB];
#pragma unroll
      for (int i = 0; i < RB; ++i) {
        v[i] = 0.0;
#pragma unroll
        for (int s = 0; s < NS; ++s)
#pragma unroll
          for (int e = 0; e < VEC; ++e) v[i] += (double)a[i][s][e] * x[s][e][j];
      }
      // RB sums at once: at each step a lane keeps half of its rows and hands
      // the other half's sums to its partner
      int off = 32;
#pragma unroll
      for (int n = RB / 2; n > 0; n >>= 1, off >>= 1) {
        const bool up = lane & off;
#pragma unroll
        for (int i = 0; i < n; ++i) {
          const double keep = up ? v[i + n] : v[i], give = up ? v[i] : v[i + n];
          v[i] = keep + __shfl_xor(give, off, 64);
        }
      }
      for (; off > 0; off >>= 1) v[0] += __shfl_xor(v[0], off, 64);
      // lanes with equal lane / (64 / RB) hold row rr + lane / (64 / RB)
      if (lane % (64 / RB) == 0) red[wave][rr + lane / (64 / RB)][j] = v[0];
    }
  }
  __syncthreads();
  if (tid < 64) {
    const int fl = P.flags, r = r0 + lane;
#pragma unroll
    for (int j = 0; j < R; ++j) {
      double v = (red[0][lane][j] + red[1][lane][j]) + (red[2][lane][j] + red[3][lane][j]);
      if (fl & V_MASK) v *= P.mask[r];
      if (fl & V_NEG) v = -v;
      if (fl & V_YIN) v += P.yin[r + j * ldy];
      P.yout[r + j * ldy] = v;
      if (fl & (V_DOT | V_DOT2)) {
        double d = (fl & V_DOT) ? dotv[P.dot_off + r + j * ldy] * v : 0.0, dd = (fl & V_DOT2) ? v * v : 0.0;
        for (int off = 32; off > 0; off >>= 1) {
          d += __shfl_xor(d, off, 64);
          dd += __shfl_xor(dd, off, 64);
        }
        if (lane == 0) {
          partial[((int64_t)wg * R + j) * 2 + 0] = d;
          partial[((int64_t)wg * R + j) * 2 + 1] = dd;
        }
      }
    }
  }
}

// Packs the spike tips row-major: part q (q = 0 .. 2(p-1)-1; block
// i = (q+1)/2, its first t rows for q odd, its last t rows for q even) to
// tips[q][r][c], r < t, c < 2t, through a 64 x 64 LDS tile so both the
// column-major reads and the row-major writes are coalesced.
template <typename T>
__global__ __launch_bounds__(256) void k_pack_tips(const BlockInfo* __restrict__ blocks, int t,
                                                   const T* __restrict__ spikes, T* __restrict__ tips) {
  __shared__ T tile[64][65];
  const int q = blockIdx.z;
  const int i = (q + 1) / 2;
  const BlockInfo B = blocks[i];
  const int64_t row0 = (q & 1) ? B.pad : B.N - t;
  const int r0 = blockIdx.y * 64, c0 = blockIdx.x * 64;
  const T* __restrict__ G = spikes + B.goff;
  T* __restrict__ out = tips + (int64_t)q * t * 2 * t;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int c = ty + 4 * k;
    tile[c][tx] = G[(int64_t)(c0 + c) * B.N + row0 + r0 + tx];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int r = ty + 4 * k;
    out[(int64_t)(r0 + r) * 2 * t + c0 + tx] = tile[tx][r];
  }
}

// whether rows of 2t entries are kept packed (at most 16 KiB each)
bool tipmv_packs(int dtype, int t) { return 2 * t * (dtype == 0 ? 8 : 4) <= 16384; }

// Workgroups (and partial sums) per 64 rows: four of 16 rows each where 64-row
// workgroups would leave CUs idle, two where four would keep so many rows of 16
// KiB in flight that they meet in the same memory channels.  One column, us with
// four / two / one to 64 rows (FP32's one: the better of rows and column split):
//   f64  1024 entries   128 workgroups 12.9 / 17.4 / 15.4, 192 18.5 / 22.0 / 18.1
//        1920           150            22.9 / 24.3 / 26.2, 210 31.1 / 30.7 / 31.6
//        2048 (16 KiB)   64            15.3 / 16.6 / 23.7,  96 20.9 / 19.7 / 24.1,
//                       128            27.0 / 24.3 / 25.4, 160 34.0 / 28.4 / 28.1
//   f32  1024           192            11.0 / 10.2 / 12.6, 224 16.1 / 12.4 / 13.2
//        1536           216            15.9 / 16.1 / 16.9, 264 18.1 / 18.3 / 18.9
//        2048           192            18.9 / 22.7 / 20.2, 256 24.5 / 30.8 / 23.4
//        3072           144            18.9 / 19.6 / 21.3, 240 28.9 / 29.0 / 26.6
//        3456           216            28.8 / 29.1 / 29.6
//        4096 (16 KiB)  128            27.7 / 24.9 / 26.1, 192 37.4 / 31.6 / 29.7
int tipmv_split(int dtype, int t, int nwg) {
  const int row = 2 * t * (dtype == 0 ? 8 : 4);   // bytes
  if (row % 16384 == 0) return nwg < 96 ? 4 : nwg <= 128 ? 2 : 1;
  if (dtype == 0) return nwg <= 160 ? 4 : 1;
  return nwg <= (row % 4096 == 0 ? 192 : 256) ? 4 : 1;
}

// FP32 with one workgroup to 64 rows: the column split where its pieces (1024
// entries of a row each, a quarter per wave) are nearly filled, else by rows.
// Column split / rows, us:
//   one column    1024 entries, 512 workgroups 24.9 / 23.5   1536, 768 56.0 / 47.3
//                 1664, 520 44.8 / 34.8                      1920, 780 74.6 / 67.0
//                 2048, 512 40.0 / 42.3, on 256 24.4 / 23.4
//                 2176, 306 28.1 / 29.9    3200, 1000 138 / 152   4096, 512 86.5 / 90.1
//   two columns   2304, 288 35.7 / 32.8
//                 2688, 1008 126 / 139     3200, 1000 153 / 166   3712, 2030 325 / 345
static bool tipmv_by_columns(int dtype, int nrhs, int t, int nwg) {
  if (dtype == 0) return false;
  if (t <= 1024) return t == 1024 && nwg > 256;
  return nrhs == 1 || 9 * 2 * t >= 7 * ((2 * t + 1023) / 1024 * 1024);
}

// the step for FP32 only where a workgroup takes few rows, so that its sums are worth taking up
bool tipmv_steps(int dtype, int t, int nwg) { return dtype == 0 || tipmv_split(dtype, t, nwg) > 1; }

void launch_tipmv(int dtype, int nrhs, int t, const GemvProb* probs, int nprob, int nwg, int64_t ldx,
                  int64_t ldy, const double* dotv, double* partial, const int32_t* stop, hipStream_t s,
                  const TipStep* step) {
  if (nwg <= 0 || nprob <= 0) return;
  const int sb = tipmv_split(dtype, t, nwg);
  const size_t lds = (size_t)2 * t * (nrhs == 1 ? 1 : 2) * sizeof(double);
  // Three workgroups of the column split fit a CU for one column and rows of two
  // pieces.  Where two to a CU take no more rounds, LDS holds it to two, which
  // share the last round evenly (2048-entry rows, 1024 workgroups: 90 instead of
  // 103 us; 640 workgroups, one round of three: 57 instead of 68 us).
  const size_t two = nwg > 768 && nwg <= 1024 ? 56 * 1024 : 0;
#define DDPS_TIPMV(L, ...) \
  hipLaunchKernelGGL((__VA_ARGS__), dim3(nwg), dim3(256), L, s, probs, nprob, nwg, ldx, ldy, dotv, partial, stop)
#define DDPS_TIPMV_S(T, R, RPW)                                                                                     \
  if (step)                                                                                                         \
    hipLaunchKernelGGL((k_tipmv<T, R, RPW, true>), dim3(nwg * sb), dim3(256), lds, s, probs, nprob, nwg, ldx, ldy,      \
                       dotv, partial, stop, *step);                                                                 \
  else                                                                                                              \
    hipLaunchKernelGGL((k_tipmv<T, R, RPW, false>), dim3(nwg * sb), dim3(256), lds, s, probs, nprob, nwg, ldx, ldy,     \
                       dotv, partial, stop, TipStep{})
#define DDPS_TIPMV_C(T, R)                                            \
  switch (ns) {                                                       \
    case 2: DDPS_TIPMV(R == 1 ? two : 0, k_tipmv_c<T, R, 2>); break;  \
    case 3: DDPS_TIPMV(0, k_tipmv_c<T, R, 3>); break;                 \
    default: DDPS_TIPMV(0, k_tipmv_c<T, R, 4>); break;                \
  }
#define DDPS_TIPMV_R(T, R)                   \
  if (sb == 4) { DDPS_TIPMV_S(T, R, 4); }      \
  else if (sb == 2) { DDPS_TIPMV_S(T, R, 8); } \
  else { DDPS_TIPMV_S(T, R, 16); }
  if (sb == 1 && tipmv_by_columns(dtype, nrhs, t, nwg)) {
    const int ns = (2 * t + 1023) / 1024;
    if (nrhs == 1) { DDPS_TIPMV_C(float, 1) }
    else { DDPS_TIPMV_C(float, 2) }
  } else if (dtype == 0) {
    if (nrhs == 1) { DDPS_TIPMV_R(double, 1) }
    else { DDPS_TIPMV_R(double, 2) }
  } else {
    if (nrhs == 1) { DDPS_TIPMV_R(float, 1) }
    else { DDPS_TIPMV_R(float, 2) }
  }
#undef DDPS_TIPMV_R
#undef DDPS_TIPMV_C
#undef DDPS_TIPMV_S
#undef DDPS_TIPMV
}

void pack_tips(int dtype, int p, int t, const BlockInfo* blocks, const void* spikes, void* tips, hipStream_t s) {
  if (p < 2) return;
  const dim3 g(2 * t / 64, t / 64, 2 * (p - 1)), b(256);
  if (dtype == 0) hipLaunchKernelGGL(k_pack_tips<double>, g, b, 0, s, blocks, t, (const double*)spikes, (double*)tips);
  else hipLaunchKernelGGL(k_pack_tips<float>, g, b, 0, s, blocks, t, (const float*)spikes, (float*)tips);
}

// ------------------------------------------------------------------------
// Many right-hand sides (R >= 4) on FP32 operands, as products on the FP32
// matrix cores (16x16x4).  One workgroup per 64-row slab; its 4 waves take
// interleaved groups of 16 columns (column ranges and the vectors' split are
// multiples of 16).  Lane l loads rows 4(l & 15) .. +3 of the columns c + 4(l >> 4)
// + u, u = 0 .. 3 (four float4, each wave load 64 rows x 4 columns), and the two
// 16-byte pairs of x(those columns, rhs l & 15), rounded to FP32 (0 for rhs >= R).
// For each u the four products q take component q of the float4, so product q
// accumulates the slab rows 4i + q.  The sums are FP32, each over a quarter of
// the columns; the four quarters are added in FP64 in a fixed order.  Register v
// of accumulator q in lane l holds slab row 16 (l >> 4) + 4 v + q, rhs l & 15.
// Triangular problems clip the column range as the other kernels do; the
// masks of packed triangles change only the columns [r0, r0 + 64) of a
// slab, so only loads of those columns go through the selects.
//
// Bound: HBM, and the vector's loads beside the matrix's.  With one vector entry
// per load and groups of 4 columns, 2.58 GB of strided spikes (t = 1600) and 8
// right-hand sides took 538 us; entries in pairs 484 us; three groups loaded ahead
// 474 us (5.4 TB/s).
// ------------------------------------------------------------------------
template <int R>
__global__ __launch_bounds__(256) void k_gemv_mf32(const GemvProb* __restrict__ probs, int nprob, int nwg,
                                                   int64_t ldx, int64_t ldy,
                                                   const double* __restrict__ dotv,
                                                   double* __restrict__ partial,
                                                   const int32_t* __restrict__ stop) {
  typedef float f32x4 __attribute__((ext_vector_type(4)));
  typedef double f64x2u __attribute__((ext_vector_type(2), aligned(8)));
  static_assert(R >= 1 && R <= 16, "right-hand sides per product");
  constexpr int DEP = 4;   // column groups of a wave held at a time
  __shared__ float red[4][64][R];
  if (stop) {
    bool all = true;
#pragma unroll
    for (int j = 0; j < R; ++j) all &= stop[j] != KS_RUNNING;
    if (all) return;
  }
  const int wg = blockIdx.x;
  const GemvProb P = probs[find_gemv(probs, nprob, wg, nwg)];
  const int r0 = (wg - P.wg0) * 64;
  int cb = P.cb, ce = P.ce;
  if (P.tri == 1) ce = min(ce, r0 + 64);
  if (P.tri == 2) cb = max(cb, r0);
  const int tid = threadIdx.x, lane = tid & 63;
  const int g = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lk = lane >> 4;
  const int fl = P.flags;
  const bool mlu = fl & V_A_MLU, mup = fl & V_A_MUP, mlo = fl & V_A_MLO;
  const bool masked = mlu || mup || mlo;
  const float* __restrict__ A = (const float*)P.A + r0 + 4 * li;
  const int64_t lda = P.lda;
  const int split = P.split;
  const bool live = li < R;
  const int jx = live ? li : 0;
  f32x4 acc[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
  // the packed-triangle masks on the 4 rows of a lane's load of column cc
  auto fix = [&](float4& a, int cc) __attribute__((always_inline)) {
    if (masked && cc >= r0 && cc < r0 + 64) {
      float e[4] = {a.x, a.y, a.z, a.w};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int rr = r0 + 4 * li + q;
        if (mlu) e[q] = rr > cc ? e[q] : (rr == cc ? 1.f : 0.f);
        if (mup) e[q] = rr <= cc ? e[q] : 0.f;
        if (mlo) e[q] = rr >= cc ? e[q] : 0.f;
      }
      a = float4{e[0], e[1], e[2], e[3]};
    }
  };
  auto mma = [&](const float4& a, float x) __attribute__((always_inline)) {
    acc[0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, x, acc[0], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, x, acc[1], 0, 0, 0);
    acc[2] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, x, acc[2], 0, 0, 0);
    acc[3] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, x, acc[3], 0, 0, 0);
  };
  // wave g takes the columns cb + 16 (g + 4 s) .. + 15, s = 0, 1, ...; lane
  // group lk their 4 lk .. 4 lk + 3, one to each product, so that a lane's four
  // vector entries are consecutive
  struct Step {
    float4 a[4];
    f64x2u x[2];
  };
  auto fetch = [&](Step& F, int c) __attribute__((always_inline)) {
    const int cl = c + 4 * lk;
    const double* __restrict__ xp = c < split ? P.x1 + cl : P.x2 + (cl - split);
    F.x[0] = *(const f64x2u*)(xp + jx * ldx);
    F.x[1] = *(const f64x2u*)(xp + jx * ldx + 2);
#pragma unroll
    for (int u = 0; u < 4; ++u) F.a[u] = *(const float4*)(A + (int64_t)(cl + u) * lda);
  };
  auto multiply = [&](Step& F, int c) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      fix(F.a[u], c + 4 * lk + u);
      mma(F.a[u], live ? (float)F.x[u / 2][u % 2] : 0.f);
    }
  };
  const int c0 = cb + 16 * g;
  Step F[DEP];
#pragma unroll
  for (int i = 0; i < DEP - 1; ++i)
    if (c0 + 64 * i < ce) fetch(F[i], c0 + 64 * i);
#pragma unroll 1
  for (int c = c0; c < ce; c += 64 * DEP) {
#pragma unroll
    for (int i = 0; i < DEP; ++i) {
      const int ci = c + 64 * i;
      if (ci + 64 * (DEP - 1) < ce) fetch(F[(i + DEP - 1) % DEP], ci + 64 * (DEP - 1));
      if (ci < ce) multiply(F[i], ci);
    }
  }
  if (live) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
      for (int v = 0; v < 4; ++v) red[g][16 * lk + 4 * v + q][li] = acc[q][v];
  }
  __syncthreads();
  if (tid < 64) {
    const int r = r0 + lane;
    double dot[R], dd[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
      double s = (double)red[0][lane][j] + (double)red[1][lane][j] + (double)red[2][lane][j] + (double)red[3][lane][j];
      if (fl & V_MASK) s *= P.mask[r];
      if (fl & V_NEG) s = -s;
      if (fl & V_YIN) s += P.yin[r + j * ldy];
      if (r >= P.row_skip) P.yout[r + j * ldy] = s;
      dot[j] = (fl & V_DOT) ? dotv[P.dot_off + r + j * ldy] * s : 0.0;
      dd[j] = (fl & V_DOT2) ? s * s : 0.0;
    }
    if (fl & V_DOT) {
#pragma unroll
      for (int j = 0; j < R; ++j) {
        double v = dot[j], w = dd[j];
        for (int off = 32; off > 0; off >>= 1) {
          v += __shfl_xor(v, off, 64);
          w += __shfl_xor(w, off, 64);
        }
        if (lane == 0) {
          partial[((int64_t)wg * R + j) * 2 + 0] = v;
          partial[((int64_t)wg * R + j) * 2 + 1] = w;
        }
      }
    }
  }
}

// rounds of workgroups that a launch of kernel K makes on the 256 CUs
template <auto K>
static int gemv_rounds(int nwg) {
  static const int per_cu = [] {
    int n = 0;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, K, 256, 0) == hipSuccess && n > 0 ? n : 1;
  }();
  return (nwg + 256 * per_cu - 1) / (256 * per_cu);
}

template <typename T>
static void gemv_dispatch(int nrhs, bool wide, int cols, const GemvProb* probs, int nprob, int nwg, int64_t ldx,
                          int64_t ldy, const double* dotv, double* partial, const int32_t* stop,
                          hipStream_t s) {
#define DDPS_GEMV(NT, ...) \
  hipLaunchKernelGGL((__VA_ARGS__), dim3(nwg), dim3(NT), 0, s, probs, nprob, nwg, ldx, ldy, dotv, partial, stop)
#define DDPS_GEMV_W(R)                                                                      \
  if (gemv_rounds<k_gemv_w<T, R, 4>>(nwg) < gemv_rounds<k_gemv_w<T, R, 8>>(nwg))            \
    DDPS_GEMV(256, k_gemv_w<T, R, 4>);                                                      \
  else                                                                                      \
    DDPS_GEMV(256, k_gemv_w<T, R, 8>)
#define DDPS_GEMV_N(NW, U, SHORT)                                     \
  if (nrhs == 1) DDPS_GEMV(64 * NW, k_gemv_n<T, 1, NW, U, SHORT>);    \
  else DDPS_GEMV(64 * NW, k_gemv_n<T, 2, NW, U, SHORT>)
  if (wide && nrhs <= 2) {
    // Ranges that four or eight waves load at once need no stage in LDS.  Chains of
    // sweeps, us per launch, with the stage / without: four waves, f64 64 columns, 4 /
    // 300 workgroups 3.7 / 2.7 and 5.5 / 4.3 (two right-hand sides 4.3 / 3.0 and 6.1 /
    // 4.9), f32 128 columns, 64 / 1000 workgroups 4.2 / 3.3 and 9.4 / 8.4 (5.5 / 4.0 and
    // 10.5 / 10.8).  Eight waves: f64 128 columns, 256 / 500 / 1000 workgroups 5.8 /
    // 5.0, 9.5 / 8.1, 14.3 / 13.8 (6.5 / 5.6, 10.1 / 10.4, 15.2 / 19.0), f32 256 columns,
    // 240 / 500 / 1000 workgroups 5.6 / 4.7, 7.9 / 6.6, 12.1 / 12.4 (7.0 / 5.5, 8.9 /
    // 9.6, 13.5 / 19.2).
    // Wider ones, one workgroup per CU or fewer: sixteen waves each, so that a
    // short launch has all its loads in flight at once; beyond, four fill the CUs with
    // less to add up.  Sixteen against four on f64 triangles of 512 rows: 128
    // workgroups 7.0 / 11.9, 512 workgroups 20.8 / 19.3 (f32 14.2 / 11.7).
    constexpr int once = 8 * 4 * 16 / (int)sizeof(T);   // columns that four waves load at once
    if (cols <= 64) { DDPS_GEMV_N(4, 512 / once, true); }
    else if (cols <= once) { DDPS_GEMV_N(4, 8, true); }
    else if (cols <= 2 * once && nwg <= (nrhs == 1 ? 512 : 256)) { DDPS_GEMV_N(8, 8, true); }
    else if (nwg <= 256) { DDPS_GEMV_N(16, 8, false); }
    else { DDPS_GEMV_N(4, 8, false); }
    return;
  }
  if (wide) {
    // Eight loads in flight, or four where the smaller kernel, of which more
    // workgroups fit a CU, makes fewer rounds.  Eight / four, f64, us: 8 columns, 512 x
    // 512 triangles, 1040 workgroups (2 / 1 rounds) 58.6 / 50.5, 2400 (3 / 2) 110
    // / 105; 1600 x 3200, 1600 (2 / 2) 477 / 514; 4 columns, 768 x 1536, 1536 (2 / 1)
    // 226 / 204, 1024 x 2048, 2048 (2 / 2) 346 / 389.
    if (nrhs == 4) DDPS_GEMV_W(4);
    else DDPS_GEMV_W(8);
    return;
  }
  switch (nrhs) {
    case 1: DDPS_GEMV(256, k_gemv<T, 1>); break;
    case 2: DDPS_GEMV(256, k_gemv<T, 2>); break;
    case 4: DDPS_GEMV(256, k_gemv<T, 4>); break;
    default: DDPS_GEMV(256, k_gemv<T, 8>); break;
  }
#undef DDPS_GEMV_N
#undef DDPS_GEMV_W
#undef DDPS_GEMV
}

void launch_gemv(int dtype, int nrhs, int form, int cols, const GemvProb* probs, int nprob, int nwg, int64_t ldx,
                 int64_t ldy, const double* dotv, double* partial, const int32_t* stop, hipStream_t s) {
  if (nwg <= 0 || nprob <= 0) return;
  if (dtype == 1 && form == 2 && nrhs >= 4) {
    if (nrhs == 4)
      hipLaunchKernelGGL(k_gemv_mf32<4>, dim3(nwg), dim3(256), 0, s, probs, nprob, nwg, ldx, ldy, dotv, partial, stop);
    else
      hipLaunchKernelGGL(k_gemv_mf32<8>, dim3(nwg), dim3(256), 0, s, probs, nprob, nwg, ldx, ldy, dotv, partial, stop);
    return;
  }
  if (dtype == 0) gemv_dispatch<double>(nrhs, form >= 1, cols, probs, nprob, nwg, ldx, ldy, dotv, partial, stop, s);
  else gemv_dispatch<float>(nrhs, form >= 1, cols, probs, nprob, nwg, ldx, ldy, dotv, partial, stop, s);
}

}  // namespace ddps
