// Diagonal sub-tile kernel of the tile LU: for each problem, one workgroup of
// eight waves factors a 64 x 64 sub-tile without pivoting (A = L U, L unit
// lower), then inverts both triangles and writes back L^{-1} strictly below
// the diagonal and U^{-1} on and above it.
//
// The kernel is latency bound (a few of them run at a time, one per block of
// the partition), so the work of one sub-tile is spread over eight waves.
//
// Elimination.  Wave w owns columns 8w .. 8w+7: lane r holds
// a[c] = A(r, 8w + c) in registers.  In round b the wave owning columns
// 8b .. 8b+7 runs their 8 elimination steps k: it reads the pivot u(k,k)
// from lane k (v_readlane), forms the multipliers l(r) = a(r,k) / u(k,k) for
// r > k, keeps them as column k of L, updates its own columns right of k and
// puts the multipliers in LDS.  After one barrier every wave right of it
// applies the same 8 steps to its columns, a(r,c) -= l(r) a(k,c), with the
// pivot row read from lane k of its own registers.  The multipliers of
// consecutive rounds alternate between two LDS buffers.  The operations and
// their order per entry are those of a one-wave elimination, so the factors
// do not depend on the split.
//
// Inversion, in place in LDS (row-major, L below the diagonal, U on and above
// it), by halves: for a triangle of blocks
//   [U00 U01]^-1   [Y00  -Y00 U01 Y11]      [L00    ]^-1   [X00             ]
//   [    U11]    = [          Y11    ]      [L10 L11]    = [-X11 L10 X00 X11]
// First the eight 16 x 16 diagonal triangles, one per wave, a lane per column
// by substitution; then the four 16 x 16 off-diagonal blocks of the 32 x 32
// triangles and the two 32 x 32 blocks of the whole, as products on the matrix
// cores (16x16x4, in the factors' own type).  By rows, each a sum over all
// earlier columns on the vector units, the inversion was about half of the
// kernel.  Alone an f64 sub-tile took 31 us, now 23 us, f32 24 and 17 us; beside
// the products of the other stream f64 66 and 31 us, because 51 instead of 110 KiB
// of LDS fit a CU that still runs half of its products.  What remains is the
// elimination's chain of 64 reciprocals and the reads of pivot rows between lanes.
//
// Pivot check, after the elimination: lane r of wave 2 tests u_rr against
// thresh[row] (the row's threshold in the padded layout); a pivot at or below
// it, or not finite, records (block, global row) in *bad through an atomic
// minimum, so the first bad pivot in (block, row) order is reported.
#include "ddps_internal.h"
#include "mma_device.h"

namespace ddps {

namespace {

constexpr int kN = kTile;      // 64
constexpr int kB = 16;         // diagonal blocks of the inversions
constexpr int kW = 8;          // waves of the workgroup
constexpr int kE = kN / kW;    // columns per wave in the elimination
constexpr int kLd = kN + 1;    // row-major LU: conflict-free column access
constexpr int kLdT = 2 * kB + 1;

// value of x in lane `lane` (wave-uniform), broadcast to the wave
__device__ __forceinline__ float lane_value(float x, int lane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), lane));
}
__device__ __forceinline__ double lane_value(double x, int lane) {
  const unsigned long long u = __builtin_bit_cast(unsigned long long, x);
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)u, lane);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(u >> 32), lane);
  return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// LDS stores of the wave's lanes before their reads by other lanes of it; the
// hardware keeps that order, so this costs no instruction
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace

template <typename T>
__global__ __launch_bounds__(64 * kW) void k_panel(const PanelProb* __restrict__ probs,
                                               const double* __restrict__ thresh,
                                               unsigned long long* __restrict__ bad) {
  __shared__ T LU[kN][kLd];   // L (c < r) and U (c >= r), row-major; then their inverses
  __shared__ T Rv[kN];        // 1 / u(k, k)
  // multipliers of the current round; then the inner products of the inversion
  __shared__ union {
    T Lm[2][kE][kN];
    T H[2][2 * kB][kLdT];
  } S;
  const PanelProb P = probs[blockIdx.x];
  T* __restrict__ D = (T*)P.D;
  const int r = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t ld = P.ld;

  T a[kE];   // a[c] = A(r, kE w + c)
#pragma unroll
  for (int c = 0; c < kE; ++c) a[c] = D[(int64_t)(kE * w + c) * ld + r];

#pragma unroll 1
  for (int kb = 0; kb < kW; ++kb) {
    // the owner eliminates its kE columns and publishes their multipliers
    if (w == kb) {
      T rv = T(0);   // lane k: 1 / u(k, k)
#pragma unroll
      for (int kc = 0; kc < kE; ++kc) {
        const int k = kE * kb + kc;
        T u[kE];   // row k, read ahead of its uses: each read stalls what follows it
#pragma unroll
        for (int c = kc; c < kE; ++c) u[c] = lane_value(a[c], k);
        __builtin_amdgcn_sched_barrier(0);
        const T rp = T(1) / u[kc];
        rv = r == k ? rp : rv;
        const T l = r > k ? a[kc] * rp : T(0);
#pragma unroll
        for (int c = kc + 1; c < kE; ++c) a[c] -= l * u[c];
        a[kc] = r > k ? l : a[kc];
        S.Lm[kb & 1][kc][r] = l;
      }
      if (r / kE == kb) Rv[r] = rv;
    }
    __syncthreads();
    // the waves right of it apply the same steps to their columns
    if (w > kb) {
#pragma unroll
      for (int kc = 0; kc < kE; ++kc) {
        const int k = kE * kb + kc;
        const T l = S.Lm[kb & 1][kc][r];
        T u[kE];
#pragma unroll
        for (int c = 0; c < kE; ++c) u[c] = lane_value(a[c], k);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < kE; ++c) a[c] -= l * u[c];
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
#pragma unroll
  for (int c = 0; c < kE; ++c) LU[r][kE * w + c] = a[c];
  __syncthreads();

  if (w == 2) {
    const double th = thresh[P.vrow0 + r];   // pivot threshold of this lane's row
    const double av = fabs((double)LU[r][r]);
    if (!(av > th) || !(av <= 1.7e308))
      atomicMin(bad, ((unsigned long long)P.block << 40) | (unsigned long long)(P.row0 + r));
  }

  // diagonal triangles: wave w < 4 that of U, else of L, of block b; lane j (of
  // each 16 lanes alike) column j
  const int o = kB * (w & 3), j = r & 15;
  T x[kB];
#pragma unroll
  for (int i = 0; i < kB; ++i) x[i] = i == j ? T(1) : T(0);
  if (w < 4) {
#pragma unroll
    for (int i = kB - 1; i >= 0; --i) {
      x[i] *= Rv[o + i];
#pragma unroll
      for (int m = 0; m < i; ++m) x[m] -= LU[o + m][o + i] * x[i];
    }
  } else {
#pragma unroll
    for (int i = 0; i < kB; ++i)
#pragma unroll
      for (int m = i + 1; m < kB; ++m) x[m] -= LU[o + m][o + i] * x[i];
  }
  __syncthreads();   // both triangles of a block are read
#pragma unroll
  for (int i = 0; i < kB; ++i)
    if (r < kB && (w < 4 ? i <= j : i > j)) LU[o + i][o + j] = x[i];
  __syncthreads();
  // entry (i, k) of the inverse of U (up) or of L on its diagonal blocks
  auto inv = [&](bool up, int i, int k) __attribute__((always_inline)) {
    const T v = LU[i][k], d = !up && i == k ? T(1) : T(0);
    return (up ? i <= k : i > k) ? v : d;
  };
  const int li = r & 15, lk = r >> 4;
  typedef typename Mma<T>::acc acc_t;
  // Off-diagonal block at (ro, co) of a triangle whose diagonal blocks start at
  // ro and at co: -inv(ro, ro) F inv(co, co), F the factor's entries there; here
  // the 16 x 16 part at (ti, tj) of blocks of size n, with the inner product in H.
  auto first = [&](bool up, int ro, int co, int n, int ti, int tj, T(*H)[kLdT]) __attribute__((always_inline)) {
    acc_t h = {};
#pragma unroll
    for (int s = 0; s < n; s += 4)
      h = Mma<T>::run(LU[ro + ti + li][co + s + lk], inv(up, co + s + lk, co + tj + li), h);
#pragma unroll
    for (int v = 0; v < 4; ++v) H[ti + Mma<T>::row(r, v)][tj + li] = h[v];
  };
  auto second = [&](bool up, int ro, int co, int n, int ti, int tj, T(*H)[kLdT]) __attribute__((always_inline)) {
    acc_t h = {};
#pragma unroll
    for (int s = 0; s < n; s += 4) h = Mma<T>::run(inv(up, ro + ti + li, ro + s + lk), H[s + lk][tj + li], h);
#pragma unroll
    for (int v = 0; v < 4; ++v) LU[ro + ti + Mma<T>::row(r, v)][co + tj + li] = -h[v];
  };
  // the 32 x 32 triangles: waves 0 and 1 of U, 2 and 3 of L, first and second
  if (w < 4) {
    const bool up = w < 2;
    const int o = 2 * kB * (w & 1), ro = up ? o : o + kB, co = up ? o + kB : o;
    T(*H)[kLdT] = &S.H[w >> 1][kB * (w & 1)];
    first(up, ro, co, kB, 0, 0, H);
    wave_sync();   // in FP32 a lane reads what other lanes stored to H
    second(up, ro, co, kB, 0, 0, H);
  }
  __syncthreads();
  // the whole: wave w takes the 16 x 16 block (ti, tj) of U's off-diagonal half
  // (w < 4) or of L's
  {
    const bool up = w < 4;
    const int ro = up ? 0 : 2 * kB, co = up ? 2 * kB : 0, ti = kB * (w >> 1 & 1), tj = kB * (w & 1);
    first(up, ro, co, 2 * kB, ti, tj, S.H[w >> 2 & 1]);
    __syncthreads();
    second(up, ro, co, 2 * kB, ti, tj, S.H[w >> 2 & 1]);
  }
  __syncthreads();
  // U^{-1} on and above the diagonal, L^{-1} strictly below it: each wave
  // writes kE of the 64 columns
#pragma unroll
  for (int cc = 0; cc < kE; ++cc) {
    const int c = kE * w + cc;
    D[c * ld + r] = LU[r][c];
  }
}

void launch_panel(int dtype, const PanelProb* probs, int nprob, const double* thresh,
                  unsigned long long* bad, hipStream_t s) {
  if (nprob <= 0) return;
  if (dtype == 0)
    hipLaunchKernelGGL(k_panel<double>, dim3(nprob), dim3(64 * kW), 0, s, probs, thresh, bad);
  else
    hipLaunchKernelGGL(k_panel<float>, dim3(nprob), dim3(64 * kW), 0, s, probs, thresh, bad);
}

}  // namespace ddps
