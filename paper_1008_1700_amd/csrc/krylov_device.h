// Device functions of the inner iteration that the vector kernels and the
// reduced products share.
#pragma once

#include "ddps_internal.h"

namespace ddps {

__device__ __forceinline__ double sum_of(const double* __restrict__ sums, int j, int q) {
  return sums[2 * j + q];
}

// The sums of a reduction for column j of R in every thread of a workgroup: read
// from `sums` when they have been reduced (W = 0), else added up from the
// [W][R][2] partials in the order of k_reduce2, the same in every workgroup, with
// the column's workgroup 0 leaving them in `sums` for later kernels.  For few
// partials this is quicker than a launch of its own (4.7 us and the gap before
// it).
__device__ __forceinline__ void take_sums(int W, int R, int j, const double* __restrict__ part,
                                          double* __restrict__ sums, double (&v)[2], double (*sh)[1][2]) {
  if (W == 0) {
    v[0] = sums[2 * j];
    v[1] = sums[2 * j + 1];
    return;
  }
  v[0] = v[1] = 0.0;
  for (int w = threadIdx.x; w < W; w += 256) {
    v[0] += part[((int64_t)w * R + j) * 2 + 0];
    v[1] += part[((int64_t)w * R + j) * 2 + 1];
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    double x = v[q];
    for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
    if (lane == 0) sh[wave][0][q] = x;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 2; ++q) v[q] = sh[0][0][q] + sh[1][0][q] + sh[2][0][q] + sh[3][0][q];
  __syncthreads();
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    sums[2 * j] = v[0];
    sums[2 * j + 1] = v[1];
  }
}

// Decisions of iteration `it` for column j, identical in every workgroup:
// they depend only on the status at the start of the iteration
// (status[it & 1], never written during the iteration) and reduced sums.
__device__ __forceinline__ bool s_ok(const KState* st, int it, int j, double rtv, double& alpha) {
  alpha = st->rho[it & 1][j] / rtv;
  return st->status[it & 1][j] == KS_RUNNING && rtv != 0.0 && isfinite(alpha);
}

}  // namespace ddps
