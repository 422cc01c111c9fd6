// Kernels of the learned initial guess: a multilayer perceptron with bf16
// weights and activations and FP32 accumulation, trained with MSE and Adam
// (FP32 master weights), and the device plumbing that turns reduced vectors
// of a DDPS handle into network inputs and back.
//
// All matrices are row-major.  k_mlp_gemm computes C = op(A) op(B) on bf16
// MFMA 32x32x16 with arbitrary (ragged) M, N, K: out-of-range elements load
// as zero and are not stored.
#include "ddps_internal.h"
#include "ddps_mlp_internal.h"

namespace ddps {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Tile T x T (T = 32, 64 or 128), 256 threads = 4 waves (2 x 2), each a
// (T/2) x (T/2) sub-tile of 32 x 32 MFMA blocks (T = 32: one block, the first
// wave's; the other waves only bring its operands); K advances in chunks of
// BK = 8192 / T through LDS in layout [row][k] (k contiguous, padded by 4).  The
// products are small (a 512 x 512 layer is 64 tiles), so what bounds them is the
// latency of their loads: every thread has four 16-byte pieces of each operand
// of each of the next two chunks in flight.  With one chunk of 32 ahead the first
// layer of 512 rows (4098 x 512) took 73 us, the others 20 us; now 27 and 7 us.
// Every operand is read in pieces of 8 elements along its contiguous dimension:
// one 16-byte load where the base and the leading dimension keep 4-byte
// alignment and the piece is inside the matrix, else one element at a time.
// Rows past the edge are read from the last row and not stored; k past the edge
// is zero.
// Per output element the products are summed in the same K order whatever
// T is (16-deep MFMAs).
// MFMA operand X = A block (32 m x 16 k): lane l holds A[l%32][8(l/32)..+8);
// operand Y = B block (16 k x 32 n): lane l holds B[8(l/32)..+8)[l%32];
// register v of lane l is C[8(v/4) + 4(l/32) + v%4][l%32].
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));
typedef u16x8 __attribute__((aligned(4))) u16x8_a4;

// 8 elements p[0..8) (contiguous), the first `valid` of them in range
__device__ __forceinline__ u16x8 load_seg(const unsigned short* __restrict__ p, int valid, bool wide) {
  u16x8 r = {};
  if (wide && valid >= 8) r = *(const u16x8_a4*)p;
  else if (!wide || valid > 0) {
#pragma unroll
    for (int e = 0; e < 8; ++e) r[e] = e < valid ? p[e] : (unsigned short)0;
  }
  return r;
}

// The four pieces a thread takes of an operand's chunk [k0, k0 + BK): k
// contiguous (KC): row q / (BK/8), k 8 (q % (BK/8)), q = tid + 256 j; rows
// contiguous: k 4 (tid / (T/8)) + j, rows 8 (tid % (T/8)) .. + 7, so that a
// thread's pieces transpose into four-k pieces of eight rows.
template <bool KC, int T>
struct MlpOperand {
  static constexpr int BK = 8192 / T, LDK = BK + 4;
  u16x8 r[4];
  __device__ __forceinline__ void fetch(const unsigned short* __restrict__ X, int ld, int row0, int rows, int k0,
                                        int K, bool wide) {
    const int tid = threadIdx.x;
    const unsigned short* p[4];
    int valid[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (KC) {
        const int q = tid + 256 * j, m = min(row0 + q / (BK / 8), rows - 1), k = k0 + 8 * (q % (BK / 8));
        p[j] = X + (int64_t)m * ld + k;
        valid[j] = K - k;
      } else {
        const int k = k0 + 4 * (tid / (T / 8)) + j, m = row0 + 8 * (tid % (T / 8));
        p[j] = X + (int64_t)k * ld + m;
        valid[j] = k < K ? rows - m : 0;
      }
    }
    if (wide && k0 + BK <= K && (KC || row0 + T <= rows)) {
#pragma unroll
      for (int j = 0; j < 4; ++j) r[j] = *(const u16x8_a4*)p[j];
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) r[j] = load_seg(p[j], valid[j], wide);
    }
  }
  __device__ __forceinline__ void stage(unsigned short (*S)[LDK]) const {
    const int tid = threadIdx.x;
    if (KC) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int q = tid + 256 * j;
        unsigned short* d = &S[q / (BK / 8)][8 * (q % (BK / 8))];
        *(u16x4*)d = __builtin_shufflevector(r[j], r[j], 0, 1, 2, 3);
        *(u16x4*)(d + 4) = __builtin_shufflevector(r[j], r[j], 4, 5, 6, 7);
      }
    } else {
      const int k = 4 * (tid / (T / 8)), m = 8 * (tid % (T / 8));
#pragma unroll
      for (int e = 0; e < 8; ++e) *(u16x4*)&S[m + e][k] = u16x4{r[0][e], r[1][e], r[2][e], r[3][e]};
    }
  }
};

template <bool TA, bool TB, int T>
__global__ __launch_bounds__(256) void k_mlp_gemm(int M, int N, int K, const __bf16* __restrict__ A_, int lda,
                                                  const __bf16* __restrict__ B_, int ldb,
                                                  const float* __restrict__ bias, const float* __restrict__ gate,
                                                  int epi, float* __restrict__ Cf, __bf16* __restrict__ Cb, int ldc,
                                                  bool wa, bool wb) {
  constexpr int BK = 8192 / T, LDK = BK + 4;
  constexpr int WB = T == 128 ? 2 : 1;    // 32 x 32 blocks per wave and dimension
  constexpr int WS = 32 * WB;             // rows and columns of a wave's sub-tile
  __shared__ __attribute__((aligned(16))) unsigned short As[T][LDK];
  __shared__ __attribute__((aligned(16))) unsigned short Bs[T][LDK];
  const unsigned short* A = (const unsigned short*)A_;
  const unsigned short* B = (const unsigned short*)B_;
  const int m0 = blockIdx.x * T, n0 = blockIdx.y * T;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = T == 32 ? 0 : wave & 1, wn = T == 32 ? 0 : wave >> 1;
  const bool works = T > 32 || wave == 0;
  f32x16 acc[WB][WB];
#pragma unroll
  for (int i = 0; i < WB; ++i)
#pragma unroll
    for (int j = 0; j < WB; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  MlpOperand<!TA, T> ra[2];
  MlpOperand<TB, T> rb[2];
  auto fetch = [&](int s, int k0) __attribute__((always_inline)) {
    ra[s].fetch(A, lda, m0, M, k0, K, wa);
    rb[s].fetch(B, ldb, n0, N, k0, K, wb);
  };
  auto frag = [&](const unsigned short* p) __attribute__((always_inline)) {
    const u16x4 a = *(const u16x4*)p, b = *(const u16x4*)(p + 4);
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  auto chunk = [&](int s, int k0) __attribute__((always_inline)) {
    __syncthreads();   // every wave is done with the previous chunk
    ra[s].stage(As);
    rb[s].stage(Bs);
    __syncthreads();
    if (k0 + 2 * BK < K) fetch(s, k0 + 2 * BK);
    auto step = [&](int ks) __attribute__((always_inline)) {
      const int kk = ks + 8 * (lane >> 5);
      bf16x8 x[WB], y[WB];
#pragma unroll
      for (int i = 0; i < WB; ++i) x[i] = frag(&As[wm * WS + 32 * i + (lane & 31)][kk]);
#pragma unroll
      for (int j = 0; j < WB; ++j) y[j] = frag(&Bs[wn * WS + 32 * j + (lane & 31)][kk]);
#pragma unroll
      for (int i = 0; i < WB; ++i)
#pragma unroll
        for (int j = 0; j < WB; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[i], y[j], acc[i][j], 0, 0, 0);
    };
    if (!works) return;
    // a whole chunk without tests between its steps, so that their LDS reads
    // go ahead of the products
    if (K - k0 >= BK) {
#pragma unroll
      for (int ks = 0; ks < BK; ks += 16) step(ks);
    } else {
#pragma unroll 1
      for (int ks = 0; ks < K - k0; ks += 16) step(ks);
    }
  };
  if (K > 0) fetch(0, 0);
  if (K > BK) fetch(1, BK);
  for (int k0 = 0; k0 < K; k0 += 2 * BK) {
    chunk(0, k0);
    if (k0 + BK < K) chunk(1, k0 + BK);
  }
  if (!works) return;
#pragma unroll
  for (int i = 0; i < WB; ++i)
#pragma unroll
    for (int j = 0; j < WB; ++j) {
      const int n = n0 + wn * WS + 32 * j + (lane & 31);
      const int mb = m0 + wm * WS + 32 * i + 4 * (lane >> 5);
      float zg[16];
      if (epi & MLP_GATE) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int m = mb + 8 * (v >> 2) + (v & 3);
          zg[v] = m < M && n < N ? gate[(int64_t)m * ldc + n] : 0.f;
        }
      }
      const float bn = (epi & MLP_BIAS) && n < N ? bias[n] : 0.f;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int m = mb + 8 * (v >> 2) + (v & 3);
        if (m < M && n < N) {
          float z = acc[i][j][v];
          if (epi & MLP_BIAS) z += bn;
          if (epi & MLP_F32) Cf[(int64_t)m * ldc + n] = z;
          if (epi & MLP_RELU_BF16) Cb[(int64_t)m * ldc + n] = (__bf16)fmaxf(z, 0.f);
          if (epi & MLP_GATE) Cb[(int64_t)m * ldc + n] = (__bf16)(zg[v] > 0.f ? z : 0.f);
        }
      }
    }
}

__global__ void k_f32_to_bf16(int64_t n, const float* __restrict__ x, __bf16* __restrict__ y) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    y[i] = (__bf16)x[i];
}

// dY = 2 (Y - T) / (rows * cols) in bf16, with per-block partial sums of (Y-T)^2
__global__ __launch_bounds__(256) void k_mse(int64_t n, float scale, const float* __restrict__ Y,
                                             const float* __restrict__ T, __bf16* __restrict__ dY,
                                             double* __restrict__ part) {
  __shared__ double sh[256];
  double acc = 0.0;
#pragma unroll 4
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const float d = Y[i] - T[i];
    dY[i] = (__bf16)(2.f * d * scale);
    acc += (double)d * d;
  }
  sh[threadIdx.x] = acc;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) part[blockIdx.x] = sh[0];
}

// db[c] = sum over rows of dZ[r][c] (bf16 input, FP32 sums) of every layer, one
// launch for all of them (four launches of 4 us each otherwise).  A workgroup
// takes 64 columns of a layer (one wave reads 64 consecutive entries of a row);
// its 16 row groups g sum rows g, g + 16, ... in order, and the 16 partial sums
// are added pairwise in a fixed tree, so the result does not depend on timing.
constexpr int kBiasGroups = 16;
__global__ __launch_bounds__(64 * kBiasGroups) void k_bias_grad(int rows, MlpBiasGrad G) {
  __shared__ float part[kBiasGroups][64];
  int l = 0, wg = blockIdx.x;
  while (l < 3 && wg >= (G.cols[l] + 63) / 64) wg -= (G.cols[l++] + 63) / 64;
  const int cols = G.cols[l];
  const __bf16* __restrict__ dZ = G.dZ[l];
  const int lc = threadIdx.x & 63, g = threadIdx.x >> 6;
  const int c = wg * 64 + lc;
  float s = 0.f;
  if (c < cols)
#pragma unroll 8
    for (int r = g; r < rows; r += kBiasGroups) s += (float)dZ[(int64_t)r * cols + c];
  part[g][lc] = s;
  __syncthreads();
  for (int h = kBiasGroups / 2; h > 0; h >>= 1) {
    if (g < h) part[g][lc] += part[g + h][lc];
    __syncthreads();
  }
  if (g == 0 && c < cols) G.db[l][c] = part[0][lc];
}

// Adam (Kingma & Ba 2015, Algorithm 1) on FP32 master parameters; the bf16
// copy used by the products is refreshed in the same pass.
__global__ void k_adam(int64_t n, float lr, float b1, float b2, float eps, float c1, float c2,
                       float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m,
                       float* __restrict__ v, __bf16* __restrict__ pb) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float pi = p[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    p[i] = pi;
    if (pb) pb[i] = (__bf16)pi;
  }
}

// ------------------------------------------------------------ guess plumbing
// Interface j of the reduced vector holds its 2t entries at [2 j t, 2 (j+1) t).
// Features of interface j: [r_j / s_j, z^prev_j / q_j, cos, sin, 0 ...] with
// s_j = max |r_j| and q_j = max |z^prev_j| on c (each 1 where the vector is
// zero); one row of d_in floats per interface.
__device__ double block_absmax(const double* v, const double* mk, int t2, double* red) {
  double mx = 0.0;
  for (int i = threadIdx.x; i < t2; i += blockDim.x) mx = fmax(mx, fabs(v[i] * (mk ? mk[i] : 1.0)));
  red[threadIdx.x] = mx;
  __syncthreads();
  for (int q = 128; q > 0; q >>= 1) {
    if ((int)threadIdx.x < q) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + q]);
    __syncthreads();
  }
  const double r = red[0] > 1e-300 ? red[0] : 1.0;
  __syncthreads();
  return r;
}

__global__ __launch_bounds__(256) void k_features(int nif, int t2, int d_in, const double* __restrict__ rr,
                                                  const double* __restrict__ zp, const double* __restrict__ mask,
                                                  double c, double s, float* __restrict__ X,
                                                  float* __restrict__ scale) {
  __shared__ double red[256];
  const int j = blockIdx.x;   // interface (j % nif) of right-hand side j / nif
  const double* r = rr + (int64_t)j * t2;
  const double* z = zp + (int64_t)j * t2;
  const double* mk = mask + (int64_t)(j % nif) * t2;
  const double sc = block_absmax(r, nullptr, t2, red);
  const double qc = block_absmax(z, mk, t2, red);
  float* x = X + (int64_t)j * d_in;
  for (int i = threadIdx.x; i < d_in; i += blockDim.x) {
    double v = 0.0;
    if (i < t2) v = r[i] / sc;
    else if (i < 2 * t2) v = z[i - t2] * mk[i - t2] / qc;
    else if (i == 2 * t2) v = c;
    else if (i == 2 * t2 + 1) v = s;
    x[i] = (float)v;
  }
  if (threadIdx.x == 0) scale[j] = (float)sc;
}

// z0 = (z^prev + s_j * Y_j) * mask; vectors of mc entries per right-hand side
__global__ void k_compose(int64_t m, int64_t mc, int t2, const double* __restrict__ zp, const float* __restrict__ Y,
                          const float* __restrict__ scale, const double* __restrict__ mask, double* __restrict__ z0) {
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < m; q += (int64_t)gridDim.x * blockDim.x) {
    const int64_t j = q / t2;
    z0[q] = (zp[q] + (double)scale[j] * (double)Y[q]) * mask[q % mc];
  }
}

// target of interface j: (z^_j - z^prev_j) / s_j
__global__ void k_target(int64_t m, int64_t mc, int t2, const double* __restrict__ zh, const double* __restrict__ zp,
                         const float* __restrict__ scale, const double* __restrict__ mask, float* __restrict__ T) {
  for (int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; q < m; q += (int64_t)gridDim.x * blockDim.x) {
    const int64_t j = q / t2;
    T[q] = (float)((zh[q] - zp[q] * mask[q % mc]) / (double)scale[j]);
  }
}

// ------------------------------------------------------------ launchers
static unsigned grid1(int64_t n) { return (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 4096)); }

template <bool TA, bool TB>
static void mlp_gemm_t(int M, int N, int K, const __bf16* A, int lda, const __bf16* B, int ldb, const float* bias,
                       const float* gate, int epi, float* Cf, __bf16* Cb, int ldc, hipStream_t s) {
  // wide loads: every piece starts on 4 bytes
  const bool wa = lda % 2 == 0 && (uintptr_t)A % 4 == 0, wb = ldb % 2 == 0 && (uintptr_t)B % 4 == 0;
  // 128 x 128 tiles where they still give every CU at least two workgroups;
  // 32 x 32 where 64 x 64 would leave half of the CUs idle (a 512 x 512 layer
  // with 4098 inputs takes 40 us on 64 tiles of 64, 30 us on 256 of 32; a whole
  // epoch of 32 steps of 512 rows 6.90 and 6.42 ms, of 700 rows, where the
  // layers have 88 tiles of 64, 7.96 and 7.57 ms)
  const int64_t big = (int64_t)((M + 127) / 128) * ((N + 127) / 128);
  if (big >= 512) {
    const dim3 g((M + 127) / 128, (N + 127) / 128);
    hipLaunchKernelGGL((k_mlp_gemm<TA, TB, 128>), g, dim3(256), 0, s, M, N, K, A, lda, B, ldb, bias, gate, epi, Cf, Cb,
                       ldc, wa, wb);
  } else if ((int64_t)((M + 63) / 64) * ((N + 63) / 64) <= 128) {
    const dim3 g((M + 31) / 32, (N + 31) / 32);
    hipLaunchKernelGGL((k_mlp_gemm<TA, TB, 32>), g, dim3(256), 0, s, M, N, K, A, lda, B, ldb, bias, gate, epi, Cf, Cb,
                       ldc, wa, wb);
  } else {
    const dim3 g((M + 63) / 64, (N + 63) / 64);
    hipLaunchKernelGGL((k_mlp_gemm<TA, TB, 64>), g, dim3(256), 0, s, M, N, K, A, lda, B, ldb, bias, gate, epi, Cf, Cb,
                       ldc, wa, wb);
  }
}

void mlp_gemm(bool ta, bool tb, int M, int N, int K, const __bf16* A, int lda, const __bf16* B, int ldb,
              const float* bias, const float* gate, int epi, float* Cf, __bf16* Cb, int ldc, hipStream_t s) {
  if (M <= 0 || N <= 0) return;
  if (!ta && !tb) mlp_gemm_t<false, false>(M, N, K, A, lda, B, ldb, bias, gate, epi, Cf, Cb, ldc, s);
  else if (ta && !tb) mlp_gemm_t<true, false>(M, N, K, A, lda, B, ldb, bias, gate, epi, Cf, Cb, ldc, s);
  else mlp_gemm_t<false, true>(M, N, K, A, lda, B, ldb, bias, gate, epi, Cf, Cb, ldc, s);
}
void mlp_to_bf16(int64_t n, const float* x, __bf16* y, hipStream_t s) {
  hipLaunchKernelGGL(k_f32_to_bf16, dim3(grid1(n)), dim3(256), 0, s, n, x, y);
}
int mlp_mse(int64_t n, float scale, const float* Y, const float* T, __bf16* dY, double* part, hipStream_t s) {
  const int W = (int)std::min<int64_t>((n + 255) / 256, 256);
  hipLaunchKernelGGL(k_mse, dim3(W), dim3(256), 0, s, n, scale, Y, T, dY, part);
  return W;
}
void mlp_bias_grad(int rows, const MlpBiasGrad& G, hipStream_t s) {
  int wgs = 0;
  for (int l = 0; l < 4; ++l) wgs += (G.cols[l] + 63) / 64;
  hipLaunchKernelGGL(k_bias_grad, dim3(wgs), dim3(64 * kBiasGroups), 0, s, rows, G);
}
void mlp_adam(int64_t n, float lr, float b1, float b2, float eps, int t, float* p, const float* g, float* m,
              float* v, __bf16* pb, hipStream_t s) {
  const float c1 = 1.f - powf(b1, (float)t), c2 = 1.f - powf(b2, (float)t);
  hipLaunchKernelGGL(k_adam, dim3(grid1(n)), dim3(256), 0, s, n, lr, b1, b2, eps, c1, c2, p, g, m, v, pb);
}
void guess_features(int nif, int k, int t2, int d_in, const double* rr, const double* zp, const double* mask,
                    double c, double sn, float* X, float* scale, hipStream_t s) {
  hipLaunchKernelGGL(k_features, dim3(nif * k), dim3(256), 0, s, nif, t2, d_in, rr, zp, mask, c, sn, X, scale);
}
void guess_compose(int64_t m, int64_t mc, int t2, const double* zp, const float* Y, const float* scale,
                   const double* mask, double* z0, hipStream_t s) {
  hipLaunchKernelGGL(k_compose, dim3(grid1(m)), dim3(256), 0, s, m, mc, t2, zp, Y, scale, mask, z0);
}
void guess_target(int64_t m, int64_t mc, int t2, const double* zh, const double* zp, const float* scale,
                  const double* mask, float* T, hipStream_t s) {
  hipLaunchKernelGGL(k_target, dim3(grid1(m)), dim3(256), 0, s, m, mc, t2, zh, zp, scale, mask, T);
}

}  // namespace ddps
