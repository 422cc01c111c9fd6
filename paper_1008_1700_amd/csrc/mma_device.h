// 16 x 16 products of four columns and four rows on the matrix cores, in FP64 and
// FP32: lane l gives a = A(l % 16, l / 16) and b = B(l / 16, l % 16).
#pragma once

namespace ddps {

typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <typename T> struct Mma;
// Accumulator layouts (lane l, register v) -> row of the 16 x 16 result:
// f32 16x16x4: 4 (l >> 4) + v;   f64 16x16x4: (l >> 4) + 4 v  (measured).
template <> struct Mma<double> {
  using acc = f64x4;
  static __device__ __forceinline__ int row(int lane, int v) { return (lane >> 4) + 4 * v; }
  static __device__ __forceinline__ acc run(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
};
template <> struct Mma<float> {
  using acc = f32x4;
  static __device__ __forceinline__ int row(int lane, int v) { return 4 * (lane >> 4) + v; }
  static __device__ __forceinline__ acc run(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
};

}  // namespace ddps
