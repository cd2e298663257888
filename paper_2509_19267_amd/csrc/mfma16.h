// MFMA 16x16x4 in FP64 and FP32 (gfx950).  Operand layout of
// v_mfma_*_16x16x4 (both precisions): lane l supplies A[l % 16][l / 16] and
// B[l / 16][l % 16]; accumulator element r of lane l is
// D[row(l / 16, r)][l % 16], row = 4 (l / 16) + r for FP32 and 4 r + l / 16
// for FP64 (measured on gfx950).
#pragma once
#include <hip/hip_runtime.h>

namespace rg {

template <typename T> struct Mfma16;
template <> struct Mfma16<double> {
  typedef double v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ v4 mma(double a, double b, v4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lk, int r) { return 4 * r + lk; }
};
template <> struct Mfma16<float> {
  typedef float v4 __attribute__((ext_vector_type(4)));
  static __device__ __forceinline__ v4 mma(float a, float b, v4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int lk, int r) { return 4 * lk + r; }
};

}  // namespace rg
