// Cross-lane sums in the vector pipeline (gfx950): DPP inside rows of 16
// lanes, v_permlane16_swap and v_permlane32_swap between them, so that no
// reduction waits on LDS.
#pragma once
#include <hip/hip_runtime.h>

#include "common.h"

namespace rg {

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(
      0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xf,
                                             0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xf,
                                             0xf, true);
  return __hiloint2double(hi, lo);
}
constexpr int DPP_XOR1 = 0xB1, DPP_XOR2 = 0x4E, DPP_HMIRROR = 0x141,
              DPP_ROR8 = 0x128;

// lanes below H (of each 2H) get a's sum over the two halves, the lanes
// above b's (H = 32 or 16)
template <int H>
__device__ __forceinline__ float fold(float a, float b) {
  if constexpr (H == 32) {
    const auto s = __builtin_amdgcn_permlane32_swap(
        __float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
  } else {
    const auto s = __builtin_amdgcn_permlane16_swap(
        __float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(s[0]) + __uint_as_float(s[1]);
  }
}
template <int H>
__device__ __forceinline__ double fold(double a, double b) {
  const unsigned al = (unsigned)__double2loint(a), ah = (unsigned)__double2hiint(a);
  const unsigned bl = (unsigned)__double2loint(b), bh = (unsigned)__double2hiint(b);
  if constexpr (H == 32) {
    const auto l = __builtin_amdgcn_permlane32_swap(al, bl, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(ah, bh, false, false);
    return __hiloint2double((int)h[0], (int)l[0]) +
           __hiloint2double((int)h[1], (int)l[1]);
  } else {
    const auto l = __builtin_amdgcn_permlane16_swap(al, bl, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(ah, bh, false, false);
    return __hiloint2double((int)h[0], (int)l[0]) +
           __hiloint2double((int)h[1], (int)l[1]);
  }
}
// the same over halves of 16 and of 8 lanes, by DPP
template <int CTRL, typename T>
__device__ __forceinline__ T fold_dpp(T a, T b, bool upper) {
  const T keep = upper ? b : a, give = upper ? a : b;
  return keep + dpp<CTRL>(give);
}
// Sum of one value over the wave, in every lane.
template <typename T>
__device__ __forceinline__ T wave_total(T v) {
  v += dpp<DPP_XOR1>(v);
  v += dpp<DPP_XOR2>(v);
  v += dpp<DPP_HMIRROR>(v);
  v += dpp<DPP_ROR8>(v);
  v = fold<16>(v, v);
  return fold<32>(v, v);
}
// Wave sums of N values: lane l ends with that of value l / (64 / N).
template <int N, typename T>
__device__ __forceinline__ T wave_totals(T (&v)[N], int lane) {
  static_assert(N == 2 || N == 4 || N == 8, "");
#pragma unroll
  for (int i = 0; i < N / 2; ++i) v[i] = fold<32>(v[i], v[i + N / 2]);
  if constexpr (N >= 4) {
#pragma unroll
    for (int i = 0; i < N / 4; ++i) v[i] = fold<16>(v[i], v[i + N / 4]);
  } else {
    v[0] = fold<16>(v[0], v[0]);
  }
  T s;
  if constexpr (N == 8) s = fold_dpp<DPP_ROR8>(v[0], v[1], (lane & 8) != 0);
  else s = v[0] + dpp<DPP_ROR8>(v[0]);
  s += dpp<DPP_HMIRROR>(s);
  s += dpp<DPP_XOR2>(s);
  return s + dpp<DPP_XOR1>(s);
}
// The value of lane K of each row of 16 lanes, in all lanes of the row.
template <int K>
__device__ __forceinline__ float row_value(float v) {
  return dpp<0x150 + K>(v);
}
template <int K>
__device__ __forceinline__ double row_value(double v) {
  const long x = __builtin_bit_cast(long, v);
  const long y =
      __builtin_amdgcn_update_dpp((long)0, x, 0x150 + K, 0xf, 0xf, true);
  return __builtin_bit_cast(double, y);
}

}  // namespace rg
