// Sums over a wavefront's lanes by register exchanges (no LDS).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace qs {

// Both words of a double exchanged between registers a and b across halves (or
// odd and even rows of 16 lanes), then added: lanes 0-31 (even rows) hold a's
// partial sums, the others b's.
__device__ __forceinline__ double fold_halves(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)__double2loint(a), (uint32_t)__double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)__double2hiint(a), (uint32_t)__double2hiint(b), false, false);
  return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
__device__ __forceinline__ double fold_rows(double a, double b) {
  const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)__double2loint(a), (uint32_t)__double2loint(b), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)__double2hiint(a), (uint32_t)__double2hiint(b), false, false);
  return __hiloint2double((int)hi[0], (int)lo[0]) + __hiloint2double((int)hi[1], (int)lo[1]);
}
template <int kN>
__device__ __forceinline__ double add_row_ror(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x120 + kN, 0xf, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x120 + kN, 0xf, 0xf, false);
  return v + __hiloint2double(hi, lo);
}

// Four values summed over the wavefront's lanes at once.  Every lane of row r
// (16 lanes) holds the sum of value wave_sum4_value(lane); each sum is formed
// in the butterfly order of wave_sum_fixed (lane distances 32, 16, 8, 4, 2, 1).
__device__ __forceinline__ double wave_sum4(const double (&v)[4]) {
  double t = fold_rows(fold_halves(v[0], v[1]), fold_halves(v[2], v[3]));
  t = add_row_ror<8>(t);
  t = add_row_ror<4>(t);
  t = add_row_ror<2>(t);
  return add_row_ror<1>(t);
}
__device__ __forceinline__ uint32_t wave_sum4_value(uint32_t lane) {
  return ((lane >> 3) & 2u) | (lane >> 5);  // rows 0..3: values 0, 2, 1, 3
}

// The largest of m over the lanes l, l ^ 16, l ^ 32, l ^ 48, and over the wavefront.
__device__ __forceinline__ float rows_max(float m) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(m), __float_as_uint(m), false, false);
  m = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(m), __float_as_uint(m), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
template <int kN>
__device__ __forceinline__ float max_row_ror(float m) {
  return fmaxf(m, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(m), 0x120 + kN, 0xf, 0xf, false)));
}
__device__ __forceinline__ float wave_max(float m) {
  return max_row_ror<1>(max_row_ror<2>(max_row_ror<4>(max_row_ror<8>(rows_max(m)))));
}

}  // namespace qs
