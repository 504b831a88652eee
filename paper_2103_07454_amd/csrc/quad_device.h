// Four consecutive elements a lane through bounded buffers, and the sum over a wavefront without LDS: what the update passes
// of kernels_walk.hip and kernels_parts.hip share.
#pragma once
#include "evg_device.h"

namespace evg {

constexpr int kNt = 2;                        // non-temporal
constexpr uint32_t kNowhere = 0xFFFFFFF0u;    // an offset past every window

struct Quad { float v[4]; };

template <bool STREAM>
__device__ __forceinline__ Quad load_quad(const float* at, uint32_t bytes, uint32_t byte) {
  const u32x4 t = __builtin_amdgcn_raw_buffer_load_b128(window(at, bytes), (int)byte, 0, STREAM ? kNt : 0);
  Quad q;
#pragma unroll
  for (int i = 0; i < 4; ++i) q.v[i] = __uint_as_float(t[i]);
  return q;
}
template <bool STREAM>
__device__ __forceinline__ void store_quad(float* at, uint32_t bytes, uint32_t byte, const Quad& q) {
  u32x4 t;
#pragma unroll
  for (int i = 0; i < 4; ++i) t[i] = __float_as_uint(q.v[i]);
  __builtin_amdgcn_raw_buffer_store_b128(t, window(at, bytes), (int)byte, 0, STREAM ? kNt : 0);
}

// The same of arrays of less than 4 GB at a byte offset of each lane's own: two scalar registers an array.
__device__ __forceinline__ Quad load_at(const float* a, uint32_t byte) {
  const f32x4 t = *reinterpret_cast<const f32x4*>(reinterpret_cast<const char*>(a) + byte);
  Quad q;
#pragma unroll
  for (int i = 0; i < 4; ++i) q.v[i] = t[i];
  return q;
}
__device__ __forceinline__ void store_at(float* a, uint32_t byte, const Quad& q) {
  f32x4 t;
#pragma unroll
  for (int i = 0; i < 4; ++i) t[i] = q.v[i];
  *reinterpret_cast<f32x4*>(reinterpret_cast<char*>(a) + byte) = t;
}
// ... and non-temporal.
__device__ __forceinline__ Quad load_nt_at(const float* a, uint32_t byte) {
  const f32x4 t = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(reinterpret_cast<const char*>(a) + byte));
  Quad q;
#pragma unroll
  for (int i = 0; i < 4; ++i) q.v[i] = t[i];
  return q;
}
__device__ __forceinline__ void store_nt_at(float* a, uint32_t byte, const Quad& q) {
  f32x4 t;
#pragma unroll
  for (int i = 0; i < 4; ++i) t[i] = q.v[i];
  __builtin_nontemporal_store(t, reinterpret_cast<f32x4*>(reinterpret_cast<char*>(a) + byte));
}
__device__ __forceinline__ double load_f64(const double* at, uint32_t bytes, uint32_t byte) {
  const auto t = __builtin_amdgcn_raw_buffer_load_b64(window(at, bytes), (int)byte, 0, 0);
  return __longlong_as_double((long long)(((uint64_t)t[1] << 32) | t[0]));
}
__device__ __forceinline__ double readlane_f64(double v, uint32_t l) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, (int)l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), (int)l);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// The sum of wave_sum, in its order of additions, without LDS: halves and rows change places for the
// first two steps; from then on a row's values repeat with the step's period, so that a rotation
// brings the same value as the exchange.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)b, CTRL, 0xF, 0xF, true);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(b >> 32), CTRL, 0xF, 0xF, true);
  return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
__device__ __forceinline__ double row_sum_dpp(double v) {
  v += dpp_f64<0x128>(v);   // row_ror:8
  v += dpp_f64<0x124>(v);   // row_ror:4
  v += dpp_f64<0x122>(v);   // row_ror:2
  v += dpp_f64<0x121>(v);   // row_ror:1
  return v;
}
__device__ __forceinline__ double wave_sum_dpp(double v) {
  uint64_t b = (uint64_t)__double_as_longlong(v);
  const auto l32 = __builtin_amdgcn_permlane32_swap((uint32_t)b, (uint32_t)b, false, false);
  const auto h32 = __builtin_amdgcn_permlane32_swap((uint32_t)(b >> 32), (uint32_t)(b >> 32), false, false);
  v = __longlong_as_double((long long)(((uint64_t)h32[0] << 32) | l32[0])) +
      __longlong_as_double((long long)(((uint64_t)h32[1] << 32) | l32[1]));
  b = (uint64_t)__double_as_longlong(v);
  const auto l16 = __builtin_amdgcn_permlane16_swap((uint32_t)b, (uint32_t)b, false, false);
  const auto h16 = __builtin_amdgcn_permlane16_swap((uint32_t)(b >> 32), (uint32_t)(b >> 32), false, false);
  v = __longlong_as_double((long long)(((uint64_t)h16[0] << 32) | l16[0])) +
      __longlong_as_double((long long)(((uint64_t)h16[1] << 32) | l16[1]));
  return row_sum_dpp(v);
}
// Four such sums at once, each in its own row of 16 lanes: in each of the first two steps two sums give each other the half, or
// the rows, that they add next, and go on in one register.
__device__ __forceinline__ double halves_added(double a, double b) {     // lanes 0 .. 31: of a, 32 .. 63: of b
  const uint64_t p = (uint64_t)__double_as_longlong(a), q = (uint64_t)__double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)p, (uint32_t)q, false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(p >> 32), (uint32_t)(q >> 32), false, false);
  return __longlong_as_double((long long)(((uint64_t)hi[0] << 32) | lo[0])) +
         __longlong_as_double((long long)(((uint64_t)hi[1] << 32) | lo[1]));
}
__device__ __forceinline__ double rows_added(double a, double b) {       // rows 0, 2: of a, 1, 3: of b
  const uint64_t p = (uint64_t)__double_as_longlong(a), q = (uint64_t)__double_as_longlong(b);
  const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)p, (uint32_t)q, false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(p >> 32), (uint32_t)(q >> 32), false, false);
  return __longlong_as_double((long long)(((uint64_t)hi[0] << 32) | lo[0])) +
         __longlong_as_double((long long)(((uint64_t)hi[1] << 32) | lo[1]));
}
__device__ __forceinline__ double wave_sums2(double a, double b) {       // lanes 0 .. 31: a, 32 .. 63: b
  const double v = halves_added(a, b);
  return row_sum_dpp(rows_added(v, v));
}
__device__ __forceinline__ double wave_sums4(double a, double b, double c, double d) {     // rows 0, 1, 2, 3: a, b, c, d
  return row_sum_dpp(rows_added(halves_added(a, c), halves_added(b, d)));
}

}  // namespace evg
