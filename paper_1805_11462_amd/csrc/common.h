// Device-side building blocks shared by the gfx950 kernels of libonmt.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace onmt {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kWave = 64;
constexpr int kMaxBeam = 16;        // largest beam the register top-K lists support
constexpr int kUnitGroup = 8;       // LSTM units per gate block in packed weights (4 gates x 8 units = 32 columns)

// Round-to-nearest-even float -> bfloat16 bits (finite inputs).
__device__ __host__ inline uint16_t f32_to_bf16_bits(float f) {
  uint32_t u = __builtin_bit_cast(uint32_t, f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

__device__ inline float bf16_bits_to_f32(uint16_t h) {
  return __builtin_bit_cast(float, (uint32_t)h << 16);
}
inline float host_bf16_to_f32(uint16_t h) { return __builtin_bit_cast(float, (uint32_t)h << 16); }

__device__ inline float sigmoidf_(float x) { return 1.0f / (1.0f + __expf(-x)); }

// Order used by every top-K: larger value first, then smaller id (ids are unique, so this is total).
template <class V, class I>
__device__ inline bool before(V v, I id, V w, I jd) {
  return v > w || (v == w && id < jd);
}

// Broadcast of lane l's value (l uniform) through the scalar unit, no LDS round trip.
__device__ inline float readlane_f(float v, int l) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}
__device__ inline int readlane_i(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ inline double readlane_d(double v, int l) {
  const long long b = __builtin_bit_cast(long long, v);
  const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffLL), l);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), l);
  return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}
__device__ inline long long readlane_ll(long long v, int l) {
  const int lo = __builtin_amdgcn_readlane((int)(v & 0xffffffffLL), l);
  const int hi = __builtin_amdgcn_readlane((int)(v >> 32), l);
  return ((long long)hi << 32) | (unsigned int)lo;
}

// Reductions over groups of N consecutive lanes (N = 2 .. 64, a power of two) with DPP moves, which cost a few cycles
// each where a shuffle is a round trip through LDS: within rows of 16 lanes by shifts, then the rows' last lanes
// broadcast to the next row (row_bcast 15) and half (row_bcast 31). The last lane of each group ends up with the
// group's result. Every lane of the wave must be active.
template <int CTRL, int ROWS>
__device__ inline float dpp_move(float old, float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, old), __builtin_bit_cast(int, v),
                                                               CTRL, ROWS, 0xf, false));
}
template <int N>
__device__ inline float group_sum(float v) {
  if constexpr (N >= 2) v += dpp_move<0x111, 0xf>(0.f, v);
  if constexpr (N >= 4) v += dpp_move<0x112, 0xf>(0.f, v);
  if constexpr (N >= 8) v += dpp_move<0x114, 0xf>(0.f, v);
  if constexpr (N >= 16) v += dpp_move<0x118, 0xf>(0.f, v);
  if constexpr (N >= 32) v += dpp_move<0x142, 0xa>(0.f, v);
  if constexpr (N >= 64) v += dpp_move<0x143, 0xc>(0.f, v);
  return v;
}
// The same over the whole wave, the result in every lane.
__device__ inline float wave_max(float v) {
  v = fmaxf(v, dpp_move<0x111, 0xf>(v, v));
  v = fmaxf(v, dpp_move<0x112, 0xf>(v, v));
  v = fmaxf(v, dpp_move<0x114, 0xf>(v, v));
  v = fmaxf(v, dpp_move<0x118, 0xf>(v, v));
  v = fmaxf(v, dpp_move<0x142, 0xa>(v, v));
  v = fmaxf(v, dpp_move<0x143, 0xc>(v, v));
  return readlane_f(v, 63);
}
__device__ inline float wave_sum(float v) { return readlane_f(group_sum<64>(v), 63); }

}  // namespace onmt
