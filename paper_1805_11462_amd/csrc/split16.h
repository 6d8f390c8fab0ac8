// Two-term fp16 operands of the MFMA products, in fragment blocks.
//
// Values: an fp32 value x is carried as hi = fp16(s) and lo = fp16((s - hi) 2^11) of s = x 2^e, round to
// nearest even each, so x = (hi + lo 2^-11) 2^-e to 22 significant bits or better (three values in four are
// exact to all 24). Activations of the recurrences are outputs of tanh and sigmoid, at most 1 in size, but a
// caller's own state may hold more: e = kActExp takes values up to 4094 and keeps the full precision down to
// 3.8e-6, and below that an absolute 5e-13 (e = 10 stopped at 63.9: larger states became infinities).
// Weights are scaled per row (e = the exponent that takes the row's largest value to [2^14, 2^15)), so every
// finite fp32 weight is in range; the kernels undo both scales in one ldexp per output. A product is
//   hi.hi + (hi.lo + lo.hi) 2^-11
// with the two parts in separate fp32 accumulators; lo.lo, below 2^-22 of the leading product, is dropped.
//
// Layout: 16 rows x 32 columns form a block of 64 x 16 bytes, lane l = (k % 32 / 8) * 16 + r % 16 holding
// columns 8 (l / 16) .. + 7 of row l % 16: what lane l of v_mfma_f32_16x16x32_f16 takes. Blocks of a row
// block follow each other along K, the lo block right after its hi block. A wave thus loads a fragment with one
// contiguous 1 KB access (reading 16-byte chunks of row-major rows, 16 rows per access, a CU moved about 16
// bytes per clock instead of 40), LDS copies of a block are read without bank conflicts, and rows picked by a
// beam parent map still share cache lines, because a sentence's rows lie next to each other.
#pragma once

#include <math.h>
#include <stdint.h>

#include "common.h"

namespace onmt {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

constexpr int kActExp = 4;           // activations: e
constexpr int kLoExp = 11;           // the lo term's extra scale
constexpr float kLoScale = 2048.f;
constexpr int kFragRows = 16, kFragK = 32, kFragElems = kFragRows * kFragK;

// fp16 operand: `rows` rows (buffers hold whole 16-row blocks), kblocks blocks of 32 columns. Columns past
// the operand's width are zeros up to the last block's end.
struct Split16 {
  const void* base;
  int rows;
  int kblocks;
};

// Halfword index of (r, k)'s hi term; its lo term lies kFragElems further (terms = 2).
__host__ __device__ inline size_t split16_at(size_t r, int k, int kblocks, int terms) {
  return ((r / kFragRows) * kblocks + k / kFragK) * (size_t)(kFragElems * terms) + (k % kFragK / 8) * (kFragRows * 8) +
         (r % kFragRows) * 8 + k % 8;
}
inline size_t split16_bytes(size_t rows, int kblocks, int terms) {
  return (rows + kFragRows - 1) / kFragRows * kblocks * (size_t)(kFragElems * terms) * 2;
}

// The two terms of a scaled value. One past fp16's range becomes an infinity (with lo = 0, so that its
// products are infinities too, as they are for an infinite fp32 value), NaN stays NaN.
__device__ inline void split_scaled(float s, uint16_t& hi, uint16_t& lo) {
  const _Float16 h = (_Float16)s;
  const float d = fabsf((float)h) == __builtin_inff() ? 0.f : s - (float)h;
  const _Float16 l = (_Float16)(d * kLoScale);
  hi = __builtin_bit_cast(uint16_t, h);
  lo = __builtin_bit_cast(uint16_t, l);
}
// The two terms of an activation.
__device__ inline void split_act(float x, uint16_t& hi, uint16_t& lo) {
  split_scaled(x * (float)(1 << kActExp), hi, lo);
}

// float -> fp16 bits, round to nearest even, on the host (weight packing).
inline uint16_t host_f32_to_f16(float f) {
  uint32_t u = __builtin_bit_cast(uint32_t, f);
  const uint16_t sign = (uint16_t)((u >> 16) & 0x8000u);
  u &= 0x7fffffffu;
  if (u >= 0x7f800000u) return sign | (u > 0x7f800000u ? 0x7e00u : 0x7c00u);
  if (u >= 0x477ff000u) return sign | 0x7c00u;                     // rounds to 65536 or more
  if (u < 0x38800000u) {                                           // below 2^-14: a multiple of 2^-24
    const float a = __builtin_bit_cast(float, u) + 0.5f;           // ulp of [0.5, 1) is 2^-24: rounds to nearest even
    return sign | (uint16_t)(__builtin_bit_cast(uint32_t, a) - 0x3f000000u);
  }
  u += 0xfffu + ((u >> 13) & 1u);
  return sign | (uint16_t)((u - 0x38000000u) >> 13);
}
inline float host_f16_to_f32(uint16_t h) {
  const uint32_t sign = (uint32_t)(h & 0x8000u) << 16, e = (h >> 10) & 31u, m = h & 0x3ffu;
  if (e == 0) return __builtin_bit_cast(float, sign) + (sign ? -1.f : 1.f) * (float)m * 0x1p-24f;
  if (e == 31) return __builtin_bit_cast(float, sign | 0x7f800000u | (m << 13));
  return __builtin_bit_cast(float, sign | ((e + 112u) << 23) | (m << 13));
}

// The terms of a weight already scaled by its row exponent (lo == nullptr: one term).
inline void host_split(float s, uint16_t* hi, uint16_t* lo) {
  const uint16_t h = host_f32_to_f16(s);
  *hi = h;
  if (lo) *lo = (h & 0x7c00u) == 0x7c00u ? 0 : host_f32_to_f16((s - host_f16_to_f32(h)) * kLoScale);
}

// Packs row `r` (w columns at column k0) of a weight matrix already scaled by its row exponent e.
inline void host_pack_row(uint16_t* dst, int r, int k0, int kblocks, int terms, const float* src, int w, int e) {
  for (int j = 0; j < w; ++j) {
    const size_t at = split16_at(r, k0 + j, kblocks, terms);
    host_split(ldexpf(src[j], e), dst + at, terms == 2 ? dst + at + kFragElems : nullptr);
  }
}
// Row exponent: the largest finite magnitude of the row goes to [2^14, 2^15); 0 for a row without one.
inline int host_row_exp(const float* src, int w) {
  float m = 0.f;
  for (int j = 0; j < w; ++j) {
    const float a = fabsf(src[j]);
    if (a > m && a <= 3.402823466e38f) m = a;
  }
  if (!(m > 0.f)) return 0;
  int ex = 0;
  frexpf(m, &ex);
  return 15 - ex;
}

}  // namespace onmt
