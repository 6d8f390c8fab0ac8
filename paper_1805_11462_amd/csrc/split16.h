// Two-term fp16 operands of the MFMA products, in fragment blocks.
//
// Values: an fp32 value x is carried as hi = fp16(s) and lo = fp16((s - hi) 2^11) of s = x 2^e, round to
// nearest even each, so x = (hi + lo 2^-11) 2^-e to 22 significant bits or better (three values in four are
// exact to all 24). Activations are outputs of tanh and sigmoid or averages of them, at most 1 in size: their e =
// kActExp keeps the full precision down to 3.8e-6 and below that an absolute 9.1e-13 (2^-40), and leaves room up to
// 4094 for a caller that replaces the memory bank. A caller's own decoder state, which may hold anything, gets an
// exponent per row (k_prepare_step).
// Weights are scaled per row (e = the exponent that takes the row's largest value to [2^14, 2^15)), so every
// finite fp32 weight is in range; the kernels undo both scales in one ldexp per output. A product is
//   hi.hi + (hi.lo + lo.hi) 2^-11
// with the two parts in separate fp32 accumulators; lo.lo, below 2^-22 of the leading product, is dropped.
//
// Infinities: a product of an infinite term and the other operand's zero lo term is NaN, where the fp32 product is an
// infinity that its gate saturates at. An infinite weight, embedding or state element is therefore carried as the
// largest finite value of its sign, which the row's scale takes in; NaN stays NaN.
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
#include <string.h>

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

// An infinite value's largest finite stand-in (`step`: 1, or 0x10000 for values of bf16 precision).
__device__ __host__ inline float finite_or_nan(float x, uint32_t step = 1) {
  const uint32_t u = __builtin_bit_cast(uint32_t, x);
  return __builtin_bit_cast(float, (u & 0x7fffffffu) == 0x7f800000u ? u - step : u);
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

// ---- weight packing on the host (built for hosts with fp16 conversion instructions, so that the loops below are
// vectorized: 50000 rows of 500 values 0.39 -> 0.064 s)

// Row exponent: the largest finite magnitude of the row goes to [2^14, 2^15); 0 for a row without one.
inline int host_row_exp(const float* src, int w) {
  uint32_t m = 0;
  for (int j = 0; j < w; ++j) {      // magnitudes are ordered like their bits
    const uint32_t a = __builtin_bit_cast(uint32_t, src[j]) & 0x7fffffffu;
    const uint32_t f = a < 0x7f800000u ? a : 0u;
    m = f > m ? f : m;
  }
  if (m == 0) return 0;
  int ex = 0;
  frexpf(__builtin_bit_cast(float, m), &ex);
  return 15 - ex;
}

// The terms of n values scaled by 2^e (lo == nullptr: one term); n a multiple of 8, hi and lo in groups of 8 that are
// `stride` halfwords apart.
inline void host_split(const float* src, int n, int e, uint16_t* hi, uint16_t* lo, int stride) {
  const float f = ldexpf(1.f, e / 2), g = ldexpf(1.f, e - e / 2);      // 2^e itself may be out of range
  for (int j = 0; j < n; j += 8) {
    uint16_t h[8], l[8];
    for (int i = 0; i < 8; ++i) {
      const float s = src[j + i] * f * g;
      const _Float16 t = (_Float16)s;
      h[i] = __builtin_bit_cast(uint16_t, t);
      const _Float16 u = (_Float16)((s - (float)t) * kLoScale);
      l[i] = (h[i] & 0x7c00u) == 0x7c00u ? (uint16_t)0 : __builtin_bit_cast(uint16_t, u);
    }
    memcpy(hi + j / 8 * stride, h, sizeof h);
    if (lo) memcpy(lo + j / 8 * stride, l, sizeof l);
  }
}

// Packs row `r` (whole K blocks) of a weight matrix, scaled by its row exponent e.
inline void host_pack_row(uint16_t* dst, int r, int kblocks, int terms, const float* src, int e) {
  for (int b = 0; b < kblocks; ++b) {
    uint16_t* d = dst + split16_at(r, b * kFragK, kblocks, terms);
    host_split(src + b * kFragK, kFragK, e, d, terms == 2 ? d + kFragElems : nullptr, kFragRows * 8);
  }
}

}  // namespace onmt
