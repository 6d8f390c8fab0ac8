// Products over many rows with a plain store for gfx950: the encoder's input projections of every position, the
// attention keys, and the embedding-gate table. The main loop is the generator's (wide_loop.h); rows are either
// consecutive rows of a two-term activation operand or rows of an embedding table picked by token id, which carry
// a power of two of their own (weights are in range only row by row).
//
// Bounds: at the default batch (3200 positions x 512 x 2048, fp32) the products take 17 us at the rate a large
// library product reaches as three fp16 terms; a 64 x 128 fp32 MFMA tile took 70.

#include "common.h"
#include "gemm_device.h"
#include "kernels.h"
#include "split16.h"
#include "wide_loop.h"

namespace onmt {

template <class C>
__global__ __launch_bounds__(C::NT, 2) void k_wide_store(WideA a, ThinW w, WideOut p, int nm, int nblocks) {
  constexpr int TM = C::TM, TN = C::TN, PA = C::PA, PB = C::PB;
  __shared__ __attribute__((aligned(16))) char smem[C::LDS];
  const int L = xcd_remap(blockIdx.x, nblocks);
  const int m0 = (L % nm) * C::BM, n0 = (L / nm) * C::BN;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i16 = lane & 15, g = lane >> 4;
  const int kb = a.kblocks, nrb = (a.rows + 15) / 16;
  uint32_t aoff[C::LPA], woff[TN];
  if (a.idx) {              // rows by id (clamped to the table): the lane's 16 bytes of its block row
#pragma unroll
    for (int i = 0; i < C::LPA; ++i) {
      const int q = wide_block<C>(wave, i);
      const int m = min(m0 + q / PA * 16 + i16, a.M - 1);
      const uint32_t r = min((uint32_t)a.idx[m], (uint32_t)a.rows - 1u);
      aoff[i] = (r / 16) * kb * (PA * 1024u) + (q % PA) * 1024u + g * 256u + (r % 16) * 16u;
    }
  } else {
    wide_rows<C>(m0, nrb, kb, aoff);
  }
#pragma unroll
  for (int y = 0; y < TN; ++y)
    woff[y] = ((uint32_t)min(n0 / 16 + wave * TN + y, w.rows / 16 - 1) * w.kblocks + w.kb0) * (PB * 1024u) + lane * 16u;
  f32x4 c0[TM][TN], c1[TM][TN];
  wide_main<C>(smem, make_rsrc(a.base, (uint32_t)nrb * kb * (PA * 1024u)), aoff,
               make_rsrc(w.base, (uint32_t)(w.rows / 16) * w.kblocks * (PB * 1024u)), woff, kb, c0, c1);
#pragma unroll
  for (int y = 0; y < TN; ++y) {
    const int col = n0 + wave * 16 * TN + 16 * y + 4 * g;
    if (col >= p.ncols) continue;                      // ncols is a multiple of 4
    const int4 ex = *(const int4*)(w.wexp + col);
    const float4 bias = p.bias ? *(const float4*)(p.bias + col) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int x = 0; x < TM; ++x) {
      const int m = m0 + 16 * x + i16;
      if (m >= a.M) continue;
      const int ae = a.aexp ? a.aexp[a.idx ? min((uint32_t)a.idx[m], (uint32_t)a.rows - 1u) : (uint32_t)m] : 0;
      f32x4 v;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        v[j] = PA * PB > 1 ? fmaf(c1[x][y][j], 1.f / kLoScale, c0[x][y][j]) : c0[x][y][j];
      const size_t row = p.B ? (size_t)(m % p.B) * p.S + m / p.B : (size_t)m;
      *(float4*)(p.out + row * p.ldo + col) =
          make_float4(ldexpf(v[0], ex.x + ae) + bias.x, ldexpf(v[1], ex.y + ae) + bias.y,
                      ldexpf(v[2], ex.z + ae) + bias.z, ldexpf(v[3], ex.w + ae) + bias.w);
    }
  }
}

template <class C>
static hipError_t launch_wide(const WideA& a, const ThinW& w, const WideOut& p, hipStream_t st) {
  const int nm = (a.M + C::BM - 1) / C::BM, nb = nm * ((w.rows + C::BN - 1) / C::BN);
  hipLaunchKernelGGL(k_wide_store<C>, dim3(nb), dim3(C::NT), 0, st, a, w, p, nm, nb);
  return hipGetLastError();
}

// 64 x 256 tiles, or 64 x 128 where those leave fewer than two workgroups per CU (the keys: 3200 x 512 x 512 gives
// 100 tiles of 64 x 256).
template <int PA, int PB>
static hipError_t wide_dispatch(const WideA& a, const ThinW& w, const WideOut& p, hipStream_t st) {
  const long tiles = (long)((a.M + 63) / 64) * ((w.rows + 255) / 256);
  if (tiles < 512) return launch_wide<WideTile<4, 2, PA, PB, 4, 3>>(a, w, p, st);
  return launch_wide<WideTile<4, 4, PA, PB, 3, 2>>(a, w, p, st);
}

hipError_t wide_store(const WideA& a, const ThinW& w, int w_terms, const WideOut& p, hipStream_t st) {
  const uint64_t lim = 1ull << 32;          // 32-bit byte offsets
  if (a.M < 1 || a.rows < 1 || a.kblocks < 1 || w.kb0 < 0 || w.kb0 + a.kblocks > w.kblocks || w.rows % 128 ||
      p.ncols % 4 || p.ncols > w.rows || (!a.idx && a.M > a.rows) ||
      split16_bytes(a.rows, a.kblocks, a.terms) >= lim || split16_bytes(w.rows, w.kblocks, w_terms) >= lim)
    return hipErrorInvalidValue;
  if (a.terms == 2 && w_terms == 2) return wide_dispatch<2, 2>(a, w, p, st);
  if (a.terms == 2 && w_terms == 1) return wide_dispatch<2, 1>(a, w, p, st);
  if (a.terms == 1 && w_terms == 1) return wide_dispatch<1, 1>(a, w, p, st);
  return hipErrorInvalidValue;
}

}  // namespace onmt
