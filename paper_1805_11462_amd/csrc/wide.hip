// Products over many rows with a plain store for gfx950: the encoder's input projections of every position, the
// attention keys, and the embedding-gate table. The main loop is the generator's (wide_loop.h); the rows are those of
// a split operand, with a power of two of their own where they are embeddings (weights are in range only row by
// row), which are first copied into such an operand by token id (reading the 16-byte chunks of table rows inside the
// loop, 64 lines per load, took 65 us at 3840 x 1000 x 4000 bf16 and 215 at 20480 x 512 x 4096).
//
// Bound by the products: 20480 x 1024 x 4096, two terms, 340 us = 1.0 PFLOP/s of fp16 products; 3200 x 512 x 2048,
// three terms, 40 us (64 x 128 fp32 MFMA tiles 70).

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
  uint32_t woff[TN];
#pragma unroll
  for (int y = 0; y < TN; ++y)
    woff[y] = ((uint32_t)min(n0 / 16 + wave * TN + y, w.rows / 16 - 1) * w.kblocks + w.kb0) * (PB * 1024u) + lane * 16u;
  f32x4 c0[TM][TN], c1[TM][TN];
  wide_main<C>(smem, WideRows<C>(a.base, m0, nrb, kb),
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
      const int ae = a.aexp ? a.aexp[a.eidx ? a.eidx[m] : m] : 0;
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

// Position m = s * B + b of the batch: its id and length checked as in the host's validation (violations recorded
// in *err, the id 0 past the length or where invalid), the id kept in ids[m], the lengths in lens, and, for m < rows,
// the id's table row ([terms][32 kblocks] halfwords) copied into row m of the operand. A thread moves 16 bytes; a
// row's reads are consecutive. max_len (optional): the longest length. err and max_len are host-visible words.
__global__ __launch_bounds__(256) void k_embed_src(const int32_t* __restrict__ src, const int32_t* __restrict__ len,
                                                   int B, int S, int V, const uint4* __restrict__ table, int terms,
                                                   int kblocks, int32_t* __restrict__ ids, int32_t* __restrict__ lens,
                                                   uint16_t* __restrict__ out, int rows, int32_t* err,
                                                   int32_t* max_len) {
  if (max_len && blockIdx.x == 0) {
    __shared__ int longest;
    if (threadIdx.x == 0) longest = 1;
    __syncthreads();
    int v = 1;
    for (int b = threadIdx.x; b < B; b += blockDim.x) v = max(v, min(len[b], S));
    atomicMax(&longest, v);
    __syncthreads();
    if (threadIdx.x == 0) *max_len = longest;
  }
  const int cpt = kblocks * 4, cpr = cpt * terms;         // 16-byte chunks per term and per row
  const size_t n = (size_t)B * S * cpr;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const int m = (int)(i / cpr), c = (int)(i % cpr);
    const int s = m / B, b = m % B;
    const int l = len[b], lc = l < 1 ? 1 : (l > S ? S : l);
    int id = 0;
    if (s < lc) {
      id = src[(size_t)b * S + s];
      if (id < 0 || id >= V) {
        if (c == 0) *err = kErrSourceId;
        id = 0;
      }
    }
    if (c == 0) {
      ids[m] = id;
      if (s == 0) {
        lens[b] = lc;
        if (l != lc) *err = kErrLength;
      }
    }
    if (m < rows)
      *(uint4*)(out + split16_at(m, c % cpt * 8, kblocks, terms) + (size_t)(c / cpt) * kFragElems) =
          table[(size_t)id * cpr + c];
  }
}

// Row m < n of the operand = the table row of the (checked) id ids[m].
__global__ __launch_bounds__(256) void k_embed_rows(const int32_t* __restrict__ ids, int n,
                                                    const uint4* __restrict__ table, int terms, int kblocks,
                                                    uint16_t* __restrict__ out) {
  const int cpt = kblocks * 4, cpr = cpt * terms;
  const size_t total = (size_t)n * cpr;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
    const int m = (int)(i / cpr), c = (int)(i % cpr);
    *(uint4*)(out + split16_at(m, c % cpt * 8, kblocks, terms) + (size_t)(c / cpt) * kFragElems) =
        table[(size_t)ids[m] * cpr + c];
  }
}

hipError_t embed_rows(const int32_t* ids, int n, const void* table, int terms, int kblocks, uint16_t* out,
                      hipStream_t st) {
  size_t blocks = ((size_t)n * kblocks * 4 * terms + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL(k_embed_rows, dim3((unsigned)blocks), dim3(256), 0, st, ids, n, (const uint4*)table, terms,
                     kblocks, out);
  return hipGetLastError();
}

hipError_t embed_src(const int32_t* src, const int32_t* len, int B, int S, int V, const void* table, int terms,
                     int kblocks, int32_t* ids, int32_t* lens, uint16_t* out, int rows, int32_t* err,
                     int32_t* max_len, hipStream_t st) {
  const size_t n = (size_t)B * S * kblocks * 4 * terms;
  size_t blocks = (n + 255) / 256;
  if (blocks > 8192) blocks = 8192;
  hipLaunchKernelGGL(k_embed_src, dim3((unsigned)blocks), dim3(256), 0, st, src, len, B, S, V, (const uint4*)table,
                     terms, kblocks, ids, lens, out, rows, err, max_len);
  return hipGetLastError();
}

// Teacher-forced targets, checked and laid out per step: in_tok [T, B] the decoder's input (BOS, then the previous
// target; pad past the length), want [T, B] the target (0 past the length), tlen [B] the lengths clamped to [1, T].
__global__ __launch_bounds__(256) void k_targets(const int32_t* __restrict__ tgt, const int32_t* __restrict__ len, int B,
                                                 int T, int V, int bos, int pad, int32_t* __restrict__ in_tok,
                                                 int32_t* __restrict__ want, int32_t* __restrict__ tlen, int32_t* err,
                                                 int32_t* max_len) {
  if (blockIdx.x == 0) {
    __shared__ int longest;
    if (threadIdx.x == 0) longest = 1;
    __syncthreads();
    int v = 1;
    for (int b = threadIdx.x; b < B; b += blockDim.x) v = max(v, min(len[b], T));
    atomicMax(&longest, v);
    __syncthreads();
    if (threadIdx.x == 0) *max_len = longest;
  }
  const size_t n = (size_t)B * T;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const int t = (int)(i / B), b = (int)(i % B);
    const int l = len[b], lc = l < 1 ? 1 : (l > T ? T : l);
    if (t == 0) {
      tlen[b] = lc;
      if (l != lc) *err = kErrLength;
    }
    const bool on = t < lc;
    int v = on ? tgt[(size_t)b * T + t] : 0, prev = on && t > 0 ? tgt[(size_t)b * T + t - 1] : 0;
    if (v < 0 || v >= V) {
      *err = kErrToken;
      v = 0;
    }
    if (prev < 0 || prev >= V) prev = 0;
    in_tok[i] = !on ? pad : (t == 0 ? bos : prev);
    want[i] = v;
  }
}

hipError_t targets(const int32_t* tgt, const int32_t* len, int B, int T, int V, int bos, int pad, int32_t* in_tok,
                   int32_t* want, int32_t* tlen, int32_t* err, int32_t* max_len, hipStream_t st) {
  size_t blocks = ((size_t)B * T + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_targets, dim3((unsigned)blocks), dim3(256), 0, st, tgt, len, B, T, V, bos, pad, in_tok, want,
                     tlen, err, max_len);
  return hipGetLastError();
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
      p.ncols % 4 || p.ncols > w.rows || a.M > a.rows ||
      split16_bytes(a.rows, a.kblocks, a.terms) >= lim || split16_bytes(w.rows, w.kblocks, w_terms) >= lim)
    return hipErrorInvalidValue;
  if (a.terms == 2 && w_terms == 2) return wide_dispatch<2, 2>(a, w, p, st);
  if (a.terms == 2 && w_terms == 1) return wide_dispatch<2, 1>(a, w, p, st);
  if (a.terms == 1 && w_terms == 1) return wide_dispatch<1, 1>(a, w, p, st);
  return hipErrorInvalidValue;
}

}  // namespace onmt
