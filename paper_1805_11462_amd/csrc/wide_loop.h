// Main loop of the GEMMs over many rows (the generator, the encoder's projections and keys): 16 TM x 64 TN tiles of
// four waves that each take all 16 TM rows and 16 TN columns, operands as split fp16 terms in fragment blocks (split16.h).
//
// A wave's weights are its own, so they go straight into registers, and LDS holds the rows all four waves read, moved
// there by LDS-destination loads: with both operands in LDS its bandwidth was the bound (reads plus stage writes 90% of
// 128 bytes per clock at 160 x 128 tiles). Weights have D register sets and rows NSTG buffers, but a stage's barrier
// lets only (NSTG - 2) LPA loads of either kind stay outstanding, since one counter holds both, and the compiler may
// place a stage's weight loads behind its products: about one stage is in flight whatever D and NSTG are. The tile
// shapes and limits that were measured (gen_wide_tm, k_thin_lstm_wide, wide_dispatch) hold for this loop.
#pragma once

#include "common.h"
#include "gemm_device.h"
#include "split16.h"

namespace onmt {

// PA, PB: terms of the rows and of the weights.
template <int TM_, int TN_, int PA_, int PB_, int NSTG_, int D_>
struct WideTile {
  static constexpr int TM = TM_, TN = TN_, PA = PA_, PB = PB_, NSTG = NSTG_, D = D_;
  static constexpr int BM = 16 * TM, BN = 64 * TN, NT = 256;
  static constexpr int LPA = (PA * TM + 3) / 4;               // 1 KB A loads per wave and stage
  static constexpr int STG = PA * TM * 1024;
  static constexpr int LDS = NSTG * STG;
};

// Block q = (row block, term) of a stage that load i of this wave moves (past the last: the last again).
template <class C>
__device__ __forceinline__ int wide_block(int wave, int i) {
  return min(wave + 4 * i, C::PA * C::TM - 1);
}

// Byte offsets of the wave's A loads at K block 0 for consecutive rows from m0 on: whole 1 KB blocks; row blocks
// past the operand's last re-read that (those rows are never stored).
template <class C>
__device__ __forceinline__ void wide_rows(int m0, int nrb, int kb, uint32_t (&aoff)[C::LPA]) {
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#pragma unroll
  for (int i = 0; i < C::LPA; ++i) {
    const int q = wide_block<C>(wave, i);
    aoff[i] = (uint32_t)min(m0 / 16 + q / C::PA, nrb - 1) * kb * (C::PA * 1024u) + (q % C::PA) * 1024u + lane * 16u;
  }
}

// load_a for such rows.
template <class C>
struct WideRows {
  __amdgpu_buffer_rsrc_t ra;
  uint32_t off[C::LPA];
  int wave;
  __device__ __forceinline__ WideRows(const void* base, int m0, int nrb, int kb)
      : ra(make_rsrc(base, (uint32_t)nrb * kb * (C::PA * 1024u))),
        wave(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) {
    wide_rows<C>(m0, nrb, kb, off);
  }
  __device__ __forceinline__ void operator()(int st, char* base) const {
#pragma unroll
    for (int i = 0; i < C::LPA; ++i)
      dma16(ra, base + wide_block<C>(wave, i) * 1024, off[i], (uint32_t)st * (C::PA * 1024u));
  }
};

// c0: sums of the leading products, c1: of the others (scaled by 2^kLoExp). load_a(st, base): moves the wave's A blocks
// of K block st (one of the operand's) to base. woff: byte offsets of the wave's 16-column weight blocks at the first
// K block. The weights are the MFMA's row operand: a lane ends up with four consecutive columns (16 y + 4 g + v) of row
// 16 x + i16. Every load has landed on return, behind a barrier.
template <class C, class LoadA>
__device__ __forceinline__ void wide_main(char* smem, LoadA load_a, __amdgpu_buffer_rsrc_t rw,
                                          const uint32_t (&woff)[C::TN], int kb, f32x4 (&c0)[C::TM][C::TN],
                                          f32x4 (&c1)[C::TM][C::TN]) {
  constexpr int TM = C::TM, TN = C::TN, PA = C::PA, PB = C::PB, NSTG = C::NSTG, D = C::D;
  const int lane = threadIdx.x & 63;
  // stages past the last re-load it into a buffer that is never read
  auto issue_a = [&](int st) { load_a(min(st, kb - 1), smem + (st % NSTG) * C::STG); };
  // stages past the last read zeros, so the loop runs whole groups of D stages (the A buffer then holds a copy
  // of the last stage: finite or, where the operand is not, as in the products before)
  uint4 wr[D][TN][PB];
  auto load_w = [&](int st, uint4 (&r)[TN][PB]) {
    const bool on = st < kb;
#pragma unroll
    for (int y = 0; y < TN; ++y)
#pragma unroll
      for (int pb = 0; pb < PB; ++pb)
        r[y][pb] = buf_load16s(rw, on ? woff[y] : kPastEnd, on ? (uint32_t)(st * PB + pb) * 1024u : 0u);
  };
#pragma unroll
  for (int x = 0; x < TM; ++x)
#pragma unroll
    for (int y = 0; y < TN; ++y) c0[x][y] = c1[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int d = 0; d < NSTG - 1; ++d) issue_a(d);
#pragma unroll
  for (int d = 0; d < D - 1; ++d) load_w(d, wr[d]);
  for (int st0 = 0; st0 < kb; st0 += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const int st = st0 + d;
      // this wave's loads complete in issue order: A(st) has landed when at most the NSTG - 2 younger stages' A
      // loads are outstanding (weights of younger stages are in the count too, so it waits for more than A(st)). The
      // barrier makes the whole stage visible and frees the buffer multiplied at st - 1; it is the bare
      // instruction, because __syncthreads' fences would also wait for the stages in flight.
      __builtin_amdgcn_s_waitcnt(waitcnt_stage((NSTG - 2) * C::LPA));
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      load_w(st + D - 1, wr[(d + D - 1) % D]);
      issue_a(st + NSTG - 1);
      const char* base = smem + (st % NSTG) * C::STG + lane * 16;
#pragma unroll
      for (int x = 0; x < TM; ++x) {
        const f16x8 ah = *(const f16x8*)(base + x * PA * 1024);
#pragma unroll
        for (int y = 0; y < TN; ++y) c0[x][y] = mfma_f16(wr[d][y][0], ah, c0[x][y]);
        if constexpr (PA == 2) {
          const f16x8 al = *(const f16x8*)(base + x * PA * 1024 + 1024);
#pragma unroll
          for (int y = 0; y < TN; ++y) c1[x][y] = mfma_f16(wr[d][y][0], al, c1[x][y]);
        }
        if constexpr (PB == 2) {
#pragma unroll
          for (int y = 0; y < TN; ++y) c1[x][y] = mfma_f16(wr[d][y][PB - 1], ah, c1[x][y]);
        }
      }
    }
  }
  __builtin_amdgcn_s_waitcnt(waitcnt_stage(0));
  __syncthreads();
}

}  // namespace onmt
