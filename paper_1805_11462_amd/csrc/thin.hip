// GEMMs of few rows for gfx950 (decoder layers, encoder recurrence, attentional output): out[r, n] =
// sum_k A[r, k] W[n, k] over at most a few hundred gathered rows, with the LSTM cell (Section 2 item (a) of the
// OpenNMT paper) or a plain store as epilogue.
//
// A step's weights are a few MB and its products take 1-6 us of MFMA time, so what bounds these launches is how
// many bytes of operands a CU keeps in flight and the fixed cost of a launch. The main loop has no LDS and no
// barrier: the workgroup's NW waves split K, each wave loads its own 32-column K blocks of the tile's A and W rows
// straight into registers, D blocks ahead, and nothing is loaded twice inside a workgroup. Operands are two-term
// fp16 splits in fragment blocks (split16.h): every load is 1 KB of consecutive addresses (A rows that come
// through a beam parent map: 16-byte chunks of a few neighbouring rows). The waves' partial tiles meet once, in
// LDS, before the epilogue.

#include "common.h"
#include "gemm_device.h"
#include "kernels.h"
#include "split16.h"
#include "wide_loop.h"

namespace onmt {

// PB: weight terms; the tile is 16 TM x 16 TN, NW waves split K, D K blocks in flight per wave.
template <int PB_, int TM_, int TN_, int NW_, int D_>
struct Thin {
  static constexpr int PB = PB_, TM = TM_, TN = TN_, NW = NW_, D = D_;
  static constexpr int BM = 16 * TM, BN = 16 * TN, NT = 64 * NW;
  static constexpr int CROW = BN + 4;
  static constexpr int PART = BM * CROW;        // floats of one wave's partial tile
  static constexpr int LDS = NW * PART * 4;
};

// Main loop: leaves NW partial tiles in LDS at red ([NW][BM][CROW] floats), no barrier after the stores.
template <class C, int NSEG>
__device__ __forceinline__ void thin_main(const ThinA& a, const ThinW& w, int m0, int n0, float* red) {
  static_assert(NSEG == 1 || NSEG == 2, "one or two A segments");
  constexpr int TM = C::TM, TN = C::TN, PB = C::PB, D = C::D;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i16 = lane & 15, g = lane >> 4;
  // byte offsets of the lane's A rows in each segment (rows past M read row M - 1; never stored)
  uint32_t ro[NSEG][TM];
#pragma unroll
  for (int s = 0; s < NSEG; ++s)
#pragma unroll
    for (int x = 0; x < TM; ++x) {
      const int m = min(m0 + 16 * x + i16, a.M - 1);
      const uint32_t r = a.seg[s].row0 + (a.seg[s].idx ? a.seg[s].idx[m] : m);
      ro[s][x] = (r / kFragRows) * a.seg[s].kblocks * 2048u + g * 256u + (r % kFragRows) * 16u;
    }
  const __amdgpu_buffer_rsrc_t rw = make_rsrc(w.base, (uint32_t)(w.rows / 16) * w.kblocks * (PB * 1024u));
  uint32_t wo[TN];
#pragma unroll
  for (int y = 0; y < TN; ++y) wo[y] = ((uint32_t)(n0 / 16 + y) * w.kblocks + w.kb0) * (PB * 1024u) + lane * 16u;
  const int kb0 = a.seg[0].kblocks, ktot = kb0 + (NSEG > 1 ? a.seg[NSEG - 1].kblocks : 0);

  struct Frag {
    uint4 a[TM][2];
    uint4 w[TN][PB];
  };
  // K block st of the segments one after the other; past the last, the offsets lie beyond the buffers (zeros)
  auto load = [&](int st, Frag& f) {
    const bool on = st < ktot, s1 = NSEG > 1 && st >= kb0;
    const __amdgpu_buffer_rsrc_t ra = make_rsrc(s1 ? a.seg[NSEG - 1].base : a.seg[0].base,
                                                s1 ? a.seg[NSEG - 1].bytes : a.seg[0].bytes);
    const uint32_t ks = on ? (uint32_t)(s1 ? st - kb0 : st) * 2048u : 0u;
#pragma unroll
    for (int x = 0; x < TM; ++x) {
      const uint32_t off = on ? (s1 ? ro[NSEG - 1][x] : ro[0][x]) : kPastEnd;
      f.a[x][0] = buf_load16s(ra, off, ks);
      f.a[x][1] = buf_load16s(ra, on ? off + 1024u : kPastEnd, ks);
    }
#pragma unroll
    for (int y = 0; y < TN; ++y)
#pragma unroll
      for (int pb = 0; pb < PB; ++pb)
        f.w[y][pb] = buf_load16s(rw, on ? wo[y] : kPastEnd, on ? (uint32_t)(st * PB + pb) * 1024u : 0u);
  };

  f32x4 c0[TM][TN], c1[TM][TN];
#pragma unroll
  for (int x = 0; x < TM; ++x)
#pragma unroll
    for (int y = 0; y < TN; ++y) c0[x][y] = c1[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
  // the weights are the MFMA's row operand, so a lane ends up with four consecutive columns of one row
  auto compute = [&](const Frag& f) {
#pragma unroll
    for (int x = 0; x < TM; ++x) {
#pragma unroll
      for (int y = 0; y < TN; ++y) c0[x][y] = mfma_f16(f.w[y][0], f.a[x][0], c0[x][y]);
#pragma unroll
      for (int y = 0; y < TN; ++y) c1[x][y] = mfma_f16(f.w[y][0], f.a[x][1], c1[x][y]);
      if constexpr (PB == 2) {
#pragma unroll
        for (int y = 0; y < TN; ++y) c1[x][y] = mfma_f16(f.w[y][PB - 1], f.a[x][0], c1[x][y]);
      }
    }
  };
  Frag f[D];
#pragma unroll
  for (int d = 0; d < D; ++d) load(wave + C::NW * d, f[d]);
  for (int st = wave; st < ktot; st += C::NW * D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      compute(f[d]);
      load(st + C::NW * (d + D), f[d]);
    }
  }
  float* Ct = red + wave * C::PART;
#pragma unroll
  for (int x = 0; x < TM; ++x)
#pragma unroll
    for (int y = 0; y < TN; ++y) {
      f32x4 v;
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = fmaf(c1[x][y][j], 1.f / kLoScale, c0[x][y][j]);
      *(f32x4*)(Ct + (16 * x + i16) * C::CROW + 16 * y + 4 * g) = v;
    }
}

template <class C>
__device__ inline float thin_sum(const float* red, int r, int c) {
  float s = red[r * C::CROW + c];
#pragma unroll
  for (int w = 1; w < C::NW; ++w) s += red[w * C::PART + r * C::CROW + c];
  return s;
}

// What the LSTM epilogue adds to this thread's (row, unit) elements: bias, the precomputed input projection
// (table rows gathered by token id) and the previous cell state, with the columns' scales, all loaded before the
// main loop. SHIFT: rows of an external step's own state, whose operands carry powers of two of their own (a variant,
// because the null checks alone cost the recurrences 3%).
template <class C, bool SHIFT>
struct ThinLstm {
  static constexpr int UPT = C::BN / 4;                          // units per tile
  static constexpr int EPT = (C::BM * UPT + C::NT - 1) / C::NT;  // elements per thread
  float z[EPT][4], c[EPT];
  int ex[EPT][4], is[EPT], os[EPT];

  __device__ __forceinline__ void load(const LstmParams& p, const int32_t* wexp, int M, int m0, int n0) {
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
      const int e = threadIdx.x + i * C::NT;
      const int r = e / UPT, uu = e % UPT;
      const int row = m0 + r, unit = n0 / 4 + uu;
      const bool ok = e < C::BM * UPT && row < M && unit < p.H;
      const int cbase = (uu / kUnitGroup) * (4 * kUnitGroup) + (uu % kUnitGroup);
      const int grow = !(ok && p.gx) ? 0 : (p.gx_idx ? min((unsigned)p.gx_idx[row], (unsigned)p.gx_rows - 1u) : row * p.gx_S + p.gx_s);
      const int crow = ok && p.c_idx ? p.c_idx[row] : row;
      c[i] = ok && p.c_in ? p.c_in[(size_t)crow * p.ld_c + unit] : 0.f;
      if constexpr (SHIFT) {
        is[i] = ok ? p.in_shift[crow] : 0;
        os[i] = ok && p.out_shift ? p.out_shift[crow] : 0;
      }
#pragma unroll
      for (int gt = 0; gt < 4; ++gt) {
        const int col = n0 + cbase + gt * kUnitGroup;
        ex[i][gt] = ok ? wexp[col] : 0;
        z[i][gt] = (ok && p.bias ? p.bias[col] : 0.f) +
                   (ok && p.gx ? p.gx[(size_t)grow * p.ld_gx + p.gx_col0 + col] : 0.f);
      }
    }
  }

  // Gate nonlinearities and cell update over the tile whose partial sums are in LDS. The rows past M of the last
  // 16-row block and the units past H of the last 32-column block of the two-term copies are zeros.
  __device__ __forceinline__ void finish(const float* red, const LstmParams& p, int M, int m0, int n0) const {
#pragma unroll
    for (int i = 0; i < EPT; ++i) {
      const int e = threadIdx.x + i * C::NT;
      const int r = e / UPT, uu = e % UPT;
      const int row = m0 + r, unit = n0 / 4 + uu;
      if (e >= C::BM * UPT) continue;
      float h_new = 0.f, y = 0.f;
      const bool on = row < M && unit < p.H;
      if (on) {
        const int cbase = (uu / kUnitGroup) * (4 * kUnitGroup) + (uu % kUnitGroup);
        float zz[4], c_new;
#pragma unroll
        for (int gt = 0; gt < 4; ++gt)
          zz[gt] = ldexpf(thin_sum<C>(red, r, cbase + gt * kUnitGroup), ex[i][gt] - (SHIFT ? is[i] : 0)) + z[i][gt];
        if (p.lens && p.y_s >= p.lens[row]) {
          c_new = c[i];
          h_new = p.h_in ? p.h_in[(size_t)row * p.ld_h_in + unit] : 0.f;
        } else {
          const float ig = sigmoidf_(zz[0]), fg = sigmoidf_(zz[1]), gg = tanhf(zz[2]), og = sigmoidf_(zz[3]);
          c_new = fg * c[i] + ig * gg;
          h_new = og * tanhf(c_new);
          y = h_new;
        }
        p.h_out[(size_t)row * p.ld_out + unit] = h_new;
        p.c_out[(size_t)row * p.ld_out + unit] = c_new;
        if (p.y_out) p.y_out[(size_t)(row * p.y_S + p.y_s) * p.ld_y + p.y_col0 + unit] = y;
      }
      if (p.h16 && row < (M + kFragRows - 1) / kFragRows * kFragRows && unit < p.kb16 * kFragK) {
        uint16_t hi, lo;
        split_act(SHIFT ? ldexpf(h_new, os[i]) : h_new, hi, lo);
        uint16_t* d = p.h16 + split16_at(row, unit, p.kb16, 2);
        d[0] = hi;
        d[kFragElems] = lo;
      }
      if (p.y16 && on) {
        uint16_t hi, lo;
        split_act(y, hi, lo);
        uint16_t* d = p.y16 + split16_at((size_t)p.y_r0 + row, p.y_col0 + unit, p.y_kb16, 2);
        d[0] = hi;
        d[kFragElems] = lo;
      }
    }
  }
};

template <class C, int NSEG, bool SHIFT = false>
__device__ __forceinline__ void thin_lstm_tile(const ThinA& a, const ThinW& w, const LstmParams& p, int nm, int nblocks,
                                               int bid, float* red) {
  const int L = xcd_remap(bid, nblocks);
  const int m0 = (L % nm) * C::BM, n0 = (L / nm) * C::BN;
  ThinLstm<C, SHIFT> ep;
  ep.load(p, w.wexp, a.M, m0, n0);
  thin_main<C, NSEG>(a, w, m0, n0, red);
  __syncthreads();
  ep.finish(red, p, a.M, m0, n0);
}

template <class C, int NSEG, bool SHIFT>
__global__ __launch_bounds__(C::NT) void k_thin_lstm(ThinA a, ThinW w, LstmParams p, int nm, int nblocks) {
  __shared__ __attribute__((aligned(16))) float red[C::LDS / 4];
  thin_lstm_tile<C, NSEG, SHIFT>(a, w, p, nm, nblocks, blockIdx.x, red);
}

// LSTM products of many rows against one-term weights: 32 x 128 tiles whose rows go through LDS, shared by the four
// waves (wide_loop.h), and whose weights go straight into registers. Both kinds are bound by what a CU can read from
// L2; per row of A this one reads half of what the K-splitting 32 x 128 tile does: 512 x 2048 x 4096 28.1 us against
// 30.9, 512 x 1024 x 4096 17.4 against 20.0, 640 rows 36 against 42; at 320 rows 25.4 against 22.5 (32 x 64).
struct ThinWide : WideTile<2, 2, 2, 1, 6, 4> {
  static constexpr int NW = 1, CROW = BN + 4, PART = BM * CROW;
  static constexpr int BYTES = LDS > PART * 4 ? LDS : PART * 4;
};

template <int NSEG, bool SHIFT>
__global__ __launch_bounds__(ThinWide::NT) void k_thin_lstm_wide(ThinA a, ThinW w, LstmParams p, int nm, int nblocks) {
  using C = ThinWide;
  constexpr int TM = C::TM, TN = C::TN, S1 = NSEG - 1;
  __shared__ __attribute__((aligned(16))) char smem[C::BYTES];
  const int L = xcd_remap(blockIdx.x, nblocks);
  const int m0 = (L % nm) * C::BM, n0 = (L / nm) * C::BN;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i16 = lane & 15, g = lane >> 4;
  ThinLstm<C, SHIFT> ep;
  ep.load(p, w.wexp, a.M, m0, n0);
  uint32_t aoff[NSEG][C::LPA], woff[TN];
#pragma unroll
  for (int s = 0; s < NSEG; ++s)
#pragma unroll
    for (int i = 0; i < C::LPA; ++i) {
      const int q = wide_block<C>(wave, i), m = min(m0 + q / 2 * 16 + i16, a.M - 1);
      const uint32_t r = a.seg[s].row0 + (a.seg[s].idx ? a.seg[s].idx[m] : m);
      aoff[s][i] = (r / kFragRows) * a.seg[s].kblocks * 2048u + (q & 1) * 1024u + g * 256u + (r % kFragRows) * 16u;
    }
#pragma unroll
  for (int y = 0; y < TN; ++y) woff[y] = ((uint32_t)(n0 / 16 + wave * TN + y) * w.kblocks + w.kb0) * 1024u + lane * 16u;
  const int kb0 = a.seg[0].kblocks;
  auto load_a = [&](int st, char* base) {
    const bool s1 = NSEG > 1 && st >= kb0;
    const __amdgpu_buffer_rsrc_t ra =
        make_rsrc(s1 ? a.seg[S1].base : a.seg[0].base, s1 ? a.seg[S1].bytes : a.seg[0].bytes);
#pragma unroll
    for (int i = 0; i < C::LPA; ++i)
      dma16(ra, base + wide_block<C>(wave, i) * 1024, s1 ? aoff[S1][i] : aoff[0][i],
            (uint32_t)(s1 ? st - kb0 : st) * 2048u);
  };
  f32x4 c0[TM][TN], c1[TM][TN];
  wide_main<C>(smem, load_a, make_rsrc(w.base, (uint32_t)(w.rows / 16) * w.kblocks * 1024u), woff,
               kb0 + (NSEG > 1 ? a.seg[S1].kblocks : 0), c0, c1);
  float* red = (float*)smem;
#pragma unroll
  for (int x = 0; x < TM; ++x)
#pragma unroll
    for (int y = 0; y < TN; ++y) {
      f32x4 v;
#pragma unroll
      for (int j = 0; j < 4; ++j) v[j] = fmaf(c1[x][y][j], 1.f / kLoScale, c0[x][y][j]);
      *(f32x4*)(red + (16 * x + i16) * C::CROW + wave * 16 * TN + 16 * y + 4 * g) = v;
    }
  __syncthreads();
  ep.finish(red, p, a.M, m0, n0);
}

// Two independent LSTM products in one launch (the encoder's two directions at one step, or two stacked layers at
// consecutive timesteps): blocks [0, nb[0]) run problem 0, the next nt[1] blocks problem 1. nb[0] is a multiple of
// 8, so both problems see the same block-to-XCD dealing.
template <class C, int NS0, int NS1>
__global__ __launch_bounds__(C::NT) void k_thin_lstm2(ThinPair q) {
  __shared__ __attribute__((aligned(16))) float red[C::LDS / 4];
  const int bid = blockIdx.x;
  if (bid < q.nb0) {
    if (bid < q.nt[0]) thin_lstm_tile<C, NS0>(q.a[0], q.w[0], q.p[0], q.nm[0], q.nt[0], bid, red);
  } else {
    thin_lstm_tile<C, NS1>(q.a[1], q.w[1], q.p[1], q.nm[1], q.nt[1], bid - q.nb0, red);
  }
}

template <class C, int NSEG>
__global__ __launch_bounds__(C::NT) void k_thin_store(ThinA a, ThinW w, StoreParams p, int nm, int nblocks) {
  __shared__ __attribute__((aligned(16))) float red[C::LDS / 4];
  const int L = xcd_remap(blockIdx.x, nblocks);
  const int m0 = (L % nm) * C::BM, n0 = (L / nm) * C::BN;
  thin_main<C, NSEG>(a, w, m0, n0, red);
  __syncthreads();
  const int pad_rows = (p.r0_16 + a.M + kFragRows - 1) / kFragRows * kFragRows - p.r0_16;
  for (int e = threadIdx.x; e < C::BM * (C::BN / 4); e += C::NT) {
    const int r = e / (C::BN / 4), c = e % (C::BN / 4) * 4;
    const int row = m0 + r, col = n0 + c;
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    if (row < a.M && col < p.ncols) {            // ncols is a multiple of 4
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        v[j] = ldexpf(thin_sum<C>(red, r, c + j), w.wexp[col + j]) + (p.bias ? p.bias[col + j] : 0.f);
        if (p.act == 1) v[j] = tanhf(v[j]);
      }
      *(float4*)(p.out + (size_t)row * p.ldo + col) = make_float4(v[0], v[1], v[2], v[3]);
    }
    // the two-term copy, with zeros in the rest of its last 16-row and 32-column blocks
    if (p.s16 && row < pad_rows && col < p.kb16 * kFragK) store_act4(p.s16, p.r0_16 + row, col, p.kb16, v);
  }
}

// ---------------------------------------------------------------- launchers

// Tile by the operand bytes a CU reads per K element when `blocks` workgroups are dealt to 256 CUs: rounds x (4
// per row of the tile + 2 per column and weight term), the least of the shapes below. Measured in us, weights cold,
// LSTM layers of two segments (the 16 x 32 / 32 x 64 tiles with LDS stages before in brackets):
//   fp32 weights, 2 x 500 columns, 2000 rows: 320 rows of A 80 x 32 11.0, 32 x 32 and 48 x 32 12.3 [18.3]; 160: 48 x 32
//   7.7, 32 x 32 9.5 [13.4]; 64: 16 x 32 5.8, 32 x 32 6.4 [11.5]; 5: 16 x 32 5.7 [11.0];
//   bf16 weights, 2 x 1000, 4000 rows: 320: 80 x 64 21.3, 32 x 64 22.7 [31]; 128: 32 x 64 9.9, 32 x 32 11.7; 64: 32 x 32
//   7.8, 16 x 32 8.7; 512 (2 x 1024, 4096 rows): 32 x 128 31.6, 32 x 64 30.9, 80 x 64 39 [42].
// Eight waves and one K block in flight each beat four waves with two or more nearly everywhere (64 rows fp32 5.8
// against 6.2, two problems of 64 rows bf16 4.6 against 5.2), as two workgroups then share a CU; the 80 x 64 tile
// needs the registers of four.
struct ThinShape {
  int tm, tn;
};
constexpr ThinShape kThin2[] = {{1, 2}, {2, 2}, {3, 2}, {5, 2}};      // two weight terms
constexpr ThinShape kThin1[] = {{1, 2}, {2, 2}, {2, 4}, {5, 4}, {2, 8}};      // one
template <int N>
static int thin_shape(const ThinShape (&list)[N], int pb, int nprob, const int* M, const int* rows) {
  int best = 0;
  long cost = -1;
  for (int i = 0; i < N; ++i) {
    long blocks = 0;
    for (int q = 0; q < nprob; ++q)
      blocks += (long)((M[q] + 16 * list[i].tm - 1) / (16 * list[i].tm)) * (rows[q] / (16 * list[i].tn));
    const long c = (blocks + 255) / 256 * (list[i].tm * 64 + list[i].tn * 32 * pb);
    if (cost < 0 || c < cost) {
      cost = c;
      best = i;
    }
  }
  return best;
}

static bool thin_ok(const ThinA& a, const ThinW& w, int pb) {
  if ((pb != 1 && pb != 2) || a.M < 1 || a.nseg < 1 || a.nseg > 2 || w.rows % 128 || w.rows < 1) return false;
  int k = w.kb0;
  for (int s = 0; s < a.nseg; ++s) k += a.seg[s].kblocks;
  return w.kb0 >= 0 && k <= w.kblocks && split16_bytes(w.rows, w.kblocks, pb) < (1ull << 31);
}

template <class C>
static hipError_t launch_thin_lstm(const ThinA& a, const ThinW& w, const LstmParams& p, hipStream_t st) {
  const int nm = (a.M + C::BM - 1) / C::BM, nb = nm * (w.rows / C::BN);
  const dim3 grid(nb), block(C::NT);
  if (p.in_shift) hipLaunchKernelGGL((k_thin_lstm<C, 2, true>), grid, block, 0, st, a, w, p, nm, nb);
  else if (a.nseg == 1) hipLaunchKernelGGL((k_thin_lstm<C, 1, false>), grid, block, 0, st, a, w, p, nm, nb);
  else hipLaunchKernelGGL((k_thin_lstm<C, 2, false>), grid, block, 0, st, a, w, p, nm, nb);
  return hipGetLastError();
}

template <class C>
static hipError_t launch_thin_store(const ThinA& a, const ThinW& w, const StoreParams& p, hipStream_t st) {
  const int nm = (a.M + C::BM - 1) / C::BM, nb = nm * (w.rows / C::BN);
  if (a.nseg == 1) hipLaunchKernelGGL((k_thin_store<C, 1>), dim3(nb), dim3(C::NT), 0, st, a, w, p, nm, nb);
  else hipLaunchKernelGGL((k_thin_store<C, 2>), dim3(nb), dim3(C::NT), 0, st, a, w, p, nm, nb);
  return hipGetLastError();
}

template <class C>
static hipError_t launch_thin_lstm2(ThinPair q, hipStream_t st) {
  for (int i = 0; i < 2; ++i) {
    q.nm[i] = (q.a[i].M + C::BM - 1) / C::BM;
    q.nt[i] = q.nm[i] * (q.w[i].rows / C::BN);
  }
  q.nb0 = (q.nt[0] + 7) / 8 * 8;
  const dim3 grid(q.nb0 + q.nt[1]), block(C::NT);
  const int n0 = q.a[0].nseg, n1 = q.a[1].nseg;
  if (n0 == 1 && n1 == 1) hipLaunchKernelGGL((k_thin_lstm2<C, 1, 1>), grid, block, 0, st, q);
  else if (n0 == 1) hipLaunchKernelGGL((k_thin_lstm2<C, 1, 2>), grid, block, 0, st, q);
  else if (n1 == 2) hipLaunchKernelGGL((k_thin_lstm2<C, 2, 2>), grid, block, 0, st, q);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

#define ONMT_THIN_DISPATCH(PB, I, CALL)                                  \
  do {                                                                   \
    if ((PB) == 2) {                                                     \
      if ((I) == 0) return CALL(Thin<2, 1, 2, 8, 1>);                    \
      if ((I) == 1) return CALL(Thin<2, 2, 2, 8, 1>);                    \
      if ((I) == 2) return CALL(Thin<2, 3, 2, 8, 1>);                    \
      return CALL(Thin<2, 5, 2, 8, 1>);                                  \
    }                                                                    \
    if ((I) == 0) return CALL(Thin<1, 1, 2, 8, 1>);                      \
    if ((I) == 1) return CALL(Thin<1, 2, 2, 8, 1>);                      \
    if ((I) == 2) return CALL(Thin<1, 2, 4, 8, 1>);                      \
    if ((I) == 3) return CALL(Thin<1, 5, 4, 4, 2>);                      \
    return CALL(Thin<1, 2, 8, 8, 1>);                                    \
  } while (0)

hipError_t thin_lstm(int w_terms, const ThinA& a, const ThinW& w, const LstmParams& p, hipStream_t st) {
  if (!thin_ok(a, w, w_terms) || (p.in_shift && a.nseg != 2)) return hipErrorInvalidValue;
  // one-term weights with two or more 32 x 128 tiles for every CU (k_thin_lstm_wide's comment has both sides)
  const int nm = (a.M + ThinWide::BM - 1) / ThinWide::BM, nb = nm * (w.rows / ThinWide::BN);
  if (w_terms == 1 && nb >= 512) {
    const dim3 grid(nb), block(ThinWide::NT);
    if (p.in_shift) hipLaunchKernelGGL((k_thin_lstm_wide<2, true>), grid, block, 0, st, a, w, p, nm, nb);
    else if (a.nseg == 1) hipLaunchKernelGGL((k_thin_lstm_wide<1, false>), grid, block, 0, st, a, w, p, nm, nb);
    else hipLaunchKernelGGL((k_thin_lstm_wide<2, false>), grid, block, 0, st, a, w, p, nm, nb);
    return hipGetLastError();
  }
  const int i = w_terms == 2 ? thin_shape(kThin2, 2, 1, &a.M, &w.rows) : thin_shape(kThin1, 1, 1, &a.M, &w.rows);
#define ONMT_CALL(...) launch_thin_lstm<__VA_ARGS__>(a, w, p, st)
  ONMT_THIN_DISPATCH(w_terms, i, ONMT_CALL);
#undef ONMT_CALL
}

hipError_t thin_lstm2(int w_terms, const ThinPair& q, hipStream_t st) {
  for (int i = 0; i < 2; ++i)
    if (!thin_ok(q.a[i], q.w[i], w_terms) || q.p[i].in_shift) return hipErrorInvalidValue;
  const int M[2] = {q.a[0].M, q.a[1].M}, rows[2] = {q.w[0].rows, q.w[1].rows};
  const int i = w_terms == 2 ? thin_shape(kThin2, 2, 2, M, rows) : thin_shape(kThin1, 1, 2, M, rows);
#define ONMT_CALL(...) launch_thin_lstm2<__VA_ARGS__>(q, st)
  ONMT_THIN_DISPATCH(w_terms, i, ONMT_CALL);
#undef ONMT_CALL
}

hipError_t thin_store(int w_terms, const ThinA& a, const ThinW& w, const StoreParams& p, hipStream_t st) {
  if (!thin_ok(a, w, w_terms) || p.ncols % 4 || p.ncols > w.rows || (p.s16 && p.kb16 * kFragK > w.rows)) return hipErrorInvalidValue;
  const int i = w_terms == 2 ? thin_shape(kThin2, 2, 1, &a.M, &w.rows) : thin_shape(kThin1, 1, 1, &a.M, &w.rows);
#define ONMT_CALL(...) launch_thin_store<__VA_ARGS__>(a, w, p, st)
  ONMT_THIN_DISPATCH(w_terms, i, ONMT_CALL);
#undef ONMT_CALL
}

// ---------------------------------------------------------------- decoder state

// Eight consecutive columns (k0 a multiple of 8) of row r of a two-term operand, scaled by 2^e.
__device__ inline void store_act8(uint16_t* dst, int r, int k0, int kblocks, const float (&v)[8], int e = kActExp) {
  uint32_t h[4], l[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    uint16_t h0, h1, l0, l1;
    split_scaled(ldexpf(v[2 * j], e), h0, l0);
    split_scaled(ldexpf(v[2 * j + 1], e), h1, l1);
    h[j] = h0 | (uint32_t)h1 << 16;
    l[j] = l0 | (uint32_t)l1 << 16;
  }
  uint16_t* d = dst + split16_at(r, k0, kblocks, 2);
  *(uint4*)d = make_uint4(h[0], h[1], h[2], h[3]);
  *(uint4*)(d + kFragElems) = make_uint4(l[0], l[1], l[2], l[3]);
}

// Thread = eight columns of one row of one of L + 1 row sets (the layers' h, then feed), rows up to the end of the
// last 16-row block and columns up to the end of the last 32-column block (zeros there). Reads 4 columns at a
// time (H is a multiple of 4).
__device__ inline void row_chunk(const float* src, int H, int k0, bool on, float (&v)[8]) {
#pragma unroll
  for (int j = 0; j < 8; j += 4) {
    const float4 q = on && k0 + j < H ? *(const float4*)(src + k0 + j) : make_float4(0.f, 0.f, 0.f, 0.f);
    v[j] = q.x, v[j + 1] = q.y, v[j + 2] = q.z, v[j + 3] = q.w;
  }
}

__global__ __launch_bounds__(256) void k_decode_init(DecodeState s, const float* __restrict__ final_h,
                                                     const float* __restrict__ final_c, int B, int K) {
  const int chunks = s.kb * 4, rows = (s.N + kFragRows - 1) / kFragRows * kFragRows;
  const size_t n = (size_t)(s.L + 1) * rows * chunks;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
    const int k0 = (int)(i % chunks) * 8, r = (int)(i / chunks % rows), l = (int)(i / chunks / rows);
    const bool on = r < s.N;
    float h[8], c[8];
    if (l < s.L) {
      const size_t src = ((size_t)l * B + r / K) * s.H;
      row_chunk(final_h + src, s.H, k0, on, h);
      row_chunk(final_c + src, s.H, k0, on, c);
      store_act8(s.h16 + l * s.plane, r, k0, s.kb, h);
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) h[j] = 0.f;
      store_act8(s.feed16, r, k0, s.kb, h);
    }
    if (!on) continue;
    const size_t o = ((size_t)(l < s.L ? l : 0) * s.N + r) * s.H + k0;
#pragma unroll
    for (int j = 0; j < 8; j += 4) {
      if (k0 + j >= s.H) break;
      *(float4*)((l < s.L ? s.h : s.feed) + o + j) = make_float4(h[j], h[j + 1], h[j + 2], h[j + 3]);
      if (l < s.L) *(float4*)(s.c + o + j) = make_float4(c[j], c[j + 1], c[j + 2], c[j + 3]);
    }
  }
}

hipError_t decode_init(const DecodeState& s, const float* final_h, const float* final_c, int B, int K, hipStream_t st) {
  const size_t n = (size_t)(s.L + 1) * ((s.N + kFragRows - 1) / kFragRows * kFragRows) * s.kb * 4;
  size_t blocks = (n + 255) / 256;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(k_decode_init, dim3((unsigned)blocks), dim3(256), 0, st, s, final_h, final_c, B, K);
  return hipGetLastError();
}

// The id checks (tok given) and the two-term copies of a caller's state (split; s.h16 and s.feed16 lie in the step's
// output state), one launch. A caller's rows may be of any size, so each row of a layer's product gets a power of two
// of its own: one wave reads what that product reads of the row (layer 0: feed and h, else h), scales its largest
// value to [2^14, 2^15) and records the power. In layers above 0 the same power also scales the output of the
// layer below, which is at most 1 in size, so there it is at most 2^14.
constexpr int kMaxChunks = 2;                 // 8-column chunks per lane (H <= 1024)

// Blocks [0, id_blocks) check the ids, the others copy, so that the two chains of loads run side by side.
__global__ __launch_bounds__(256) void k_prepare_step(DecodeState s, int id_blocks, const int32_t* __restrict__ tok,
                                                      const int32_t* __restrict__ parent, int V,
                                                      int32_t* __restrict__ tok_out, int32_t* __restrict__ par_out,
                                                      int32_t* err) {
  if ((int)blockIdx.x < id_blocks) {
    for (size_t r = (size_t)blockIdx.x * blockDim.x + threadIdx.x; r < (size_t)s.N; r += (size_t)id_blocks * blockDim.x) {
      int t = tok[r];
      if (t < 0 || t >= V) {
        *err = kErrToken;
        t = 0;
      }
      tok_out[r] = t;
      if (parent) {
        int p = parent[r];
        if (p < 0 || p >= s.N) {
          *err = kErrParent;
          p = (int)r;
        }
        par_out[r] = p;
      }
    }
    return;
  }
  const int block = blockIdx.x - id_blocks, blocks = gridDim.x - id_blocks;
  const size_t nshift = (size_t)s.L * s.N;
  if (block == 0 && threadIdx.x < (kShiftPad - nshift % kShiftPad) % kShiftPad) s.shift[nshift + threadIdx.x] = 0;
  const int lane = threadIdx.x & 63;
  const unsigned chunks = s.kb * 4, rows = (s.N + kFragRows - 1) / kFragRows * kFragRows;
  for (unsigned i = block * (256 / kWave) + threadIdx.x / kWave; i < s.L * rows; i += blocks * (256 / kWave)) {
    const int r = i % rows, l = i / rows;            // L <= 64, N < 2^22 (state operands below 2 GiB)
    const bool on = r < s.N;
    float h[kMaxChunks][8], f[kMaxChunks][8], m = 0.f;
#pragma unroll
    for (int j = 0; j < kMaxChunks; ++j) {
      const int k0 = (lane + j * kWave) * 8;
      row_chunk(s.h + ((size_t)l * s.N + r) * s.H, s.H, k0, on, h[j]);
      row_chunk(s.feed + (size_t)r * s.H, s.H, k0, on && l == 0, f[j]);
#pragma unroll
      for (int v = 0; v < 8; ++v) {
        h[j][v] = finite_or_nan(h[j][v]);
        f[j][v] = finite_or_nan(f[j][v]);
        m = fmaxf(m, fmaxf(fabsf(h[j][v]), fabsf(f[j][v])));      // a NaN is passed over
      }
    }
    m = wave_max(m);
    // m < 2^(biased exponent - 126), also for zero and subnormal values with 1 in the place of their exponent
    int e = 15 - (max((int)(__builtin_bit_cast(uint32_t, m) >> 23), 1) - 126);
    if (l > 0) e = min(e, 14);
    if (on && lane == 0) s.shift[(size_t)l * s.N + r] = e - kActExp;
#pragma unroll
    for (int j = 0; j < kMaxChunks; ++j) {
      const int k0 = (lane + j * kWave) * 8;
      if (k0 >= (int)chunks * 8) continue;
      store_act8(s.h16 + l * s.plane, r, k0, s.kb, h[j], e);
      if (l == 0) store_act8(s.feed16, r, k0, s.kb, f[j], e);
    }
  }
}

hipError_t prepare_step(const DecodeState& s, int split, const int32_t* tok, const int32_t* parent, int V,
                        int32_t* tok_out, int32_t* par_out, int32_t* err, hipStream_t st) {
  if (split && (!s.shift || s.kb * 4 > kMaxChunks * kWave)) return hipErrorInvalidValue;
  auto blocks = [](size_t threads) { return (int)((threads + 255) / 256 < 4096 ? (threads + 255) / 256 : 4096); };
  const int id_blocks = tok ? blocks(s.N) : 0;
  const size_t rows = (size_t)(s.N + kFragRows - 1) / kFragRows * kFragRows;
  const int copy_blocks = split ? blocks((size_t)s.L * rows * kWave) : 0;
  if (id_blocks + copy_blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(k_prepare_step, dim3(id_blocks + copy_blocks), dim3(256), 0, st, s, id_blocks, tok, parent, V,
                     tok_out, par_out, err);
  return hipGetLastError();
}

}  // namespace onmt
