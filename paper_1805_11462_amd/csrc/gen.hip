// The vocabulary projection (generator) for gfx950: logits = A W^T + b over the whole target vocabulary, with
// the log-softmax partials (per row and 128-column tile: largest logit, sum of exponentials) in the epilogue.
//
// Operands are two-term fp16 splits in fragment blocks (see split16.h): A the attentional vector, W the
// weights (fp32 models: both terms; bf16 models: one, exact down to 2^-31 of its row's largest). Products hi.hi go to one
// fp32 accumulator, hi.lo and lo.hi to a second that is scaled down when the two are added, so three
// v_mfma_f32_16x16x32_f16 per fp32 product (two for bf16 weights). The dropped lo.lo product lies below 2^-22
// of the leading one; against 64 bits the sums are closer than fp32 MFMA's, because an accumulator is rounded
// once per 32 products (relative error of a 512-wide product, uniform operands: 1.6e-7; fp32 MFMA 4.1e-7, six
// bf16 term products 3.5e-7).
//
// The weights take part as the MFMA's row operand, so a lane holds four consecutive vocabulary columns of one
// row: the epilogue works on the accumulators in registers, and the logits it stores for the beam step's
// exact top-K are 16-byte stores. No list of candidates is built here: the beam step reads the logits of the
// few tiles whose maximum reaches the row's K-th largest tile maximum. (K rounds of a masked argmax per tile
// cost 10 us of the 110 at 320 rows, K = 5.) The stores are nontemporal: with ordinary ones the step's other
// weights fell out of the caches (bf16 4 x 1000 model: step 274 us, 249 with them). At K = 1 the tile's best
// candidate is known here and nothing else is stored.

#include "common.h"
#include "gemm_device.h"
#include "kernels.h"
#include "split16.h"
#include "wide_loop.h"

namespace onmt {

typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));

// Few rows (up to 64): 32 TM x 128 tile, four waves of 16 TM rows x 64 columns, both operands through LDS. What
// bounds it is the weights' stream (100 MB at 50000 x 512 fp32: 18 us at 5 rows; the fp32 MFMA kernel before it
// took 42). NSTG: K stages of 32 in LDS, NSTG - 1 in flight while one is multiplied. PB: weight terms.
template <int TM_, int PB_, int NSTG_>
struct GenTile {
  static constexpr int TM = TM_, PB = PB_, NSTG = NSTG_, TN = 4, WN = 2;
  static constexpr int BM = 32 * TM, BN = 128, NT = 256;
  static constexpr int LPW = TM + 2 * PB;                     // 1 KB loads per wave and stage
  static constexpr int ASTG = 2 * TM * 2 * 1024;              // bytes of a stage's A blocks
  static constexpr int STG = ASTG + 8 * PB * 1024;
  static constexpr int CROW = BN + 4;                         // LISTS: staged output rows
  static constexpr int LDS = NSTG * STG;
};

// More rows: the wide tiles (wide_loop.h), 16 TM x 256, four waves of all 16 TM rows x 64 columns.
// 320 rows x 50000 x 512, fp32 weights: 56 us (160 x 128 tiles through LDS 64; six bf16 term products in 64 x 128
// tiles 110-126); bf16 weights, 512 x 32000 x 1024: 58 us with the weights in the caches, 72 from HBM (two
// products; with two bf16 terms 65-67 in the same step). 6400 rows, fp32 weights: 0.88 ms = 1.1 PFLOP/s of fp16
// products, 0.94 of the rate an 8192-cubed library product reaches on the same card.
template <int TM, int PB, int NSTG, int D>
struct GenWide : WideTile<TM, 4, 2, PB, NSTG, D> {
  static constexpr int WN = 4;
};

// Top-K lists of a 64 x 128 tile staged in LDS: 4 threads per row, 32 interleaved columns each, K rounds of a
// 4-lane argmax (larger logit first, smaller id on ties), each thread skipping the columns it gave away and those
// that are no candidates (hypothesis filters).
__device__ inline void gen_lists(const float* Ct, int crow, const GenParams& p, int M, int m0, int n0, int nt, int tid) {
  const int r = tid >> 2, part = tid & 3;
  const int row = m0 + r;
  const float ninf = -__builtin_inff();
  float z[32];
#pragma unroll
  for (int j = 0; j < 32; ++j) z[j] = Ct[r * crow + 4 * j + part];
  if (p.pfmax) {
    const bool unk = p.unk_cnt && row < M && p.max_unk >= 0 && p.unk_cnt[row] >= p.max_unk;
#pragma unroll
    for (int j = 0; j < 32; ++j) {
      const int c = n0 + 4 * j + part;
      if (c >= p.V) continue;
      const bool banned = p.banned_bits && ((p.banned_bits[c >> 5] >> (c & 31)) & 1u);
      if (banned || (unk && c == p.unk_id)) z[j] = ninf;
    }
  }
  const size_t o = ((size_t)row * p.ntiles + nt) * p.K;
  uint32_t taken = 0;
  for (int k = 0; k < p.K; ++k) {
    float bv = ninf;
    int bj = 0;
#pragma unroll
    for (int j = 0; j < 32; ++j) {
      if (!((taken >> j) & 1u) && z[j] > bv) {       // strict: the earlier (smaller id) column wins ties
        bv = z[j];
        bj = j;
      }
    }
    int bid = bv > ninf ? n0 + 4 * bj + part : 0x7fffffff;
    const int mine = bid;
#pragma unroll
    for (int x = 1; x <= 2; x <<= 1) {
      const float ov = __shfl_xor(bv, x, kWave);
      const int oi = __shfl_xor(bid, x, kWave);
      if (before(ov, oi, bv, bid)) {
        bv = ov;
        bid = oi;
      }
    }
    if (bid == mine && bv > ninf) taken |= 1u << bj;
    if (part == 0 && row < M) {
      p.pval[o + k] = bv;
      p.pid[o + k] = bid;
    }
  }
}

// Bias, log-softmax partials and logits of a tile from the accumulators (c0: leading products, c1: the scaled
// rest); c0 holds the logits afterwards. Wave (wm, wn): lane (i16, g) has rows 16 x + i16 of the wave's rows and
// columns 16 y + 4 g + v of its 64.
template <class C>
__device__ __forceinline__ void gen_epilogue(char* smem, const GenParams& p, int M, int Np, int m0, int n0, int wm,
                                             int wn, f32x4 (&c0)[C::TM][C::TN], const f32x4 (&c1)[C::TM][C::TN]) {
  constexpr int TM = C::TM, TN = C::TN;
  static_assert(C::WN * C::BM * 4 * 4 <= C::LDS, "epilogue LDS");
  const int tid = threadIdx.x, lane = tid & 63, i16 = lane & 15, g = lane >> 4;
  const float ninf = -__builtin_inff();
  const int nw0 = n0 + wn * 64;
  f32x4 bias[TN];
  int ex[TN][4];
  const int t0 = nw0 / 128 * 128;              // the wave's partials tile; past the packed matrix nothing is stored
#pragma unroll
  for (int y = 0; y < TN; ++y) {
    const int c = (t0 < Np ? nw0 : 0) + 16 * y + 4 * g;
    bias[y] = *(const f32x4*)(p.bias + c);
    const int4 e = *(const int4*)(p.wexp + c);
    ex[y][0] = e.x, ex[y][1] = e.y, ex[y][2] = e.z, ex[y][3] = e.w;
  }
  // bit 4 y + v: the column is not a candidate (hypothesis filters)
  uint32_t banned = 0;
  if (p.banned_bits) {
#pragma unroll
    for (int y = 0; y < TN; ++y) {
      const int c = nw0 + 16 * y + 4 * g;
      const uint32_t word = c < p.V ? p.banned_bits[c >> 5] : 0u;
      banned |= ((word >> (c & 31)) & 15u) << (4 * y);
    }
  }
  const bool whole = t0 + 128 <= p.V;          // uniform: every column is a vocabulary entry
  float* red = (float*)smem;                   // [wn][BM][max, sum, allowed max, its column]
  float rmx[TM], rsm[TM], rfx[TM];
  int rid[TM];
#pragma unroll
  for (int x = 0; x < TM; ++x) {
    const int row = m0 + wm * 16 * TM + 16 * x + i16;
    float z[TN][4];
    float mx = ninf;
#pragma unroll
    for (int y = 0; y < TN; ++y)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        float q = ldexpf(fmaf(c1[x][y][v], 1.f / kLoScale, c0[x][y][v]), ex[y][v]) + bias[y][v];
        if (!whole && nw0 + 16 * y + 4 * g + v >= p.V) q = ninf;
        z[y][v] = q;
        c0[x][y][v] = q;
        mx = fmaxf(mx, q);
      }
    const bool on = row < M;
    if (p.want && on) {
      const int wc = p.want[row] - nw0 - 4 * g;        // columns 16 y + v of this lane
#pragma unroll
      for (int y = 0; y < TN; ++y)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (wc == 16 * y + v) p.want_logit[row] = z[y][v];
    }
    if (p.logits && on) {
      float* lr = p.logits + (size_t)row * p.ld_logits + nw0 + 4 * g;
      if (whole) {
#pragma unroll
        for (int y = 0; y < TN; ++y)
          __builtin_nontemporal_store(f32x4{z[y][0], z[y][1], z[y][2], z[y][3]}, (f32x4_a4*)(lr + 16 * y));
      } else {
#pragma unroll
        for (int y = 0; y < TN; ++y)
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if (nw0 + 16 * y + 4 * g + v < p.V) lr[16 * y + v] = z[y][v];
      }
    }
    mx = fmaxf(mx, __shfl_xor(mx, 16, kWave));
    mx = fmaxf(mx, __shfl_xor(mx, 32, kWave));
    float sm = 0.f;
#pragma unroll
    for (int y = 0; y < TN; ++y)
#pragma unroll
      for (int v = 0; v < 4; ++v) sm += mx > ninf ? __expf(z[y][v] - mx) : 0.f;   // exp(-inf) = 0 past V
    sm += __shfl_xor(sm, 16, kWave);
    sm += __shfl_xor(sm, 32, kWave);
    float fx = ninf;
    int fid = 0x7fffffff;
    if (p.pfmax || (p.pval && p.K == 1)) {      // the best candidate, smaller column on ties
      uint32_t out = banned;
      if (p.unk_cnt && on && p.max_unk >= 0 && p.unk_cnt[row] >= p.max_unk) {
        const int wc = p.unk_id - nw0 - 4 * g;
        if (wc >= 0 && wc < 64 && (wc & 15) < 4) out |= 1u << (4 * (wc >> 4) + (wc & 15));
      }
#pragma unroll
      for (int y = 0; y < TN; ++y)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (z[y][v] > fx && !((out >> (4 * y + v)) & 1u)) {
            fx = z[y][v];
            fid = nw0 + 16 * y + 4 * g + v;
          }
#pragma unroll
      for (int o = 16; o <= 32; o <<= 1) {
        const float of = __shfl_xor(fx, o, kWave);
        const int oi = __shfl_xor(fid, o, kWave);
        if (before(of, oi, fx, fid)) {
          fx = of;
          fid = oi;
        }
      }
    }
    rid[x] = fid;
    rmx[x] = mx;
    rsm[x] = sm;
    rfx[x] = fx;
  }
  // the two 64-column halves of a partials tile meet in LDS
  if (g == 0) {
#pragma unroll
    for (int x = 0; x < TM; ++x) {
      float* q = red + (wn * C::BM + wm * 16 * TM + 16 * x + i16) * 4;
      q[0] = rmx[x];
      q[1] = rsm[x];
      q[2] = rfx[x];
      q[3] = __builtin_bit_cast(float, rid[x]);
    }
  }
  __syncthreads();
  for (int e = tid; e < C::WN / 2 * C::BM; e += C::NT) {
    const int r = e % C::BM, h = e / C::BM, nt = n0 / 128 + h;
    if (m0 + r >= M || nt * 128 >= Np) continue;
    const float *q0 = red + (2 * h * C::BM + r) * 4, *q1 = q0 + C::BM * 4;
    const float mx = fmaxf(q0[0], q1[0]);
    const size_t o = (size_t)(m0 + r) * p.ntiles + nt;
    p.pmax[o] = mx;
    p.psum[o] = (q0[0] > ninf ? q0[1] * __expf(q0[0] - mx) : 0.f) + (q1[0] > ninf ? q1[1] * __expf(q1[0] - mx) : 0.f);
    if (p.pfmax) p.pfmax[o] = fmaxf(q0[2], q1[2]);
    if (p.pval && p.K == 1) {
      const bool second = q1[2] > q0[2];              // the first half's columns are the smaller ones
      p.pval[o] = second ? q1[2] : q0[2];
      p.pid[o] = __builtin_bit_cast(int, second ? q1[3] : q0[3]);
    }
  }
}

// LISTS: per-tile top-K lists instead of logits (callers without room for [M, V] logits; TM = 2).
template <class C, bool LISTS>
__global__ __launch_bounds__(C::NT, 2) void k_gen(Split16 a, Split16 w, GenParams p, int nm, int nblocks) {
  constexpr int TM = C::TM, TN = C::TN, PB = C::PB, NSTG = C::NSTG;
  __shared__ __attribute__((aligned(16))) char smem[C::LDS];
  static_assert(!LISTS || (TM == 2 && C::BM * C::CROW * 4 <= C::LDS), "epilogue LDS");
  static_assert(C::LPW * (NSTG - 2) < 64, "wait count");
  const int L = xcd_remap(blockIdx.x, nblocks);
  const int mt = L % nm, nt = L / nm;
  const int m0 = mt * C::BM, n0 = nt * C::BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i16 = lane & 15, g = lane >> 4;
  const int wn = wave & 1, wm = wave >> 1;

  // load i of a stage moves 1 KB block wave + 4 i: first the A blocks (row block, then term), then W's. Row
  // blocks past the last re-read it (those rows are never stored).
  const int nrb = (a.rows + 15) / 16, kb = a.kblocks;
  const __amdgpu_buffer_rsrc_t ra = make_rsrc(a.base, (uint32_t)nrb * kb * 2048u);
  const __amdgpu_buffer_rsrc_t rw = make_rsrc(w.base, (uint32_t)(w.rows / 16) * kb * (PB * 1024u));
  uint32_t off[C::LPW];
#pragma unroll
  for (int i = 0; i < C::LPW; ++i) {
    if (i < TM) {
      const int q = wave + 4 * i;
      off[i] = (uint32_t)min(m0 / 16 + q / 2, nrb - 1) * kb * 2048u + (q & 1) * 1024u + lane * 16u;
    } else {
      const int q = wave + 4 * (i - TM);
      off[i] = (uint32_t)(n0 / 16 + q / PB) * kb * (PB * 1024u) + (q % PB) * 1024u + lane * 16u;
    }
  }
  auto issue = [&](int st) {         // stages past the last re-load it into a buffer that is never multiplied
    char* sb = smem + (st % NSTG) * C::STG + wave * 1024;
    const uint32_t ks = (uint32_t)min(st, kb - 1);
#pragma unroll
    for (int i = 0; i < C::LPW; ++i) {
      if (i < TM) dma16(ra, sb + i * 4096, off[i], ks * 2048u);
      else dma16(rw, sb + i * 4096, off[i], ks * (PB * 1024u));
    }
  };

  f32x4 c0[TM][TN], c1[TM][TN];
#pragma unroll
  for (int x = 0; x < TM; ++x)
#pragma unroll
    for (int y = 0; y < TN; ++y) c0[x][y] = c1[x][y] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int st = 0; st < NSTG - 1; ++st) issue(st);
  for (int st = 0; st < kb; ++st) {
    // this wave's loads complete in issue order: its share of stage st has landed; the barrier makes the
    // whole stage visible and frees the buffer multiplied at st - 1 (bare: __syncthreads' fences would also
    // wait for the stages in flight)
    __builtin_amdgcn_s_waitcnt(waitcnt_stage(C::LPW * (NSTG - 2)));
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    issue(st + NSTG - 1);
    const char* base = smem + (st % NSTG) * C::STG + lane * 16;
    f16x8 wv[PB][TN], ah[TM], al[TM];
#pragma unroll
    for (int y = 0; y < TN; ++y)
#pragma unroll
      for (int pb = 0; pb < PB; ++pb)
        wv[pb][y] = *(const f16x8*)(base + C::ASTG + ((wn * TN + y) * PB + pb) * 1024);
#pragma unroll
    for (int x = 0; x < TM; ++x) {
      ah[x] = *(const f16x8*)(base + (wm * TM + x) * 2048);
      al[x] = *(const f16x8*)(base + (wm * TM + x) * 2048 + 1024);
    }
#pragma unroll
    for (int x = 0; x < TM; ++x) {
#pragma unroll
      for (int y = 0; y < TN; ++y) c0[x][y] = mfma_f16(wv[0][y], ah[x], c0[x][y]);
#pragma unroll
      for (int y = 0; y < TN; ++y) c1[x][y] = mfma_f16(wv[0][y], al[x], c1[x][y]);
      if constexpr (PB == 2) {
#pragma unroll
        for (int y = 0; y < TN; ++y)
          c1[x][y] = mfma_f16(wv[PB - 1][y], ah[x], c1[x][y]);
      }
    }
  }
  // every load (including the re-loads past the end) has landed before the epilogue reuses the buffers
  __builtin_amdgcn_s_waitcnt(waitcnt_stage(0));
  __syncthreads();

  gen_epilogue<C>(smem, p, a.rows, w.rows, m0, n0, wm, wn, c0, c1);
  if constexpr (LISTS) {
    float* red = (float*)smem;
    __syncthreads();
#pragma unroll
    for (int x = 0; x < TM; ++x)
#pragma unroll
      for (int y = 0; y < TN; ++y)
        *(f32x4*)(red + (wm * 16 * TM + 16 * x + i16) * C::CROW + wn * 64 + 16 * y + 4 * g) = c0[x][y];
    __syncthreads();
    gen_lists(red, C::CROW, p, a.rows, m0, n0, nt, tid);
  }
}

template <class C>
__global__ __launch_bounds__(C::NT, 2) void k_gen_wide(Split16 a, Split16 w, GenParams p, int nm, int nblocks) {
  constexpr int TM = C::TM, TN = C::TN, PB = C::PB;
  __shared__ __attribute__((aligned(16))) char smem[C::LDS];
  const int L = xcd_remap(blockIdx.x, nblocks);
  const int mt = L % nm, nt = L / nm;
  const int m0 = mt * C::BM, n0 = nt * C::BN;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

  const int nrb = (a.rows + 15) / 16, kb = a.kblocks;
  uint32_t woff[TN];
#pragma unroll
  for (int y = 0; y < TN; ++y)
    woff[y] = (uint32_t)min(n0 / 16 + wave * TN + y, w.rows / 16 - 1) * kb * (PB * 1024u) + lane * 16u;
  f32x4 c0[TM][TN], c1[TM][TN];
  wide_main<C>(smem, WideRows<C>(a.base, m0, nrb, kb), make_rsrc(w.base, (uint32_t)(w.rows / 16) * kb * (PB * 1024u)),
               woff, kb, c0, c1);
  gen_epilogue<C>(smem, p, a.rows, w.rows, m0, n0, 0, wave, c0, c1);
}

// More than 64 rows: TM = 3, 4 or 5 (48-, 64- or 80-row tiles), the least of (rounds of workgroups at two per CU)
// x (tile rows + 16): a round lasts as long as a tile, whose time is its rows' products plus a part every tile
// pays. Measured in us, fp32 weights, 50000 x 512: 160 rows 33.5 (TM 5), 43.0 (4), 43.9 (3); 320 rows 61.3, 55.9,
// 62.1; 6400 rows 875, 923, 919; bf16 weights, 512 rows x 32000 x 1024: 76.9 (5), 65.3 (4), 72.7 (3).
static int gen_wide_tm(int M, int Np) {
  const long cols = (Np + 255) / 256, slots = 512;
  int best = 3;
  long cost = -1;
  for (int tm = 3; tm <= 5; ++tm) {
    const long blocks = (M + 16 * tm - 1) / (16 * tm) * cols;
    const long c = (blocks + slots - 1) / slots * (16 * tm + 16);
    if (cost < 0 || c < cost) {
      cost = c;
      best = tm;
    }
  }
  return best;
}

int gen_tile_cols() { return 128; }

template <class C, bool LISTS = false>
static hipError_t launch_gen(const Split16& a, const Split16& w, const GenParams& p, hipStream_t st) {
  const int nm = (a.rows + C::BM - 1) / C::BM, nb = nm * (w.rows / C::BN);
  hipLaunchKernelGGL((k_gen<C, LISTS>), dim3(nb), dim3(C::NT), 0, st, a, w, p, nm, nb);
  return hipGetLastError();
}

template <class C>
static hipError_t launch_wide(const Split16& a, const Split16& w, const GenParams& p, hipStream_t st) {
  const int nm = (a.rows + C::BM - 1) / C::BM, nb = nm * ((w.rows + C::BN - 1) / C::BN);
  hipLaunchKernelGGL(k_gen_wide<C>, dim3(nb), dim3(C::NT), 0, st, a, w, p, nm, nb);
  return hipGetLastError();
}

template <int PB>
static hipError_t gen_dispatch(const Split16& a, const Split16& w, const GenParams& p, hipStream_t st) {
  if (p.pval && p.K > 1) return launch_gen<GenTile<2, PB, 3>, true>(a, w, p, st);
  if (a.rows <= 32) return launch_gen<GenTile<1, PB, 4>>(a, w, p, st);
  if (a.rows <= 64) return launch_gen<GenTile<2, PB, PB == 1 ? 3 : 2>>(a, w, p, st);
  switch (gen_wide_tm(a.rows, w.rows)) {
    case 3: return launch_wide<GenWide<3, PB, 3, 2>>(a, w, p, st);
    case 4:     // one-term weights: four stages of them fit the registers (bf16 step at 320 rows 207 -> 204 us)
      return launch_wide<GenWide<4, PB, PB == 1 ? 5 : 3, PB == 1 ? 4 : 2>>(a, w, p, st);
    default: return launch_wide<GenWide<5, PB, 4, 2>>(a, w, p, st);
  }
}

hipError_t gemm_gen(const Split16& a, const Split16& w, int w_terms, const GenParams& p, hipStream_t st) {
  // buffer descriptors and their offsets are 32-bit byte counts
  const uint64_t lim = 1ull << 32;
  if ((w_terms != 1 && w_terms != 2) || a.rows < 1 || w.rows < 1 || w.rows % 128 || a.kblocks < 1 || a.kblocks != w.kblocks ||
      split16_bytes(a.rows, a.kblocks, 2) >= lim || split16_bytes(w.rows, w.kblocks, w_terms) >= lim ||
      (p.pval && (p.logits || p.K < 1)) || (p.pfmax && !p.logits && !p.pval))
    return hipErrorInvalidValue;
  return w_terms == 1 ? gen_dispatch<1>(a, w, p, st) : gen_dispatch<2>(a, w, p, st);
}

}  // namespace onmt
