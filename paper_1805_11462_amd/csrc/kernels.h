// Host-visible launch interface of the libonmt kernels (internal to the library).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "split16.h"

namespace onmt {

// Model-size refusals count K segments padded to multiples of this many elements.
constexpr int kSegK = 128;

// Plain store epilogue: out[r, n] = act(acc + bias[n]) for n < ncols. act: 0 none, 1 tanh. Optionally
// (s16 != nullptr) also as a two-term fp16 operand whose row r0_16 + r holds columns n < 32 kb16 (zeros past ncols).
struct StoreParams {
  const float* bias;
  float* out;
  int ldo;
  int ncols;
  int act;
  uint16_t* s16;
  int kb16, r0_16;
};

// LSTM cell epilogue over gate-blocked columns (groups of 32 = 4 gates x kUnitGroup = 8 units).
struct LstmParams {
  const float* bias;            // packed [Np]
  const float* gx;              // optional precomputed input projection (packed columns)
  int ld_gx, gx_col0, gx_S, gx_s;   // gx row for GEMM row b is b * gx_S + gx_s ...
  const int32_t* gx_idx;        // ... or gx_idx[b] when given (a table row per GEMM row), clamped to
  int gx_rows;                  // [0, gx_rows)
  const float* c_in;            // previous cell state rows, through c_idx (nullable = identity)
  const int32_t* c_idx;
  int ld_c;
  const float* h_in;            // previous hidden (identity rows), used when a row is masked
  int ld_h_in;
  float* h_out;
  float* c_out;
  int ld_out;
  float* y_out;                 // optional layer output row b * y_S + y_s, column offset y_col0
  int ld_y, y_S, y_s, y_col0;
  const int32_t* lens;          // optional: GEMM row b is active iff y_s < lens[b]
  int H;                        // real units
  uint16_t* h16;                // optional two-term copy of h_out (kb16 blocks of 32 columns)
  int kb16;
  const int32_t* in_shift;      // optional (two segments), through c_idx: operands of 2^(kActExp + in_shift) ...
  const int32_t* out_shift;     // ... and its h16 is to carry 2^(kActExp + out_shift)
  uint16_t* y16;                // optional two-term copy of the layer output, row y_r0 + b, columns as y_out
  int y_kb16, y_r0;
};

// Operands of the few-row GEMMs: A rows in up to two two-term segments (row r of segment s is row
// row0 + (idx ? idx[r] : r) of its buffer of `bytes` bytes), K one after the other; W the weights' rows in fragment
// blocks, of which K blocks kb0 .. are multiplied, with the power of two that undoes each column's scales.
struct ThinSeg {
  const void* base;
  const int32_t* idx;
  int row0;
  int kblocks;
  uint32_t bytes;
};
struct ThinA {
  ThinSeg seg[2];
  int nseg;
  int M;
};
struct ThinW {
  const void* base;
  const int32_t* wexp;
  int rows;
  int kblocks;
  int kb0;
};

// Two LSTM problems for one launch (nm/nt/nb0 are filled in by the launcher).
struct ThinPair {
  ThinA a[2];
  ThinW w[2];
  LstmParams p[2];
  int nm[2];     // row tiles
  int nt[2];     // tiles
  int nb0;       // blocks of problem 0, rounded up to a multiple of 8
};

// Generator epilogue: per (row, column tile) max and sum of exp, and the raw logits or per-tile top-K lists.
struct GenParams {
  const float* bias;            // [ceil128(V)]
  const int32_t* wexp;          // [ceil128(V)]: power of two that undoes a column's operand scales
  int V;
  int K;
  int ntiles;
  float* pmax;                  // [M, ntiles]
  float* psum;                  // [M, ntiles]
  float* pval;                  // optional [M, ntiles, K] top-K lists instead of logits: K = 1, or callers without
  int32_t* pid;                 // room for logits
  float* logits;                // optional [M, ld_logits]
  int ld_logits;
  const int32_t* want;          // optional [M]: column whose logit is copied to want_logit[row]
  float* want_logit;
  // hypothesis filters (with pfmax): columns that are no candidates: banned_bits[c >> 5] bit c & 31, and unk_id
  // on rows whose UNK count has reached max_unk (max_unk < 0: no limit). pfmax = each tile's largest allowed
  // logit; max and sum of exp still cover every column.
  const uint32_t* banned_bits;
  const int32_t* unk_cnt;       // [M]
  int unk_id, max_unk;
  float* pfmax;                 // [M, ntiles]
};

// w_terms: fp16 terms per weight (1 or 2).
hipError_t thin_lstm(int w_terms, const ThinA& a, const ThinW& w, const LstmParams& p, hipStream_t st);
// Two problems of segment counts 1+1, 1+2 or 2+2 in one launch.
hipError_t thin_lstm2(int w_terms, const ThinPair& q, hipStream_t st);
hipError_t thin_store(int w_terms, const ThinA& a, const ThinW& w, const StoreParams& p, hipStream_t st);

constexpr int kShiftPad = 64;
// A decoder state of N rows: fp32 h, c [L, N, H] and feed [N, H], and the two-term copies of h (one operand of
// `plane` halfwords per layer) and feed that the products read (kb blocks of 32 columns).
struct DecodeState {
  float* h;
  float* c;
  float* feed;
  uint16_t* h16;
  uint16_t* feed16;
  size_t plane;
  int L, N, H, kb;
  int32_t* shift;               // [L, N] in whole groups of kShiftPad, written by prepare_step (split; zeros at the end)
};
// Rows b * K + k of the state = the encoder's final rows b; feed = 0.
hipError_t decode_init(const DecodeState& s, const float* final_h, const float* final_c, int B, int K, hipStream_t st);
// split: the two-term copies from h and feed, each row of a layer's product under a power of two of its own: the
// copies of h (and of feed, with layer 0's h) are scaled by 2^(kActExp + shift[l, r]). tok != NULL: tok_out [N] =
// tok with invalid ids set to 0; par_out [N] (parent != NULL) = parent with rows outside [0, N) replaced by the row
// itself; violations recorded in *err.
hipError_t prepare_step(const DecodeState& s, int split, const int32_t* tok, const int32_t* parent, int V,
                        int32_t* tok_out, int32_t* par_out, int32_t* err, hipStream_t st);

// The first M rows of an operand of `rows` rows and kblocks blocks of `terms` terms; aexp (optional): power of two
// aexp[eidx ? eidx[m] : m] added to the columns' for row m.
struct WideA {
  const void* base;
  const int32_t* eidx;
  const int32_t* aexp;
  int M;
  int rows;
  int kblocks;
  int terms;
};
// out[row(m), n] = product + bias[n] for n < ncols; row(m) = m, or (B > 0) (m % B) * S + m / B.
struct WideOut {
  const float* bias;
  float* out;
  int ldo;
  int ncols;
  int B, S;
};
hipError_t wide_store(const WideA& a, const ThinW& w, int w_terms, const WideOut& p, hipStream_t st);

// The generator: a two-term operand of M = a.rows rows against the vocabulary's weights (w.rows = ceil128(V)
// rows of w_terms terms).
hipError_t gemm_gen(const Split16& a, const Split16& w, int w_terms, const GenParams& p, hipStream_t st);
int gen_tile_cols();

// Attention coverage of the hypotheses (optional): out[r, s] = in[parent[r], s] + a[r, s] for the real
// positions (0 at pads), cp[r] = beta * sum over the real positions of log(min(out[r, s], 1)).
struct Coverage {
  const float* in;              // [N, S_max]
  float* out;                   // [N, S_max]
  const int32_t* parent;        // [N]
  double beta;
  double* cp;                   // [N]
};

// Optional per-row outputs of the attention softmax (beyond the weights themselves).
struct AttnExtra {
  const Coverage* cov;          // coverage update and penalty
  int32_t* align;               // [N]: position of the largest weight (smaller position on ties)
};

// ctx16: the contexts as a two-term operand of ceil32(Hm) columns. v_a != nullptr selects concat scores v_a .
// tanh(q_k + keys[s]) (q = the projected query); else q_k . keys[s].
hipError_t attention(const float* q, int ld_q, const float* keys, const float* v_a, const float* mem,
                     const int32_t* lens, int B, int S_max, int H, int Hm, int K, float* scores, uint16_t* ctx16,
                     float* attn, const AttnExtra& ex, hipStream_t st);
size_t attention_lds_bytes(int S_max, int H, int K);

// Generator partials of one decoder step (per row and column tile), as written by gemm_gen: the top-K comes from
// the lists (pval, pid) or, where those are null, from the logits.
struct GenPartials {
  const float* pmax;
  const float* psum;
  const float* pval;
  const int32_t* pid;
  int ntiles;
  const float* logits;
  int ld_logits, V;
  // filters (logits only), as in GenParams
  const float* pfmax;
  const uint32_t* banned_bits;
  const int32_t* unk_cnt;
  int unk_id, max_unk;
};

hipError_t lse_topk_merge(const GenPartials& gp, int M, int K, float* out_val, int32_t* out_id, float* out_lse,
                          hipStream_t st);
// Teacher-forced scoring of all steps: rows r = t * B + b of the generator partials; logp[b * ld + t] =
// want_logit[r] - logsumexp(r) for t < len[b] (0 otherwise, t < steps); nll[b] = -sum_t logp[b, t] in fp64.
hipError_t score_rows(const float* pmax, const float* psum, int ntiles, const float* want_logit, const int32_t* len,
                      int B, int steps, float* logp, int ld, double* nll, hipStream_t st);
// x [M, ncols] (the logits) -= each row's logsumexp, which goes to out_lse.
hipError_t log_probs(float* x, int ncols, const GenPartials& gp, int M, float* out_lse, hipStream_t st);

struct BeamParams {
  int B, K, V, T_max, eos, pad;
  double alpha, lp_tmax;
  double* score;
  int32_t* parent;
  int32_t* tok;
  int32_t* bp_slot;
  int32_t* bp_tok;
  float* bp_logp;
  int32_t* done;
  int32_t* steps;
  int32_t* done_count;
  double* best_norm;
  double* best_raw;
  int32_t* best_t;
  int32_t* best_slot;
  int32_t* best_tok;
  float* best_logp;
  const double* cp;             // optional coverage penalty of each row's hypothesis this step [N]
  const int32_t* align;         // optional [N]: attention argmax of each row at this step
  int32_t* bp_align;            // [T_max, N] (with align)
  int32_t* best_align;          // [B] (with align)
  int32_t* unk_cnt;             // [N] UNK tokens of each slot's hypothesis
  int unk_id;
  int32_t* tr_slot;             // optional trace [T_max, B, K]
  int32_t* tr_tok;
  double* tr_cand;
};

hipError_t beam_init(const BeamParams& p, int bos, hipStream_t st);
hipError_t beam_step(const BeamParams& p, const GenPartials& gp, int t, hipStream_t st);
hipError_t backtrack(const BeamParams& p, int32_t* out_tok, int32_t* out_len, double* out_raw, double* out_norm,
                     float* out_tok_logp, int32_t* out_align, hipStream_t st);

// out [B, T] = the source id at the aligned position of every UNK output token (t < len[b]), -1 elsewhere.
hipError_t replace_unk(const int32_t* src, int B, int S, const int32_t* tok, const int32_t* len, const int32_t* align,
                       int T, int unk, int32_t* out, hipStream_t st);

// Input validation on the device: kinds of violation recorded in a host-visible word (several threads may store
// different ones; any nonzero value reports the failure). Invalid values are replaced by safe ones.
enum { kErrLength = 1, kErrSourceId = 2, kErrToken = 3, kErrParent = 4 };
// max_len (optional): the longest length. ids [S, B] = src [B, S] with ids past each length (and invalid ids) set to
// 0; lens [B] = len clamped to [1, S]; out = the first `rows` ids' rows of the embedding table ([V][terms][32 kblocks]
// halfwords) as an operand.
hipError_t embed_src(const int32_t* src, const int32_t* len, int B, int S, int V, const void* table, int terms,
                     int kblocks, int32_t* ids, int32_t* lens, uint16_t* out, int rows, int32_t* err,
                     int32_t* max_len, hipStream_t st);
// out = the table rows of n checked ids.
hipError_t embed_rows(const int32_t* ids, int n, const void* table, int terms, int kblocks, uint16_t* out,
                      hipStream_t st);
// Teacher-forced targets per step: in_tok, want [T, B], tlen [B]; violations in *err, the longest length in *max_len.
hipError_t targets(const int32_t* tgt, const int32_t* len, int B, int T, int V, int bos, int pad, int32_t* in_tok,
                   int32_t* want, int32_t* tlen, int32_t* err, int32_t* max_len, hipStream_t st);

hipError_t fill_f32(float* dst, size_t n, float v, hipStream_t st);
// Zeros in columns width .. 32 kblocks of every row (rows rounded up to whole blocks) of up to two two-term operands.
hipError_t zero_pad16(uint16_t* a, uint16_t* b, int rows, int width, int kblocks, hipStream_t st);

}  // namespace onmt
