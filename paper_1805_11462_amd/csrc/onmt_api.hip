// C ABI of libonmt: validation, weight packing, workspace carving and the encode / decode-step /
// beam-search orchestration. All arithmetic runs in the kernels of thin.hip, wide.hip, gen.hip, attention.hip and
// beam.hip.

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <initializer_list>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/onmt.h"
#include "common.h"
#include "kernels.h"

using namespace onmt;

namespace {

thread_local std::string g_err;

int fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  g_err = buf;
  return code;
}

#define HIP_TRY(expr)                                                                              \
  do {                                                                                             \
    hipError_t e_ = (expr);                                                                        \
    if (e_ != hipSuccess) return fail(ONMT_EDEVICE, "%s: %s", #expr, hipGetErrorString(e_));       \
  } while (0)

constexpr size_t kAlign = 256;
inline size_t align_up(size_t x, size_t a = kAlign) { return (x + a - 1) / a * a; }
inline int ceil_to(int x, int m) { return (x + m - 1) / m * m; }

// Byte-offset allocator over a caller-provided buffer (used for sizing with base == 0, then carving).
struct Carver {
  size_t off = 0;
  char* base = nullptr;
  template <class T>
  T* take(size_t count) {
    off = align_up(off);
    T* p = base ? (T*)(base + off) : nullptr;
    off += count * sizeof(T);
    return p;
  }
};

// A weight matrix (rows a multiple of 128) or embedding table in fragment blocks of 1 or 2 fp16 terms, with each row's
// power of two, inside the model buffer.
struct ThinMat {
  size_t off = 0, exp_off = 0;
  int rows = 0, kblocks = 0;
  const char* base = nullptr;
  ThinW w(int kb0 = 0) const { return ThinW{base + off, (const int32_t*)(base + exp_off), rows, kblocks, kb0}; }
};

struct Dims {
  int L, ndir, Hd, Hm, H, E, Vs, Vt;
  int Hd_pad, H_pad;   // units padded to multiples of 32 (gate-blocked groups, 128-column tiles)
  bool bf16;
  int esz;             // operand element size
  int attn;            // ONMT_ATTN_GENERAL / _DOT / _CONCAT
  // fp16 terms per weight of the two-term products (split16.h): bf16 weights fit one, fp32 weights take two
  int wterms;
  // columns as the model-size refusals count them
  int pad(int w) const { return ceil_to(w, kSegK); }
  int kb(int w) const { return ceil_to(w, kFragK) / kFragK; }     // 32-column blocks of a two-term operand
};

bool dims_of(const onmt_config* c, Dims* d) {
  if (!c) return false;
  d->L = c->enc_layers;
  d->ndir = c->bidirectional ? 2 : 1;
  d->H = c->hidden;
  d->Hd = c->bidirectional ? c->hidden / 2 : c->hidden;
  d->Hm = d->ndir * d->Hd;
  d->E = c->emb;
  d->Vs = c->src_vocab;
  d->Vt = c->tgt_vocab;
  d->Hd_pad = ceil_to(d->Hd, 32);
  d->H_pad = ceil_to(d->H, 32);
  d->bf16 = c->wdtype == 1;
  d->esz = d->bf16 ? 2 : 4;
  d->attn = c->attn_type;
  d->wterms = d->bf16 ? 1 : 2;
  return true;
}

// The GEMMs address their operands through buffer descriptors, whose byte counts and row offsets are
// 32-bit and which treat offsets from 2 GiB on as "no row" (zeros): every operand read that way must be
// smaller than 2 GiB. These checks run before anything is enqueued.
constexpr uint64_t kDescLimit = 1ull << 31;
size_t model_layout(const onmt_config* c, onmt_model* m, std::vector<uint64_t>* mats = nullptr);

int check_model_limits(const onmt_config* c) {
  std::vector<uint64_t> mats;
  model_layout(c, nullptr, &mats);   // embeddings, packed LSTM / attention / generator matrices
  for (uint64_t b : mats)
    if (b >= kDescLimit)
      return fail(ONMT_EUNSUPPORTED, "a packed weight matrix or embedding table needs %llu bytes (limit 2 GiB)",
                  (unsigned long long)b);
  return ONMT_OK;
}

int check_config(const onmt_config* c) {
  if (!c) return fail(ONMT_EINVAL, "config is NULL");
  if (c->enc_layers < 1 || c->dec_layers < 1) return fail(ONMT_EINVAL, "layers must be >= 1");
  if (c->enc_layers != c->dec_layers)
    return fail(ONMT_EINVAL, "enc_layers (%d) must equal dec_layers (%d)", c->enc_layers, c->dec_layers);
  if (c->bidirectional != 0 && c->bidirectional != 1) return fail(ONMT_EINVAL, "bidirectional must be 0 or 1");
  if (c->wdtype != 0 && c->wdtype != 1) return fail(ONMT_EINVAL, "wdtype must be 0 (fp32) or 1 (bf16)");
  if (c->attn_type < ONMT_ATTN_GENERAL || c->attn_type > ONMT_ATTN_CONCAT)
    return fail(ONMT_EINVAL, "attn_type must be 0 (general), 1 (dot) or 2 (concat)");
  if (c->emb < 4 || c->hidden < 4 || c->src_vocab < 1 || c->tgt_vocab < 4)
    return fail(ONMT_EINVAL, "emb/hidden >= 4, src_vocab >= 1, tgt_vocab >= 4 required");
  if (c->emb > 8192 || c->hidden > 8192 || c->enc_layers > 64) return fail(ONMT_EUNSUPPORTED, "model too large");
  if (c->tgt_vocab > 131072) return fail(ONMT_EUNSUPPORTED, "target vocabulary larger than 131072");
  const int Hd = c->bidirectional ? c->hidden / 2 : c->hidden;
  if (c->bidirectional && c->hidden % 2) return fail(ONMT_EINVAL, "bidirectional needs an even hidden size");
  if (c->emb % 4 || c->hidden % 4 || Hd % 4)
    return fail(ONMT_EUNSUPPORTED, "emb, hidden and per-direction hidden must be multiples of 4");
  if (c->wdtype == 1 && c->emb % 8) return fail(ONMT_EUNSUPPORTED, "bf16 models need emb a multiple of 8");
  const int ids[4] = {c->pad_id, c->unk_id, c->bos_id, c->eos_id};
  for (int i = 0; i < 4; ++i)
    if (ids[i] < 0 || ids[i] >= c->tgt_vocab) return fail(ONMT_EINVAL, "special ids must be in [0, tgt_vocab)");
  return check_model_limits(c);
}

struct WeightSpec {
  int64_t rows, cols;   // cols = 1 for vectors
};

std::vector<WeightSpec> weight_specs(const onmt_config* c) {
  Dims d;
  dims_of(c, &d);
  std::vector<WeightSpec> v;
  v.push_back({d.Vs, d.E});
  for (int l = 0; l < d.L; ++l) {
    const int in = l == 0 ? d.E : d.Hm;
    for (int dir = 0; dir < d.ndir; ++dir) {
      v.push_back({4LL * d.Hd, in + d.Hd});
      v.push_back({4LL * d.Hd, 1});
    }
  }
  v.push_back({d.Vt, d.E});
  for (int l = 0; l < d.L; ++l) {
    const int in = l == 0 ? d.E + d.H : d.H;
    v.push_back({4LL * d.H, in + d.H});
    v.push_back({4LL * d.H, 1});
  }
  if (d.attn == ONMT_ATTN_GENERAL) v.push_back({d.H, d.Hm});
  if (d.attn == ONMT_ATTN_CONCAT) {
    v.push_back({d.H, d.H + d.Hm});
    v.push_back({d.H, 1});
  }
  v.push_back({d.H, d.Hm + d.H});
  v.push_back({d.Vt, d.H});
  v.push_back({d.Vt, 1});
  return v;
}

// Row of packed gate-blocked matrices for (gate, unit): groups of kUnitGroup units hold 4 gates x kUnitGroup rows.
inline int gate_row(int gate, int unit) {
  return (unit / kUnitGroup) * (4 * kUnitGroup) + gate * kUnitGroup + unit % kUnitGroup;
}

}  // namespace

struct onmt_model {
  onmt_config cfg;
  Dims d;
  char* dev = nullptr;
  ThinMat E_src, E_tgt;                    // rows carry the power of two that undoes their own scale; E_src's rows are
                                           // contiguous ([terms][32 kblocks]), gathered by token id
  // Encoder. Bidirectional: every layer has an input projection (both directions stacked) and a recurrent
  // matrix per direction. Unidirectional: layer 0 likewise; layers >= 1 keep [input | recurrent] in one
  // matrix, so that they can run one timestep behind the layer below in the same launch.
  std::vector<ThinMat> enc_x;              // per layer: both directions stacked [ndir * 4 Hd_pad, in]
  std::vector<const float*> enc_bias;      // per layer [ndir * 4 Hd_pad]
  std::vector<ThinMat> enc_h;              // per layer * ndir: [4 Hd_pad, Hd]
  std::vector<ThinMat> enc_xh;             // unidirectional layers >= 1: [4 Hd_pad, [in | Hd]]
  ThinMat dec_emb;                         // decoder layer 0's embedding columns (for emb_gates) [4 H_pad, E]
  std::vector<ThinMat> dec_t;              // per layer, columns [feed | recurrent] or [below | recurrent]
  std::vector<const float*> dec_bias;      // per layer [4 H_pad]
  ThinMat W_a;                             // memory side of the score: general W_a, concat's memory columns
  ThinMat W_q;                             // concat: the query columns of W_a
  const float* v_a = nullptr;              // concat [H]
  ThinMat W_c;                             // columns [context | query]
  size_t W_s_off = 0;
  Split16 W_s{};                           // the generator's weights: ceil128(Vt) rows of wterms fp16 terms
  const int32_t* W_s_exp = nullptr;        // power of two that undoes a vocabulary column's operand scales
  const float* b_s = nullptr;
  // decoder layer 0's input-projection rows for every target token, E_tgt[v] W_e^T in the packed (gate-
  // blocked) column order, fp32 [Vt, 4 H_pad]; computed on the device when the model is created
  float* emb_gates = nullptr;
  size_t image_bytes = 0;    // the uploaded part of the model buffer (everything before emb_gates)
  // kernel timing
  int prof = 0;              // time every prof-th generator launch (0: off)
  unsigned prof_kinds = 0;                      // bit k: launches of kind k are timed
  long long prof_seq[ONMT_KERNEL_KINDS] = {};   // launches of each kind seen while timing is on
  bool prof_open[ONMT_KERNEL_KINDS] = {};       // the current launch of the kind has a start event
  size_t prof_pair[ONMT_KERNEL_KINDS] = {};     // ... recorded as event pair ev[prof_pair], ev[prof_pair + 1]
  int prof_n[ONMT_KERNEL_KINDS] = {};
  double prof_ms[ONMT_KERNEL_KINDS] = {};
  std::vector<hipEvent_t> ev;   // reusable start/stop pairs
  std::vector<int> ev_kind;     // kind of each recorded pair
  size_t ev_used = 0;
  // finish checks of the beam search: two pinned host words the done count is copied into, one event each
  int32_t* done_host = nullptr;
  hipEvent_t done_ev[2] = {nullptr, nullptr};
  // input validation: ONMT_VALIDATE_HOST or ONMT_VALIDATE_DEVICE. err_host: pinned words the checking kernels write:
  // [0] violations since the last onmt_device_status (device mode), then, for calls that wait for their checks
  // (host mode), [1] violations and [2], [3] the longest source and target length.
  int validation = ONMT_VALIDATE_HOST;
  int32_t* err_host = nullptr;
};

namespace {

// Model buffer layout (offsets only); fills m's offsets when m != nullptr, and the byte size of every
// matrix the GEMMs read through buffer descriptors into *mats when given.
size_t model_layout(const onmt_config* c, onmt_model* m, std::vector<uint64_t>* mats) {
  Dims d;
  dims_of(c, &d);
  Carver cv;
  auto vec = [&](size_t n) {
    cv.off = align_up(cv.off);
    size_t o = cv.off;
    cv.off += n * sizeof(float);
    return o;
  };
  // limit: the size the refusal rule counts for the matrix (128-column padding of each segment)
  auto thin = [&](int rows, int kblocks, uint64_t limit) {
    ThinMat t;
    t.rows = rows;
    t.kblocks = kblocks;
    cv.off = align_up(cv.off);
    t.off = cv.off;
    cv.off += split16_bytes(rows, kblocks, d.wterms);
    t.exp_off = vec(rows);
    if (mats) mats->push_back(limit);
    return t;
  };
  auto lim = [&](int rows, int kp) { return (uint64_t)rows * kp * d.esz; };
  const ThinMat esrc = thin(d.Vs, d.kb(d.E), lim(d.Vs, d.E));
  std::vector<ThinMat> ex, eh, exh, dt;
  std::vector<size_t> eb, db;
  for (int l = 0; l < d.L; ++l) {
    const int in = l == 0 ? d.E : d.Hm, r = 4 * d.Hd_pad;
    if (d.ndir == 1 && l > 0) {
      ex.push_back(ThinMat{});
      eh.push_back(ThinMat{});
      exh.push_back(thin(r, d.kb(in) + d.kb(d.Hd), lim(r, d.pad(in) + d.pad(d.Hd))));
    } else {
      ex.push_back(thin(d.ndir * r, d.kb(in), lim(d.ndir * r, d.pad(in))));
      for (int dir = 0; dir < d.ndir; ++dir) eh.push_back(thin(r, d.kb(d.Hd), lim(r, d.pad(d.Hd))));
      exh.push_back(ThinMat{});
    }
    eb.push_back(vec((size_t)d.ndir * r));
  }
  const ThinMat etgt = thin(d.Vt, d.kb(d.E), lim(d.Vt, d.E));
  for (int l = 0; l < d.L; ++l) {
    const uint64_t kp = (l == 0 ? d.pad(d.E) : 0) + 2 * d.pad(d.H);
    dt.push_back(thin(4 * d.H_pad, 2 * d.kb(d.H), 4 * d.H_pad * kp * d.esz));
    db.push_back(vec((size_t)4 * d.H_pad));
  }
  const ThinMat demb = thin(4 * d.H_pad, d.kb(d.E), lim(4 * d.H_pad, d.pad(d.E)));
  const int hr = ceil_to(d.H, 128);
  const ThinMat wa = d.attn != ONMT_ATTN_DOT ? thin(hr, d.kb(d.Hm), lim(hr, d.pad(d.Hm))) : ThinMat{};
  ThinMat wq = d.attn == ONMT_ATTN_CONCAT ? thin(hr, d.kb(d.H), lim(hr, d.pad(d.H))) : ThinMat{};
  const size_t va = d.attn == ONMT_ATTN_CONCAT ? vec(d.H) : 0;
  ThinMat wc = thin(hr, d.kb(d.Hm) + d.kb(d.H), lim(hr, d.pad(d.Hm) + d.pad(d.H)));
  cv.off = align_up(cv.off);
  const size_t ws_off = cv.off;
  const Split16 ws{nullptr, ceil_to(d.Vt, 128), d.kb(d.H)};
  const uint64_t ws_bytes = split16_bytes(ws.rows, ws.kblocks, d.wterms);
  cv.off += ws_bytes;
  if (mats) mats->push_back((uint64_t)ws.rows * d.pad(d.H) * d.esz);   // the limit is set on 128-column padding
  const size_t wse = vec(ws.rows);
  size_t bs = vec(ceil_to(d.Vt, 128));
  const size_t image = align_up(cv.off);
  const size_t eg = vec((size_t)d.Vt * 4 * d.H_pad);
  const size_t total = align_up(cv.off);
  if (m) {
    char* base = m->dev;
    auto fix_thin = [&](ThinMat t) {
      t.base = base;
      return t;
    };
    m->E_src = fix_thin(esrc);
    m->E_tgt = fix_thin(etgt);
    for (auto& t : ex) m->enc_x.push_back(fix_thin(t));
    for (auto o : eb) m->enc_bias.push_back((const float*)(base + o));
    for (auto& t : eh) m->enc_h.push_back(fix_thin(t));
    for (auto& t : exh) m->enc_xh.push_back(fix_thin(t));
    m->dec_emb = fix_thin(demb);
    for (auto& t : dt) m->dec_t.push_back(fix_thin(t));
    for (auto o : db) m->dec_bias.push_back((const float*)(base + o));
    if (d.attn != ONMT_ATTN_DOT) m->W_a = fix_thin(wa);
    if (d.attn == ONMT_ATTN_CONCAT) {
      m->W_q = fix_thin(wq);
      m->v_a = (const float*)(base + va);
    }
    m->W_c = fix_thin(wc);
    m->W_s_off = ws_off;
    m->W_s = ws;
    m->W_s.base = base + ws_off;
    m->W_s_exp = (const int32_t*)(base + wse);
    m->b_s = (const float*)(base + bs);
    m->emb_gates = (float*)(base + eg);
    m->image_bytes = image;
  }
  return total;
}

// Host-side packing into the image of the device buffer.
struct HostImage {
  std::vector<char> buf;
  bool bf16;
  std::vector<float> row;      // scratch of pack_thin
  void putf(size_t off, size_t idx, float v) { ((float*)(buf.data() + off))[idx] = v; }
};

// n weights as the products take them (bf16 models: rounded).
void weight_row(const HostImage& img, const float* src, int n, float* dst) {
  for (int j = 0; j < n; ++j)
    dst[j] = img.bf16 ? finite_or_nan(host_bf16_to_f32(f32_to_bf16_bits(src[j])), 0x10000u) : finite_or_nan(src[j]);
}

// Row r of a matrix or embedding table: columns w[i] values of src[i] from K block kb[i] on, under one row exponent.
struct RowPart {
  const float* src;
  int w, kb;
};
void pack_thin(HostImage& img, const ThinMat& t, int terms, int r, std::initializer_list<RowPart> parts,
               bool table = false) {
  std::vector<float>& row = img.row;
  row.assign((size_t)t.kblocks * kFragK, 0.f);
  for (const RowPart& q : parts) weight_row(img, q.src, q.w, row.data() + (size_t)q.kb * kFragK);
  const int e = host_row_exp(row.data(), (int)row.size());
  // a product column is undone by -(kActExp + e); a table's rows take the place of activations scaled by kActExp
  ((int32_t*)(img.buf.data() + t.exp_off))[r] = table ? kActExp - e : -(kActExp + e);
  host_pack_row((uint16_t*)(img.buf.data() + t.off), r, t.kblocks, terms, row.data(), e);
}

}  // namespace

// ====================================================================== allocation-free step scratch

// Scratch of onmt_decode_step_noalloc: the step workspace of one decoder step (attention scores and
// context, generator partials, checked ids), a file-scope device array instead of a caller's buffer. Each
// GPU holds its own copy, at its own address, until the process ends. In host code `scratch` names a
// host-side stand-in, never the device memory: kernels get the address hipGetSymbolAddress returns for
// the current device, kept per device below.
// The refusal rule counts ONMT_NOALLOC_SCRATCH_BYTES with unpadded contexts; the array leaves room for their
// padding to whole fragment blocks, at most 112 bytes on a row of 56 or more.
constexpr size_t kScratchBytes = 3 * (size_t)ONMT_NOALLOC_SCRATCH_BYTES;
static __device__ __align__(256) char scratch[kScratchBytes];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// The current device's address of `scratch`, looked up once per device (at onmt_model_create, the
// library's set-up call, or at the entry point's first call on a device no model was created on).
int noalloc_scratch(void** out) {
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= kMaxDevices) return fail(ONMT_EUNSUPPORTED, "device index %d beyond %d", dev, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (!p) return fail(ONMT_EDEVICE, "no device address for the step scratch");
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return ONMT_OK;
}

}  // namespace

// ====================================================================== ABI

extern "C" {

const char* onmt_last_error(void) { return g_err.c_str(); }

int onmt_num_weights(const onmt_config* cfg) {
  int rc = check_config(cfg);
  if (rc) return rc;
  return (int)weight_specs(cfg).size();
}

int64_t onmt_weight_numel(const onmt_config* cfg, int i) {
  int rc = check_config(cfg);
  if (rc) return rc;
  auto v = weight_specs(cfg);
  if (i < 0 || i >= (int)v.size()) return fail(ONMT_EINVAL, "weight index %d out of range", i);
  return v[i].rows * v[i].cols;
}

size_t onmt_model_bytes(const onmt_config* cfg) {
  if (check_config(cfg)) return 0;
  return model_layout(cfg, nullptr);
}

int onmt_model_create(const onmt_config* cfg, const float* const* host_weights, int n_weights, void* dev_buf,
                      size_t dev_bytes, void* stream, onmt_model** out) {
  int rc = check_config(cfg);
  if (rc) return rc;
  if (!out) return fail(ONMT_EINVAL, "out is NULL");
  *out = nullptr;
  auto specs = weight_specs(cfg);
  if (n_weights != (int)specs.size()) return fail(ONMT_EINVAL, "expected %d weight arrays, got %d", (int)specs.size(), n_weights);
  if (!host_weights) return fail(ONMT_EINVAL, "host_weights is NULL");
  for (int i = 0; i < n_weights; ++i)
    if (!host_weights[i]) return fail(ONMT_EINVAL, "host weight %d is NULL", i);
  if (!dev_buf) return fail(ONMT_EINVAL, "dev_buf is NULL");
  if ((uintptr_t)dev_buf % kAlign) return fail(ONMT_EINVAL, "dev_buf must be 256-byte aligned");
  const size_t need = model_layout(cfg, nullptr);
  if (dev_bytes < need) return fail(ONMT_ESIZE, "model buffer %zu bytes < %zu", dev_bytes, need);

  onmt_model* m = new onmt_model();
  m->cfg = *cfg;
  dims_of(cfg, &m->d);
  m->dev = (char*)dev_buf;
  model_layout(cfg, m);
  const Dims& d = m->d;

  HostImage img;
  img.bf16 = d.bf16;
  img.buf.assign(m->image_bytes, 0);
  auto off_of = [&](const void* p) { return (size_t)((const char*)p - m->dev); };
  int wi = 0;
  // E_src
  {
    const float* s = host_weights[wi++];
    const int ld = d.kb(d.E) * kFragK;
    std::vector<float> row(ld, 0.f);
    for (int r = 0; r < d.Vs; ++r) {
      weight_row(img, s + (size_t)r * d.E, d.E, row.data());
      const int e = host_row_exp(row.data(), d.E);
      ((int32_t*)(img.buf.data() + m->E_src.exp_off))[r] = kActExp - e;
      uint16_t* hi = (uint16_t*)(img.buf.data() + m->E_src.off) + (size_t)r * ld * d.wterms;
      host_split(row.data(), ld, e, hi, d.wterms == 2 ? hi + ld : nullptr, 8);
    }
  }
  for (int l = 0; l < d.L; ++l) {
    const int in = l == 0 ? d.E : d.Hm;
    const size_t bo = off_of(m->enc_bias[l]);
    const bool joint = d.ndir == 1 && l > 0;
    for (int dir = 0; dir < d.ndir; ++dir) {
      const float* W = host_weights[wi++];
      const float* bvec = host_weights[wi++];
      for (int g = 0; g < 4; ++g)
        for (int u = 0; u < d.Hd; ++u) {
          const float* row = W + (size_t)(g * d.Hd + u) * (in + d.Hd);
          const int xr = dir * 4 * d.Hd_pad + gate_row(g, u);
          if (joint) {   // segments [layer below | recurrent]
            pack_thin(img, m->enc_xh[l], d.wterms, xr, {{row, in, 0}, {row + in, d.Hd, d.kb(in)}});
          } else {
            pack_thin(img, m->enc_x[l], d.wterms, xr, {{row, in, 0}});
            pack_thin(img, m->enc_h[l * d.ndir + dir], d.wterms, gate_row(g, u), {{row + in, d.Hd, 0}});
          }
          img.putf(bo, xr, bvec[g * d.Hd + u]);
        }
    }
  }
  {
    const float* s = host_weights[wi++];
    for (int r = 0; r < d.Vt; ++r) pack_thin(img, m->E_tgt, d.wterms, r, {{s + (size_t)r * d.E, d.E, 0}}, true);
  }
  for (int l = 0; l < d.L; ++l) {
    const float* W = host_weights[wi++];
    const float* bvec = host_weights[wi++];
    const size_t bo = off_of(m->dec_bias[l]);
    const int in = l == 0 ? d.E + d.H : d.H, kb = d.kb(d.H);
    for (int g = 0; g < 4; ++g)
      for (int u = 0; u < d.H; ++u) {
        const float* row = W + (size_t)(g * d.H + u) * (in + d.H);
        const int pr = gate_row(g, u);
        if (l == 0) {   // [embedding] apart; [feed | recurrent]
          pack_thin(img, m->dec_emb, d.wterms, pr, {{row, d.E, 0}});
          pack_thin(img, m->dec_t[l], d.wterms, pr, {{row + d.E, d.H, 0}, {row + d.E + d.H, d.H, kb}});
        } else {        // [layer below | recurrent]
          pack_thin(img, m->dec_t[l], d.wterms, pr, {{row, d.H, 0}, {row + d.H, d.H, kb}});
        }
        img.putf(bo, pr, bvec[g * d.H + u]);
      }
  }
  {
    if (d.attn == ONMT_ATTN_GENERAL) {
      const float* Wa = host_weights[wi++];
      for (int r = 0; r < d.H; ++r) pack_thin(img, m->W_a, d.wterms, r, {{Wa + (size_t)r * d.Hm, d.Hm, 0}});
    } else if (d.attn == ONMT_ATTN_CONCAT) {   // columns [query | memory]
      const float* Wa = host_weights[wi++];
      for (int r = 0; r < d.H; ++r) {
        pack_thin(img, m->W_q, d.wterms, r, {{Wa + (size_t)r * (d.H + d.Hm), d.H, 0}});
        pack_thin(img, m->W_a, d.wterms, r, {{Wa + (size_t)r * (d.H + d.Hm) + d.H, d.Hm, 0}});
      }
      const float* va = host_weights[wi++];
      const size_t vo = off_of(m->v_a);
      for (int r = 0; r < d.H; ++r) img.putf(vo, r, va[r]);
    }
    const float* Wc = host_weights[wi++];
    for (int r = 0; r < d.H; ++r) {
      const float* row = Wc + (size_t)r * (d.Hm + d.H);
      pack_thin(img, m->W_c, d.wterms, r, {{row, d.Hm, 0}, {row + d.Hm, d.H, d.kb(d.Hm)}});
    }
    const float* Ws = host_weights[wi++];
    {
      uint16_t* o = (uint16_t*)(img.buf.data() + m->W_s_off);
      int32_t* ex = (int32_t*)(img.buf.data() + off_of(m->W_s_exp));
      std::vector<float> row((size_t)m->W_s.kblocks * kFragK, 0.f);
      for (int r = 0; r < d.Vt; ++r) {
        weight_row(img, Ws + (size_t)r * d.H, d.H, row.data());
        const int e = host_row_exp(row.data(), d.H);
        ex[r] = -(kActExp + e);
        host_pack_row(o, r, m->W_s.kblocks, d.wterms, row.data(), e);
      }
    }
    const float* bs = host_weights[wi++];
    const size_t bo = off_of(m->b_s);
    for (int r = 0; r < d.Vt; ++r) img.putf(bo, r, bs[r]);
  }
  hipStream_t st = (hipStream_t)stream;
  hipError_t e = hipMemcpyAsync(dev_buf, img.buf.data(), m->image_bytes, hipMemcpyHostToDevice, st);
  if (e == hipSuccess) {
    // decoder layer 0: the embedding columns of its packed matrix against every target embedding row
    const WideA a{m->E_tgt.w().base, nullptr, m->E_tgt.w().wexp, d.Vt, d.Vt, d.kb(d.E), d.wterms};
    e = wide_store(a, m->dec_emb.w(), d.wterms, WideOut{nullptr, m->emb_gates, 4 * d.H_pad, 4 * d.H_pad, 0, 0}, st);
  }
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e == hipSuccess) {
    e = hipHostMalloc((void**)&m->err_host, 4 * sizeof(int32_t), hipHostMallocDefault);
    if (e == hipSuccess) memset(m->err_host, 0, 4 * sizeof(int32_t));
  }
  if (e != hipSuccess) {
    if (m->err_host) hipHostFree(m->err_host);
    delete m;
    return fail(ONMT_EDEVICE, "weight upload failed: %s", hipGetErrorString(e));
  }
  void* sp = nullptr;
  rc = noalloc_scratch(&sp);    // this device's copy of the allocation-free entry point's scratch array
  if (rc) {
    hipHostFree(m->err_host);
    delete m;
    return rc;
  }
  *out = m;
  return ONMT_OK;
}

int onmt_model_destroy(onmt_model* m) {
  if (!m) return fail(ONMT_EINVAL, "model is NULL");
  for (auto e : m->ev) hipEventDestroy(e);
  for (auto e : m->done_ev)
    if (e) hipEventDestroy(e);
  if (m->done_host) hipHostFree(m->done_host);
  if (m->err_host) hipHostFree(m->err_host);
  delete m;
  return ONMT_OK;
}

}  // extern "C"

// ====================================================================== workspaces

namespace {

struct EncWs {
  int32_t* lens;
  int32_t* src;      // [S, B] checked token ids
  float* memory;     // [B*S, Hm]
  float* keys;       // [B*S, H]: W_a m_s (general), the memory-side term of concat, the memory itself (dot)
  float* final_h;    // [L, B, H]
  float* final_c;
  float* gx;         // [S*B, ndir * 4 Hd_pad], row s * B + b
  uint16_t* x16;     // source embeddings as an operand of wterms terms: x16_rows of the rows s * B + b at a time
  int x16_rows;
  // Two-term operands of the layers' outputs (one layer writes y16[l & 1] while it reads the other), row s * B + b
  uint16_t* y16[2];
  // state after an even / odd timestep, one slot per layer and direction: h, c [slots, B, Hd] and h as an operand
  float* hs[2];
  float* cs[2];
  uint16_t* hs16[2];
  size_t hs_plane;   // halfwords of one slot of hs16
  size_t zero_n;     // floats from hs[1] on that hold the zero state before the first step (hs[1], cs[1], hs16[1])
};

// The source embeddings are gathered in slices of at most this many bytes (whole 64-row tiles): their width does not
// depend on the memory's, so a batch within the memory's limits could need more than the 4 GiB a product addresses.
constexpr size_t kEmbedSliceBytes = 256u << 20;

size_t enc_layout(const Dims& d, int B, int S, char* base, EncWs* w) {
  Carver c;
  c.base = base;
  EncWs t;
  const size_t BS = (size_t)B * S;
  t.lens = c.take<int32_t>(B);
  t.src = c.take<int32_t>(BS);
  t.memory = c.take<float>(BS * d.Hm);
  t.keys = d.attn == ONMT_ATTN_DOT ? t.memory : c.take<float>(BS * d.H);
  t.final_h = c.take<float>((size_t)d.L * B * d.H);
  t.final_c = c.take<float>((size_t)d.L * B * d.H);
  t.gx = c.take<float>(BS * d.ndir * 4 * d.Hd_pad);
  const size_t slice = kEmbedSliceBytes / (split16_bytes(64, d.kb(d.E), d.wterms)) * 64;
  t.x16_rows = (int)(BS < slice ? BS : slice);
  t.x16 = c.take<uint16_t>(split16_bytes(t.x16_rows, d.kb(d.E), d.wterms) / 2);
  for (int i = 0; i < 2; ++i) t.y16[i] = c.take<uint16_t>(split16_bytes(BS, d.kb(d.Hm), 2) / 2);
  const size_t slots = (size_t)d.ndir * d.L;
  t.hs_plane = split16_bytes(B, d.kb(d.Hd), 2) / 2;
  size_t zero0 = 0;
  for (int i = 0; i < 2; ++i) {
    zero0 = align_up(c.off);
    t.hs[i] = c.take<float>(slots * B * d.Hd);
    t.cs[i] = c.take<float>(slots * B * d.Hd);
    t.hs16[i] = c.take<uint16_t>(slots * t.hs_plane);
  }
  t.zero_n = (c.off - zero0) / sizeof(float);
  if (w) *w = t;
  return align_up(c.off);
}

// Whether an external step makes the two-term copies of its input state from the fp32 h and feed, which a caller may
// have written: always for fp32 models, and for bf16 models whose hidden size is not a multiple of 8 (the others
// read the copies their producer left beside them).
int split_state(const Dims& d) { return !d.bf16 || d.H % 8 != 0; }

struct State {
  float* h;      // [L, N, H]
  float* c;
  float* feed;   // [N, H]
  // h and feed as two-term fp16 operands, one of `plane` halfwords per layer (written by their producers). Models that
  // split their input state have one plane more (step_input).
  uint16_t* h16;
  uint16_t* feed16;
  size_t plane;
  int32_t* split_shift;  // [L, N]: powers of two of the copies an external step makes
  const int32_t* shift = nullptr;   // those of this state's h16 and feed16 (null: none, as their producers write them)
  // scoring keeps every step's feed16 in one operand of feed16_rows rows, this step's from row feed16_r0 on
  int feed16_r0 = 0, feed16_rows = 0;
};

size_t state_layout(const Dims& d, int N, char* base, State* s) {
  Carver c;
  c.base = base;
  State t;
  t.h = c.take<float>((size_t)d.L * N * d.H);
  t.c = c.take<float>((size_t)d.L * N * d.H);
  t.feed = c.take<float>((size_t)N * d.H);
  t.plane = split16_bytes(N, d.kb(d.H), 2) / 2;
  t.h16 = c.take<uint16_t>((d.L + split_state(d)) * t.plane);
  t.feed16 = c.take<uint16_t>(t.plane);
  t.split_shift = split_state(d) ? c.take<int32_t>(align_up((size_t)d.L * N, kShiftPad)) : nullptr;
  if (s) *s = t;
  return align_up(c.off);
}

// What an external step reads of the state `in` when it writes the state `out`. Copies that the step makes itself go
// into `out` (a caller's `in` is not written): layer l's h into plane l + 1, which layer l reads while it writes plane
// l, and the feed into the place of the next one, which is written after layer 0 has read this.
State step_input(const Dims& d, const State& in, const State& out) {
  State s = in;
  if (split_state(d)) {
    s.h16 = out.h16 + out.plane;
    s.feed16 = out.feed16;
    s.split_shift = out.split_shift;
    s.shift = out.split_shift;
  }
  return s;
}

// The parts of a State the kernels that fill it write.
DecodeState decode_state(const Dims& d, const State& s, int N) {
  return DecodeState{s.h, s.c, s.feed, s.h16, s.feed16, s.plane, d.L, N, d.H, d.kb(d.H), s.split_shift};
}

struct StepWs {
  uint16_t* ctx16; // [N, Hm] attention contexts as a two-term operand
  float* scores;   // [N, S_max] raw attention scores
  float* qproj;    // [N, H] concat: query columns of W_a times the decoder output
  float* pmax;     // [N, ntiles]
  float* psum;
  float* logits;   // [N, ld_logits] (null: lists instead)
  float* pval;     // [N, ntiles, K] top-K lists: K = 1, too many logits, and the allocation-free step's scratch
  int32_t* pid;
  float* lse;      // [N]
  int32_t* align;  // [N] attention argmax
  float* pfmax;    // [N, ntiles] largest allowed logit per tile (hypothesis filters)
  int32_t* tok_s;  // [N] previous tokens and parents checked on the device (device validation)
  int32_t* par_s;
  int ntiles;
  int ld_logits;
};

// A workspace holds logits up to this size (1/18 of the card's memory), beyond it per-tile top-K lists (8 K bytes per 128
// logits), so that batches of very many rows do not need 4 bytes per row and word. Lists take less room and more
// time: step of 44000 rows of 50000 words, K = 10: 1.4 GB and 16.7 ms against 8.8 GB and 12.4.
constexpr size_t kMaxLogitsBytes = 16ull << 30;

size_t step_layout(const Dims& d, int B, int S, int K, char* base, StepWs* w, bool lists = false) {
  Carver c;
  c.base = base;
  StepWs t;
  const size_t N = (size_t)B * K;
  t.ntiles = (d.Vt + gen_tile_cols() - 1) / gen_tile_cols();
  t.ctx16 = c.take<uint16_t>(split16_bytes(N, d.kb(d.Hm), 2) / 2);
  t.scores = c.take<float>(N * S);
  t.qproj = d.attn == ONMT_ATTN_CONCAT ? c.take<float>(N * d.H) : nullptr;
  t.pmax = c.take<float>(N * t.ntiles);
  t.psum = c.take<float>(N * t.ntiles);
  t.ld_logits = t.ntiles * gen_tile_cols();
  lists = lists || K == 1 || N * t.ld_logits * sizeof(float) > kMaxLogitsBytes;
  t.logits = lists ? nullptr : c.take<float>(N * t.ld_logits);
  t.pval = lists ? c.take<float>(N * t.ntiles * K) : nullptr;
  t.pid = lists ? c.take<int32_t>(N * t.ntiles * K) : nullptr;
  t.lse = c.take<float>(N);
  t.align = c.take<int32_t>(N);
  t.pfmax = c.take<float>(N * t.ntiles);
  t.tok_s = c.take<int32_t>(N);
  t.par_s = c.take<int32_t>(N);
  if (w) *w = t;
  return align_up(c.off);
}

struct SearchWs {
  EncWs enc;
  State st[2];
  StepWs step;
  BeamParams bp;
  float* cov[2];     // [N, S] attention coverage of the hypotheses (ping-pong with the state)
  double* cp;        // [N] coverage penalty of each row's hypothesis at the current step
  uint32_t* banned_bits;   // [ceil(V / 32)]
};

size_t search_layout(const Dims& d, int B, int S, int K, int T, char* base, SearchWs* w) {
  Carver c;
  c.base = base;
  SearchWs t{};
  const size_t N = (size_t)B * K;
  const size_t eb = enc_layout(d, B, S, nullptr, nullptr);
  char* e = c.take<char>(eb);
  enc_layout(d, B, S, e, &t.enc);
  for (int i = 0; i < 2; ++i) {
    const size_t sb = state_layout(d, (int)N, nullptr, nullptr);
    char* s = c.take<char>(sb);
    state_layout(d, (int)N, s, &t.st[i]);
  }
  const size_t pb = step_layout(d, B, S, K, nullptr, nullptr);
  char* p = c.take<char>(pb);
  step_layout(d, B, S, K, p, &t.step);
  BeamParams& q = t.bp;
  q.score = c.take<double>(N);
  q.parent = c.take<int32_t>(N);
  q.tok = c.take<int32_t>(N);
  q.bp_slot = c.take<int32_t>((size_t)T * N);
  q.bp_tok = c.take<int32_t>((size_t)T * N);
  q.bp_logp = c.take<float>((size_t)T * N);
  q.done = c.take<int32_t>(B);
  q.steps = c.take<int32_t>(B);
  q.done_count = c.take<int32_t>(1);
  q.best_norm = c.take<double>(B);
  q.best_raw = c.take<double>(B);
  q.best_t = c.take<int32_t>(B);
  q.best_slot = c.take<int32_t>(B);
  q.best_tok = c.take<int32_t>(B);
  q.best_logp = c.take<float>(B);
  for (int i = 0; i < 2; ++i) t.cov[i] = c.take<float>(N * S);
  t.cp = c.take<double>(N);
  q.bp_align = c.take<int32_t>((size_t)T * N);
  q.best_align = c.take<int32_t>(B);
  q.unk_cnt = c.take<int32_t>(N);
  t.banned_bits = c.take<uint32_t>((size_t)(d.Vt + 31) / 32);
  if (w) *w = t;
  return align_up(c.off);
}

struct ScoreWs {
  EncWs enc;
  State st[2];
  StepWs step;
  int32_t* in_tok;     // [T, B] decoder input at step t
  int32_t* want;       // [T, B] target predicted at step t
  int32_t* tlen;       // [B]
  float* feeds;        // [T, B, H] attentional vector of every step (the generator's input)
  uint16_t* feeds16;   // the same as a two-term fp16 operand of T * B rows
  float* gpmax;        // [T * B, ntiles] generator partials of all steps
  float* gpsum;
  float* want_logit;   // [T, B]
  double* nll;         // [B]
};

size_t score_layout(const Dims& d, int B, int S, int T, char* base, ScoreWs* w) {
  Carver c;
  c.base = base;
  ScoreWs t{};
  const size_t eb = enc_layout(d, B, S, nullptr, nullptr);
  char* e = c.take<char>(eb);
  enc_layout(d, B, S, e, &t.enc);
  for (int i = 0; i < 2; ++i) {
    const size_t sb = state_layout(d, B, nullptr, nullptr);
    char* p = c.take<char>(sb);
    state_layout(d, B, p, &t.st[i]);
  }
  const size_t pb = step_layout(d, B, S, 1, nullptr, nullptr, true);   // no per-step logits in scoring
  char* p = c.take<char>(pb);
  step_layout(d, B, S, 1, p, &t.step, true);
  t.in_tok = c.take<int32_t>((size_t)T * B);
  t.want = c.take<int32_t>((size_t)T * B);
  t.tlen = c.take<int32_t>(B);
  t.feeds = c.take<float>((size_t)T * B * d.H);
  t.feeds16 = c.take<uint16_t>(split16_bytes((size_t)T * B, d.kb(d.H), 2) / 2);
  t.gpmax = c.take<float>((size_t)T * B * t.step.ntiles);
  t.gpsum = c.take<float>((size_t)T * B * t.step.ntiles);
  t.want_logit = c.take<float>((size_t)T * B);
  t.nll = c.take<double>(B);
  if (w) *w = t;
  return align_up(c.off);
}

// Workspace operands that the GEMMs read through buffer descriptors (see kDescLimit): the encoder's
// memory, layer outputs and keys [B * S, Hm or H], the decoder's state rows and attentional vectors
// [B * K, Hm or H] (as two-term operands no wider), and scoring's attentional vectors of all steps [T * B, H].
int check_ws_limits(const Dims& d, long long B, long long S, long long K, long long T) {
  const long long w = d.Hm > d.H ? d.Hm : d.H;
  const uint64_t enc = (uint64_t)(B * S) * (uint64_t)ceil_to((int)w, kSegK) * 4;
  const uint64_t dec = (uint64_t)(B * K) * (uint64_t)ceil_to((int)w, kSegK) * 4;
  const uint64_t sco = (uint64_t)(B * T) * (uint64_t)ceil_to(d.H, kSegK) * 4;
  if (enc >= kDescLimit)
    return fail(ONMT_EUNSUPPORTED, "B * S_max = %lld source positions need a %llu-byte memory bank (limit 2 GiB)",
                B * S, (unsigned long long)enc);
  if (dec >= kDescLimit)
    return fail(ONMT_EUNSUPPORTED, "B * beam = %lld hypothesis rows need %llu-byte state operands (limit 2 GiB)",
                B * K, (unsigned long long)dec);
  if (sco >= kDescLimit)
    return fail(ONMT_EUNSUPPORTED, "B * T_max = %lld scored rows need %llu bytes of attentional vectors (limit 2 GiB)",
                B * T, (unsigned long long)sco);
  return ONMT_OK;
}

// Unidirectional encoders with fewer rows than this run their layers as a wavefront (see encode_compute).
constexpr int kWavefrontMaxRows = 256;

// The checked ids and lengths (w.src, w.lens) and the first slice of the source embeddings (w.x16).
hipError_t embed(const onmt_model* m, const int32_t* src, const int32_t* len, int B, int S, const EncWs& w, int32_t* err,
                 int32_t* max_len, hipStream_t st) {
  return embed_src(src, len, B, S, m->cfg.src_vocab, m->E_src.w().base, m->d.wterms, m->d.kb(m->d.E), w.src, w.lens,
                   w.x16, w.x16_rows, err, max_len, st);
}

// What the checking kernel found wrong with ids [rows, ld] and their lengths, named by a second look on the host.
int name_violation(const int32_t* ids, const int32_t* len, int rows, int ld, int V, const char* name, const char* lname,
                   hipStream_t st) {
  std::vector<int32_t> hl(rows), hs((size_t)rows * ld);
  HIP_TRY(hipMemcpyAsync(hl.data(), len, sizeof(int32_t) * rows, hipMemcpyDeviceToHost, st));
  HIP_TRY(hipMemcpyAsync(hs.data(), ids, sizeof(int32_t) * hs.size(), hipMemcpyDeviceToHost, st));
  HIP_TRY(hipStreamSynchronize(st));
  for (int b = 0; b < rows; ++b) {
    if (hl[b] < 1 || hl[b] > ld) return fail(ONMT_EINVAL, "%s[%d] = %d outside [1, %d]", lname, b, hl[b], ld);
    for (int s = 0; s < hl[b]; ++s) {
      const int v = hs[(size_t)b * ld + s];
      if (v < 0 || v >= V) return fail(ONMT_EINVAL, "%s[%d, %d] = %d outside [0, %d)", name, b, s, v, V);
    }
  }
  return ONMT_OK;
}

// Source ids and lengths: a kernel checks them and writes the working copies w.src, w.lens and w.x16. Host mode
// (ONMT_VALIDATE_HOST): the call waits for it and refuses bad inputs before any compute is enqueued; the longest
// length bounds the encoder's steps. (Copying the inputs over instead, two pageable copies with their waits, took
// about 40 us more.) Device mode: nothing waits, violations are recorded, and the encoder steps over all S_max
// positions, which the packed padding leaves unchanged past each sentence's length.
int checked_source(onmt_model* m, const int32_t* src, const int32_t* len, int B, int S, const EncWs& w, hipStream_t st,
                   int* max_len, bool host) {
  if (!src || !len) return fail(ONMT_EINVAL, "src/len is NULL");
  if ((long long)B * S > (1LL << 28)) return fail(ONMT_EUNSUPPORTED, "B * S_max too large");
  if (!host) {
    HIP_TRY(embed(m, src, len, B, S, w, m->err_host, nullptr, st));
    *max_len = S;
    return ONMT_OK;
  }
  volatile int32_t* words = m->err_host;
  words[1] = 0;
  HIP_TRY(embed(m, src, len, B, S, w, m->err_host + 1, m->err_host + 2, st));
  HIP_TRY(hipStreamSynchronize(st));
  if (words[1]) {
    const int rc = name_violation(src, len, B, S, m->cfg.src_vocab, "src", "len", st);
    return rc ? rc : fail(ONMT_EINVAL, "invalid src or len");
  }
  *max_len = words[2];
  return ONMT_OK;
}

// Encoder compute on checked inputs in w.src and w.lens (Section 2 encoder RNN; Tables 3-4 bidirectional; readings
// R2-R5). Positions are the outer index of every per-position operand (row s * B + b), so a step reads whole
// fragment blocks of consecutive rows.
int encode_compute(onmt_model* m, int B, int S, int max_len, const EncWs& w, hipStream_t st) {
  const Dims& d = m->d;
  const int BS = B * S, kbm = d.kb(d.Hm), kbd = d.kb(d.Hd);
  const int gxw = d.ndir * 4 * d.Hd_pad;
  const size_t SB = (size_t)B * d.Hd;       // one state slot
  const bool uni = d.ndir == 1, keys = d.attn != ONMT_ATTN_DOT;
  HIP_TRY(fill_f32(w.hs[1], w.zero_n, 0.f, st));
  if (max_len < S) {   // positions no step reaches: memory 0, and 0 as the keys' operand
    HIP_TRY(fill_f32(w.memory, (size_t)BS * d.Hm, 0.f, st));
    if (keys) HIP_TRY(fill_f32((float*)w.y16[(d.L - 1) & 1], split16_bytes(BS, kbm, 2) / 4, 0.f, st));
  }
  HIP_TRY(zero_pad16(w.y16[0], d.L > 1 ? w.y16[1] : nullptr, BS, d.Hm, kbm, st));
  // Recurrent product of (layer l, direction dir) at position s, its step-th step: the state after step k goes to
  // buffer k & 1 and step k reads the other buffer (buffer 1 holds the zero state before step 0); after the last
  // step it goes to the final states.
  // Unidirectional layers >= 1 keep [W_x | W_h] in one matrix: `joint` steps read [y_{l-1} at s | h]
  // against all of it; otherwise the step reads h against the W_h columns and adds the projection gx.
  auto recurrent = [&](int l, int dir, int s, int step, bool joint, ThinA& r, ThinW& wb, LstmParams& lp) {
    const int pin = (step + 1) & 1, slot = l * d.ndir + dir;
    r = ThinA{};
    r.M = B;
    ThinSeg h{w.hs16[pin] + slot * w.hs_plane, nullptr, 0, kbd, (uint32_t)(w.hs_plane * 2)};
    if (joint) {   // [output of layer l-1 at position s | h]
      r.nseg = 2;
      r.seg[0] = ThinSeg{w.y16[(l - 1) & 1], nullptr, s * B, kbm, (uint32_t)split16_bytes(BS, kbm, 2)};
      r.seg[1] = h;
      wb = m->enc_xh[l].w();
    } else {       // h, plus the precomputed input projection
      r.nseg = 1;
      r.seg[0] = h;
      wb = uni && l > 0 ? m->enc_xh[l].w(kbm) : m->enc_h[slot].w();
    }
    lp = LstmParams{};
    lp.bias = joint ? m->enc_bias[l] : nullptr;
    lp.gx = joint ? nullptr : w.gx;
    lp.ld_gx = gxw;
    lp.gx_col0 = dir * 4 * d.Hd_pad;
    lp.gx_S = 1;
    lp.gx_s = s * B;
    lp.c_in = w.cs[pin] + slot * SB;
    lp.ld_c = d.Hd;
    lp.h_in = w.hs[pin] + slot * SB;
    lp.ld_h_in = d.Hd;
    if (step == max_len - 1) {
      const size_t o = (size_t)l * B * d.H + (size_t)dir * d.Hd;
      lp.h_out = w.final_h + o;
      lp.c_out = w.final_c + o;
      lp.ld_out = d.H;
    } else {
      lp.h_out = w.hs[pin ^ 1] + slot * SB;
      lp.c_out = w.cs[pin ^ 1] + slot * SB;
      lp.ld_out = d.Hd;
      lp.h16 = w.hs16[pin ^ 1] + slot * w.hs_plane;
      lp.kb16 = kbd;
    }
    const bool top = l == d.L - 1;
    lp.y_out = top ? w.memory : nullptr;
    lp.ld_y = d.Hm;
    lp.y_S = S;
    lp.y_s = s;
    lp.y_col0 = dir * d.Hd;
    lp.y16 = !top || keys ? w.y16[l & 1] : nullptr;
    lp.y_kb16 = kbm;
    lp.y_r0 = s * B;
    lp.lens = w.lens;
    lp.H = d.Hd;
  };
  auto run_one = [&](int l, int dir, int s, int step, bool joint) -> int {
    ThinA r;
    ThinW wb;
    LstmParams lp;
    recurrent(l, dir, s, step, joint, r, wb, lp);
    HIP_TRY(thin_lstm(d.wterms, r, wb, lp, st));
    return ONMT_OK;
  };
  auto run_two = [&](int l0, int dir0, int s0, int step0, bool joint0, int l1, int dir1, int s1, int step1,
                     bool joint1) -> int {
    ThinPair q{};
    recurrent(l0, dir0, s0, step0, joint0, q.a[0], q.w[0], q.p[0]);
    recurrent(l1, dir1, s1, step1, joint1, q.a[1], q.w[1], q.p[1]);
    HIP_TRY(thin_lstm2(d.wterms, q, st));
    return ONMT_OK;
  };
  auto project = [&](int l) -> int {   // input projection of every position, both directions at once
    const int rows = max_len * B;
    if (l > 0) {   // unidirectional: the W_x columns of the joint matrix
      HIP_TRY(wide_store(WideA{w.y16[(l - 1) & 1], nullptr, nullptr, rows, BS, kbm, 2},
                         uni ? m->enc_xh[l].w() : m->enc_x[l].w(), d.wterms,
                         WideOut{m->enc_bias[l], w.gx, gxw, gxw, 0, 0}, st));
      return ONMT_OK;
    }
    for (int r0 = 0, n; r0 < rows; r0 += n) {   // slice by slice, the first gathered by the checking kernel
      n = rows - r0 < w.x16_rows ? rows - r0 : w.x16_rows;
      if (r0) HIP_TRY(embed_rows(w.src + r0, n, m->E_src.w().base, d.wterms, d.kb(d.E), w.x16, st));
      HIP_TRY(wide_store(WideA{w.x16, w.src + r0, m->E_src.w().wexp, n, w.x16_rows, d.kb(d.E), d.wterms},
                         m->enc_x[0].w(), d.wterms,
                         WideOut{m->enc_bias[0], w.gx + (size_t)r0 * gxw, gxw, gxw, 0, 0}, st));
    }
    return ONMT_OK;
  };
  int rc = ONMT_OK;
  if (uni && B < kWavefrontMaxRows) {
    // few rows per step (launch-bound): layer l processes position s = wave - l, one step behind the
    // layer below, and the layers of one wave go out two per launch
    if ((rc = project(0))) return rc;
    for (int wave = 0; wave < max_len + d.L - 1; ++wave) {
      const int lo = wave - max_len + 1 > 0 ? wave - max_len + 1 : 0;
      const int hi = wave < d.L - 1 ? wave : d.L - 1;
      for (int l = lo; l <= hi; l += 2) {
        const int t0 = wave - l, t1 = wave - l - 1;   // position = step for a forward layer
        rc = l + 1 <= hi ? run_two(l, 0, t0, t0, l > 0, l + 1, 0, t1, t1, true) : run_one(l, 0, t0, t0, l > 0);
        if (rc) return rc;
      }
    }
  } else if (uni) {
    // many rows per step (compute-bound): layer by layer, each with its input projection of every
    // position done as one large GEMM first
    for (int l = 0; l < d.L; ++l) {
      if ((rc = project(l))) return rc;
      for (int step = 0; step < max_len; ++step)
        if ((rc = run_one(l, 0, step, step, false))) return rc;
    }
  } else {
    // both directions of a layer step together, one launch per step
    for (int l = 0; l < d.L; ++l) {
      if ((rc = project(l))) return rc;
      for (int step = 0; step < max_len; ++step)
        if ((rc = run_two(l, 0, step, step, false, l, 1, max_len - 1 - step, step, false))) return rc;
    }
  }
  // attention keys W_a m_s (concat: its memory columns), once per batch; dot scores read the memory
  if (!keys) return ONMT_OK;
  HIP_TRY(wide_store(WideA{w.y16[(d.L - 1) & 1], nullptr, nullptr, BS, BS, kbm, 2}, m->W_a.w(), d.wterms,
                     WideOut{nullptr, w.keys, d.H, d.H, B, S}, st));
  return ONMT_OK;
}

int decode_init_compute(onmt_model* m, const EncWs& w, int B, int K, const State& s, hipStream_t st) {
  HIP_TRY(decode_init(decode_state(m->d, s, B * K), w.final_h, w.final_c, B, K, st));
  return ONMT_OK;
}

// Kernel timing: an event pair around every prof-th launch of each kind (ONMT_KERNEL_*), on the stream the
// kernel is launched on; the pairs are read back by time_collect once the stream has been synchronized.
void time_begin(onmt_model* m, hipStream_t st, int kind = ONMT_KERNEL_GENERATOR) {
  m->prof_open[kind] = false;
  if (!m->prof || !((m->prof_kinds >> kind) & 1u) || (m->prof_seq[kind]++ % m->prof) != 0) return;
  while (m->ev.size() < m->ev_used + 2) {
    hipEvent_t e;
    // timing-only events: no system-scope fence, so recording them does not stall the next kernel
    if (hipEventCreateWithFlags(&e, hipEventDisableSystemFence) != hipSuccess) return;
    m->ev.push_back(e);
  }
  if (m->ev_kind.size() < m->ev.size()) m->ev_kind.resize(m->ev.size());
  hipEventRecord(m->ev[m->ev_used], st);
  m->ev_kind[m->ev_used] = kind;
  m->prof_pair[kind] = m->ev_used;
  m->ev_used += 2;
  m->prof_open[kind] = true;
}
void time_end(onmt_model* m, hipStream_t st, int kind = ONMT_KERNEL_GENERATOR) {
  if (!m->prof_open[kind]) return;
  m->prof_open[kind] = false;
  hipEventRecord(m->ev[m->prof_pair[kind] + 1], st);
}
void time_collect(onmt_model* m) {
  for (size_t i = 0; i + 1 < m->ev_used; i += 2) {
    float ms = 0.f;
    if (hipEventSynchronize(m->ev[i + 1]) == hipSuccess && hipEventElapsedTime(&ms, m->ev[i], m->ev[i + 1]) == hipSuccess) {
      m->prof_ms[m->ev_kind[i]] += ms;
      m->prof_n[m->ev_kind[i]] += 1;
    }
  }
  m->ev_used = 0;
}

// What the merge of a step's generator launch reads.
GenPartials gen_partials(const GenParams& gp) {
  GenPartials q{};
  q.pmax = gp.pmax;
  q.psum = gp.psum;
  q.pval = gp.pval;
  q.pid = gp.pid;
  q.ntiles = gp.ntiles;
  q.logits = gp.logits;
  q.ld_logits = gp.ld_logits;
  q.V = gp.V;
  q.pfmax = gp.pfmax;
  q.banned_bits = gp.banned_bits;
  q.unk_cnt = gp.unk_cnt;
  q.unk_id = gp.unk_id;
  q.max_unk = gp.max_unk;
  return q;
}

// One decoder step on validated inputs (Section 2; Figure 1(a); items (a)-(c); Section 4.2 attention).
// mode 0: logp [N, V] full log-softmax; mode 1: top-K (logp [N, K], ids [N, K]); mode 2 (beam search):
// stop after the generator, leaving its per-tile partials in the step workspace for the beam step;
// mode 3 (teacher forcing): stop after the attentional vector (out.feed), the generator runs later over
// all steps at once.
// Optional work of a decoder step beyond the log-distribution.
struct StepExtras {
  const int32_t* want = nullptr;        // the logit of column want[r] of every row goes to want_logit[r]
  float* want_logit = nullptr;
  const Coverage* cov = nullptr;        // attention coverage and its penalty
  int32_t* align = nullptr;             // attention argmax per row
  const uint32_t* banned_bits = nullptr;   // hypothesis filters of the generator's top-K lists
  const int32_t* unk_cnt = nullptr;
  int unk_id = 0, max_unk = -1;
  float* pfmax = nullptr;
};

int decode_compute(onmt_model* m, const EncWs& w, int B, int S, int K, const State& in, const State& out,
                   const int32_t* prev_tok, const int32_t* parent, int mode, float* logp, int32_t* ids, float* lse,
                   float* attn, const StepWs& sw, hipStream_t st, const StepExtras& ex = StepExtras{},
                   bool timing = true) {
  const Dims& d = m->d;
  const int N = B * K;
  const size_t LH = (size_t)N * d.H;
  const int kb = d.kb(d.H);
  auto rows16 = [&](const uint16_t* base, const int32_t* idx, int row0, int width, int rows) {
    return ThinSeg{base, idx, row0, d.kb(width), (uint32_t)split16_bytes(rows, d.kb(width), 2)};
  };
  for (int l = 0; l < d.L; ++l) {
    ThinA a{};
    a.M = N;
    LstmParams lp{};
    a.nseg = 2;
    if (l == 0) {
      // [feed ; h] against the feed and recurrent columns; the embedding columns' product is the
      // precomputed row of the previous token (emb_gates), added in the epilogue
      a.seg[0] = rows16(in.feed16, parent, in.feed16_r0, d.H, in.feed16_rows ? in.feed16_rows : N);
      lp.gx = m->emb_gates;
      lp.gx_idx = prev_tok;
      lp.gx_rows = d.Vt;
      lp.ld_gx = 4 * d.H_pad;
    } else {
      a.seg[0] = rows16(out.h16 + (l - 1) * out.plane, nullptr, 0, d.H, N);
    }
    a.seg[1] = rows16(in.h16 + l * in.plane, parent, 0, d.H, N);
    lp.bias = m->dec_bias[l];
    lp.c_in = in.c + l * LH;
    lp.c_idx = parent;
    lp.ld_c = d.H;
    lp.h_out = out.h + l * LH;
    lp.c_out = out.c + l * LH;
    lp.ld_out = d.H;
    lp.H = d.H;
    lp.h16 = out.h16 + l * out.plane;
    lp.kb16 = kb;
    if (in.shift) {   // the next layer's product takes this one's output beside its own row of `in`
      lp.in_shift = in.shift + (size_t)l * N;
      if (l + 1 < d.L) lp.out_shift = in.shift + (size_t)(l + 1) * N;
    }
    if (timing) time_begin(m, st, ONMT_KERNEL_LSTM);
    HIP_TRY(thin_lstm(d.wterms, a, m->dec_t[l].w(), lp, st));
    if (timing) time_end(m, st, ONMT_KERNEL_LSTM);
  }
  const ThinSeg q16 = rows16(out.h16 + (d.L - 1) * out.plane, nullptr, 0, d.H, N);
  const float* q = out.h + (d.L - 1) * LH;
  const float* sq = q;
  if (d.attn == ONMT_ATTN_CONCAT) {   // the query side of concat's tanh argument, W_q q
    ThinA a{};
    a.M = N;
    a.nseg = 1;
    a.seg[0] = q16;
    StoreParams sp{};
    sp.out = sw.qproj;
    sp.ldo = sp.ncols = d.H;
    HIP_TRY(thin_store(d.wterms, a, m->W_q.w(), sp, st));
    sq = sw.qproj;
  }
  const AttnExtra ax{ex.cov, ex.align};
  if (timing) time_begin(m, st, ONMT_KERNEL_ATTENTION);
  HIP_TRY(attention(sq, d.H, w.keys, m->v_a, w.memory, w.lens, B, S, d.H, d.Hm, K, sw.scores, sw.ctx16, attn, ax,
                    st));
  if (timing) time_end(m, st, ONMT_KERNEL_ATTENTION);
  {
    ThinA a{};
    a.M = N;
    a.nseg = 2;
    a.seg[0] = rows16(sw.ctx16, nullptr, 0, d.Hm, N);
    a.seg[1] = q16;
    StoreParams sp{};
    sp.out = out.feed;
    sp.ldo = sp.ncols = d.H;
    sp.act = 1;
    sp.s16 = out.feed16;             // the operand of the generator and of the next step's first layer
    sp.r0_16 = out.feed16_r0;
    sp.kb16 = kb;
    if (timing) time_begin(m, st, ONMT_KERNEL_OUTPUT);
    HIP_TRY(thin_store(d.wterms, a, m->W_c.w(), sp, st));
    if (timing) time_end(m, st, ONMT_KERNEL_OUTPUT);
  }
  if (mode == 3) return ONMT_OK;
  GenPartials part{};
  {
    GenParams gp{};
    gp.bias = m->b_s;
    gp.wexp = m->W_s_exp;
    gp.V = d.Vt;
    gp.K = K;
    gp.ntiles = sw.ntiles;
    gp.pmax = sw.pmax;
    gp.psum = sw.psum;
    gp.logits = mode == 0 ? logp : sw.logits;
    gp.ld_logits = mode == 0 ? d.Vt : sw.ld_logits;
    gp.pval = mode == 0 ? nullptr : sw.pval;
    gp.pid = sw.pid;
    gp.want = ex.want;
    gp.want_logit = ex.want_logit;
    gp.banned_bits = ex.banned_bits;
    gp.unk_cnt = ex.unk_cnt;
    gp.unk_id = ex.unk_id;
    gp.max_unk = ex.max_unk;
    gp.pfmax = ex.pfmax;
    part = gen_partials(gp);
    if (timing) time_begin(m, st);
    HIP_TRY(gemm_gen(Split16{out.feed16, N, d.kb(d.H)}, m->W_s, d.wterms, gp, st));
    if (timing) time_end(m, st);
  }
  if (mode == 2) return ONMT_OK;
  float* lse_out = lse ? lse : sw.lse;
  if (mode == 0) {
    HIP_TRY(log_probs(logp, d.Vt, part, N, lse_out, st));
  } else {
    HIP_TRY(lse_topk_merge(part, N, K, logp, ids, lse_out, st));
  }
  return ONMT_OK;
}

int check_beam(const onmt_model* m, int S, int K) {
  if (K < 1 || K > kMaxBeam) return fail(ONMT_EUNSUPPORTED, "beam %d outside [1, %d]", K, kMaxBeam);
  if (K > m->cfg.tgt_vocab) return fail(ONMT_EINVAL, "beam %d larger than the vocabulary", K);
  if (m->d.H > 1024) return fail(ONMT_EUNSUPPORTED, "attention supports hidden <= 1024");
  if (attention_lds_bytes(S, m->d.H, K) > 64 * 1024)
    return fail(ONMT_EUNSUPPORTED, "beam * max(hidden, S_max) too large for the attention workgroups");
  return ONMT_OK;
}

}  // namespace

extern "C" {

size_t onmt_encode_ws_bytes(const onmt_model* m, int B, int S) {
  if (!m || B < 1 || S < 1) return 0;
  return enc_layout(m->d, B, S, nullptr, nullptr);
}

int onmt_encode(onmt_model* m, const int32_t* src, const int32_t* len, int B, int S, void* ws, size_t ws_bytes,
                void* stream) {
  if (!m) return fail(ONMT_EINVAL, "model is NULL");
  if (!ws) return fail(ONMT_EINVAL, "enc_ws is NULL");
  hipStream_t st = (hipStream_t)stream;
  if (B < 1 || S < 1) return fail(ONMT_EINVAL, "B and S_max must be >= 1");
  int rc = check_ws_limits(m->d, B, S, 1, 0);
  if (rc) return rc;
  if (ws_bytes < enc_layout(m->d, B, S, nullptr, nullptr)) return fail(ONMT_ESIZE, "encoder workspace too small");
  EncWs w;
  enc_layout(m->d, B, S, (char*)ws, &w);
  int mx = 0;
  rc = checked_source(m, src, len, B, S, w, st, &mx, m->validation == ONMT_VALIDATE_HOST);
  if (rc) return rc;
  return encode_compute(m, B, S, mx, w, st);
}

size_t onmt_state_bytes(const onmt_model* m, int N) {
  if (!m || N < 1) return 0;
  return state_layout(m->d, N, nullptr, nullptr);
}

size_t onmt_step_ws_bytes(const onmt_model* m, int B, int S, int K) {
  if (!m || B < 1 || S < 1 || K < 1) return 0;
  return step_layout(m->d, B, S, K, nullptr, nullptr);
}

int onmt_decode_init(onmt_model* m, const void* enc_ws, int B, int S, int K, void* state_out, void* stream) {
  if (!m || !enc_ws || !state_out) return fail(ONMT_EINVAL, "NULL argument");
  if (B < 1 || S < 1 || K < 1) return fail(ONMT_EINVAL, "B, S_max, K must be >= 1");
  int rc = check_ws_limits(m->d, B, S, K, 0);
  if (rc) return rc;
  EncWs w;
  enc_layout(m->d, B, S, (char*)enc_ws, &w);
  State s;
  state_layout(m->d, B * K, (char*)state_out, &s);
  return decode_init_compute(m, w, B, K, s, (hipStream_t)stream);
}

int onmt_decode_step(onmt_model* m, const void* enc_ws, int B, int S, int K, const void* state_in, void* state_out,
                     const int32_t* prev_tok, const int32_t* parent, int mode, float* logp, int32_t* ids, float* lse,
                     float* attn, void* step_ws, size_t step_ws_bytes, void* stream) {
  if (!m || !enc_ws || !state_in || !state_out || !prev_tok || !logp || !step_ws) return fail(ONMT_EINVAL, "NULL argument");
  if (state_in == state_out) return fail(ONMT_EINVAL, "state_in and state_out must differ");
  if (B < 1 || S < 1) return fail(ONMT_EINVAL, "B and S_max must be >= 1");
  int rc = check_beam(m, S, K);
  if (rc) return rc;
  if ((rc = check_ws_limits(m->d, B, S, K, 0))) return rc;
  if (mode != 0 && mode != 1) return fail(ONMT_EINVAL, "mode must be 0 (full) or 1 (top-K)");
  if (mode == 1 && !ids) return fail(ONMT_EINVAL, "ids is NULL in top-K mode");
  if (step_ws_bytes < step_layout(m->d, B, S, K, nullptr, nullptr)) return fail(ONMT_ESIZE, "step workspace too small");
  hipStream_t st = (hipStream_t)stream;
  const int N = B * K;
  StepWs sw;
  step_layout(m->d, B, S, K, (char*)step_ws, &sw);
  State si, so;
  state_layout(m->d, N, (char*)state_in, &si);
  state_layout(m->d, N, (char*)state_out, &so);
  si = step_input(m->d, si, so);
  const bool host = m->validation == ONMT_VALIDATE_HOST;
  volatile int32_t* words = m->err_host;
  if (host) words[1] = 0;
  HIP_TRY(prepare_step(decode_state(m->d, si, N), split_state(m->d), prev_tok, parent, m->cfg.tgt_vocab, sw.tok_s,
                       sw.par_s, m->err_host + (host ? 1 : 0), st));
  if (host) {
    HIP_TRY(hipStreamSynchronize(st));
    if (words[1]) {                     // name the value with a second look on the host
      std::vector<int32_t> ht(N), hp(parent ? N : 0);
      HIP_TRY(hipMemcpyAsync(ht.data(), prev_tok, sizeof(int32_t) * N, hipMemcpyDeviceToHost, st));
      if (parent) HIP_TRY(hipMemcpyAsync(hp.data(), parent, sizeof(int32_t) * N, hipMemcpyDeviceToHost, st));
      HIP_TRY(hipStreamSynchronize(st));
      for (int r = 0; r < N; ++r) {
        if (ht[r] < 0 || ht[r] >= m->cfg.tgt_vocab) return fail(ONMT_EINVAL, "prev_tok[%d] = %d out of range", r, ht[r]);
        if (parent && (hp[r] < 0 || hp[r] >= N)) return fail(ONMT_EINVAL, "parent[%d] = %d out of range", r, hp[r]);
      }
      return fail(ONMT_EINVAL, "invalid prev_tok or parent");
    }
  }
  prev_tok = sw.tok_s;
  parent = parent ? sw.par_s : nullptr;
  EncWs w;
  enc_layout(m->d, B, S, (char*)enc_ws, &w);
  rc = decode_compute(m, w, B, S, K, si, so, prev_tok, parent, mode, logp, ids, lse, attn, sw, st);
  if (m->prof) {
    HIP_TRY(hipStreamSynchronize(st));
    time_collect(m);
  }
  return rc;
}

int onmt_set_validation(onmt_model* m, int mode) {
  if (!m) return fail(ONMT_EINVAL, "model is NULL");
  if (mode != ONMT_VALIDATE_HOST && mode != ONMT_VALIDATE_DEVICE)
    return fail(ONMT_EINVAL, "validation mode must be ONMT_VALIDATE_HOST or ONMT_VALIDATE_DEVICE");
  m->validation = mode;
  return ONMT_OK;
}

int onmt_decode_step_noalloc(onmt_model* m, const void* enc_ws, int B, int S, int K, const void* state_in,
                             void* state_out, const int32_t* prev_tok, const int32_t* parent, int mode, float* logp,
                             int32_t* ids, float* lse, float* attn, void* stream) {
  if (!m || !enc_ws || !state_in || !state_out || !prev_tok || !logp) return fail(ONMT_EINVAL, "NULL argument");
  if (state_in == state_out) return fail(ONMT_EINVAL, "state_in and state_out must differ");
  if (B < 1 || S < 1) return fail(ONMT_EINVAL, "B and S_max must be >= 1");
  int rc = check_beam(m, S, K);
  if (rc) return rc;
  if ((rc = check_ws_limits(m->d, B, S, K, 0))) return rc;
  if (mode != 0 && mode != 1) return fail(ONMT_EINVAL, "mode must be 0 (full) or 1 (top-K)");
  if (mode == 1 && !ids) return fail(ONMT_EINVAL, "ids is NULL in top-K mode");
  const size_t bytes = step_layout(m->d, B, S, K, nullptr, nullptr, true), rows = (size_t)B * K;
  const size_t need = bytes - align_up(split16_bytes(rows, m->d.kb(m->d.Hm), 2)) +
                      align_up(rows * m->d.Hm * sizeof(float)) + 2 * align_up(rows * K * sizeof(float));
  if (need > ONMT_NOALLOC_SCRATCH_BYTES || bytes > kScratchBytes)
    return fail(ONMT_EUNSUPPORTED, "this step needs %zu bytes of scratch, more than the %u of the allocation-free call",
                need, (unsigned)ONMT_NOALLOC_SCRATCH_BYTES);
  void* sp = nullptr;
  if ((rc = noalloc_scratch(&sp))) return rc;
  hipStream_t st = (hipStream_t)stream;
  const int N = B * K;
  StepWs sw;
  step_layout(m->d, B, S, K, (char*)sp, &sw, true);
  EncWs w;
  enc_layout(m->d, B, S, (char*)enc_ws, &w);
  State si, so;
  state_layout(m->d, N, (char*)state_in, &si);
  state_layout(m->d, N, (char*)state_out, &so);
  si = step_input(m->d, si, so);
  HIP_TRY(prepare_step(decode_state(m->d, si, N), split_state(m->d), prev_tok, parent, m->cfg.tgt_vocab, sw.tok_s,
                       sw.par_s, m->err_host, st));
  return decode_compute(m, w, B, S, K, si, so, sw.tok_s, parent ? sw.par_s : nullptr, mode, logp, ids, lse, attn, sw,
                        st, StepExtras{}, false);
}

int onmt_device_status(onmt_model* m, int* code) {
  if (!m || !code) return fail(ONMT_EINVAL, "NULL argument");
  volatile int32_t* e = m->err_host;
  const int32_t kind = *e;
  *e = 0;
  *code = kind ? ONMT_EINVAL : ONMT_OK;
  if (kind) {
    static const char* what[] = {"", "a source length outside [1, S_max]", "a source id outside [0, src_vocab)",
                                 "a previous token outside [0, tgt_vocab)", "a parent row outside [0, B * beam)"};
    fail(ONMT_EINVAL, "device validation found %s (replaced by a safe value)", kind >= 1 && kind <= 4 ? what[kind] : "an invalid input");
  }
  return ONMT_OK;
}

size_t onmt_search_ws_bytes(const onmt_model* m, int B, int S, const onmt_search_params* p) {
  if (!m || !p || B < 1 || S < 1 || p->beam < 1 || p->max_len < 1) return 0;
  return search_layout(m->d, B, S, p->beam, p->max_len, nullptr, nullptr);
}

int onmt_beam_search(onmt_model* m, const int32_t* src, const int32_t* len, int B, int S,
                     const onmt_search_params* prm, void* ws, size_t ws_bytes, int32_t* out_tok, int32_t* out_len,
                     double* out_raw, double* out_norm, float* out_tok_logp, int32_t* out_align,
                     const onmt_trace* trace, void* stream) {
  if (!m || !prm || !ws) return fail(ONMT_EINVAL, "NULL argument");
  if (!out_tok || !out_len || !out_raw || !out_norm) return fail(ONMT_EINVAL, "NULL output pointer");
  const int K = prm->beam, T = prm->max_len;
  if (T < 1 || T > 100000) return fail(ONMT_EINVAL, "max_len %d outside [1, 100000]", T);
  if (!(prm->alpha >= 0.0) || !std::isfinite(prm->alpha)) return fail(ONMT_EINVAL, "alpha must be finite and >= 0");
  if (!(prm->beta >= 0.0) || !std::isfinite(prm->beta)) return fail(ONMT_EINVAL, "beta must be finite and >= 0");
  if (prm->n_banned < 0 || (prm->n_banned > 0 && !prm->banned)) return fail(ONMT_EINVAL, "banned list invalid");
  for (int i = 0; i < prm->n_banned; ++i)
    if (prm->banned[i] < 0 || prm->banned[i] >= m->cfg.tgt_vocab)
      return fail(ONMT_EINVAL, "banned[%d] = %d outside [0, %d)", i, prm->banned[i], m->cfg.tgt_vocab);
  if (trace && (!trace->slot || !trace->tok || !trace->cand || !trace->steps))
    return fail(ONMT_EINVAL, "trace given with a NULL array");
  if (B < 1 || S < 1) return fail(ONMT_EINVAL, "B and S_max must be >= 1");
  int rc = check_beam(m, S, K);
  if (rc) return rc;
  if ((rc = check_ws_limits(m->d, B, S, K, 0))) return rc;
  if (ws_bytes < search_layout(m->d, B, S, K, T, nullptr, nullptr)) return fail(ONMT_ESIZE, "search workspace too small");
  hipStream_t st = (hipStream_t)stream;
  SearchWs w;
  search_layout(m->d, B, S, K, T, (char*)ws, &w);
  int mx = 0;
  rc = checked_source(m, src, len, B, S, w.enc, st, &mx, m->validation == ONMT_VALIDATE_HOST);
  if (rc) return rc;

  BeamParams bp = w.bp;
  bp.B = B;
  bp.K = K;
  bp.V = m->cfg.tgt_vocab;
  bp.T_max = T;
  bp.eos = m->cfg.eos_id;
  bp.pad = m->cfg.pad_id;
  bp.alpha = prm->alpha;
  bp.lp_tmax = std::pow((5.0 + T) / 6.0, prm->alpha);
  bp.tr_slot = trace ? trace->slot : nullptr;
  bp.tr_tok = trace ? trace->tok : nullptr;
  bp.tr_cand = trace ? trace->cand : nullptr;

  GenPartials gp{};
  gp.pmax = w.step.pmax;
  gp.psum = w.step.psum;
  gp.ntiles = w.step.ntiles;
  gp.logits = w.step.logits;
  gp.pval = w.step.pval;
  gp.pid = w.step.pid;
  gp.ld_logits = w.step.ld_logits;
  gp.V = m->cfg.tgt_vocab;
  rc = encode_compute(m, B, S, mx, w.enc, st);
  if (rc) return rc;
  rc = decode_init_compute(m, w.enc, B, K, w.st[0], st);
  if (rc) return rc;
  const bool coverage = prm->beta > 0.0;
  bp.cp = coverage ? w.cp : nullptr;
  const bool filtering = prm->n_banned > 0 || prm->max_unk >= 0;
  bp.unk_cnt = filtering ? bp.unk_cnt : nullptr;
  bp.unk_id = m->cfg.unk_id;
  bp.align = out_align ? w.step.align : nullptr;
  std::vector<uint32_t> bits;
  if (prm->n_banned > 0) {
    bits.assign((size_t)(m->cfg.tgt_vocab + 31) / 32, 0u);
    for (int i = 0; i < prm->n_banned; ++i) bits[prm->banned[i] >> 5] |= 1u << (prm->banned[i] & 31);
    HIP_TRY(hipMemcpyAsync(w.banned_bits, bits.data(), bits.size() * sizeof(uint32_t), hipMemcpyHostToDevice, st));
  }
  StepExtras ex;
  ex.align = bp.align ? w.step.align : nullptr;
  if (filtering) {
    ex.banned_bits = prm->n_banned > 0 ? w.banned_bits : nullptr;
    ex.unk_cnt = prm->max_unk >= 0 ? bp.unk_cnt : nullptr;
    ex.unk_id = m->cfg.unk_id;
    ex.max_unk = prm->max_unk;
    ex.pfmax = w.step.pfmax;
    gp.pfmax = w.step.pfmax;
    gp.banned_bits = ex.banned_bits;
    gp.unk_cnt = ex.unk_cnt;
    gp.unk_id = ex.unk_id;
    gp.max_unk = ex.max_unk;
  }
  HIP_TRY(beam_init(bp, m->cfg.bos_id, st));
  if (coverage) HIP_TRY(fill_f32(w.cov[0], (size_t)B * K * S, 0.f, st));
  const int every = prm->check_every > 0 ? prm->check_every : (T <= 32 ? 1 : 8);
  if (!m->done_host) {
    HIP_TRY(hipHostMalloc((void**)&m->done_host, 2 * sizeof(int32_t), hipHostMallocDefault));
    for (auto& e : m->done_ev) HIP_TRY(hipEventCreateWithFlags(&e, hipEventDisableTiming));
  } else {
    // a search that returned early on an error may have left a count copy queued (possibly on another
    // stream): it must land before this search's copies reuse the two slots
    for (auto& e : m->done_ev) HIP_TRY(hipEventSynchronize(e));
  }
  int cur = 0, nchk = 0;
  for (int t = 1; t <= T; ++t) {
    // coverage of the rows' hypotheses: the parents' coverage (previous layout) plus this step's weights
    const Coverage cv{w.cov[cur], w.cov[cur ^ 1], bp.parent, prm->beta, w.cp};
    ex.cov = coverage ? &cv : nullptr;
    rc = decode_compute(m, w.enc, B, S, K, w.st[cur], w.st[cur ^ 1], bp.tok, bp.parent, 2, nullptr, nullptr,
                        nullptr, nullptr, w.step, st, ex);
    if (rc) return rc;
    time_begin(m, st, ONMT_KERNEL_BEAM);
    HIP_TRY(beam_step(bp, gp, t, st));
    time_end(m, st, ONMT_KERNEL_BEAM);
    cur ^= 1;
    if (t < T && t % every == 0) {
      // this step's done count goes to the host asynchronously and the host waits only for the previous
      // check's, so a check period of steps stays queued on the device; a finished batch runs at most one
      // extra period, in which the beam step leaves every finished sentence unchanged
      const int slot = nchk & 1;
      HIP_TRY(hipMemcpyAsync(m->done_host + slot, bp.done_count, sizeof(int32_t), hipMemcpyDeviceToHost, st));
      HIP_TRY(hipEventRecord(m->done_ev[slot], st));
      if (nchk++ > 0) {
        HIP_TRY(hipEventSynchronize(m->done_ev[slot ^ 1]));
        if (m->done_host[slot ^ 1] >= B) break;
      }
    }
  }
  HIP_TRY(backtrack(bp, out_tok, out_len, out_raw, out_norm, out_tok_logp, out_align, st));
  if (trace) HIP_TRY(hipMemcpyAsync(trace->steps, bp.steps, sizeof(int32_t) * B, hipMemcpyDeviceToDevice, st));
  HIP_TRY(hipStreamSynchronize(st));
  if (m->prof) time_collect(m);
  return ONMT_OK;
}

int onmt_replace_unk(onmt_model* m, const int32_t* src, int B, int S, const int32_t* out_tok, const int32_t* out_len,
                     const int32_t* out_align, int T, int32_t* out_src, void* stream) {
  if (!m || !src || !out_tok || !out_len || !out_align || !out_src) return fail(ONMT_EINVAL, "NULL argument");
  if (B < 1 || S < 1 || T < 1) return fail(ONMT_EINVAL, "B, S_max and max_len must be >= 1");
  if ((long long)B * T > (1LL << 30) || (long long)B * S > (1LL << 30)) return fail(ONMT_EUNSUPPORTED, "batch too large");
  HIP_TRY(replace_unk(src, B, S, out_tok, out_len, out_align, T, m->cfg.unk_id, out_src, (hipStream_t)stream));
  return ONMT_OK;
}

size_t onmt_score_ws_bytes(const onmt_model* m, int B, int S, int T) {
  if (!m || B < 1 || S < 1 || T < 1) return 0;
  return score_layout(m->d, B, S, T, nullptr, nullptr);
}

int onmt_score(onmt_model* m, const int32_t* src, const int32_t* len, int B, int S, const int32_t* tgt,
               const int32_t* tgt_len, int T, void* ws, size_t ws_bytes, float* out_logp, double* out_nll,
               void* stream) {
  if (!m || !ws || !tgt || !tgt_len) return fail(ONMT_EINVAL, "NULL argument");
  if (!out_logp || !out_nll) return fail(ONMT_EINVAL, "NULL output pointer");
  if (B < 1 || S < 1) return fail(ONMT_EINVAL, "B and S_max must be >= 1");
  if (T < 1 || T > 100000) return fail(ONMT_EINVAL, "T_max %d outside [1, 100000]", T);
  int rc = check_beam(m, S, 1);
  if (rc) return rc;
  if ((rc = check_ws_limits(m->d, B, S, 1, T))) return rc;
  if (ws_bytes < score_layout(m->d, B, S, T, nullptr, nullptr)) return fail(ONMT_ESIZE, "score workspace too small");
  hipStream_t st = (hipStream_t)stream;
  ScoreWs w;
  score_layout(m->d, B, S, T, (char*)ws, &w);
  int mx = 0;
  // sources and targets checked by kernels that also lay them out; the call waits once for both
  if (!src || !len) return fail(ONMT_EINVAL, "src/len is NULL");
  if ((long long)B * S > (1LL << 28)) return fail(ONMT_EUNSUPPORTED, "B * S_max too large");
  volatile int32_t* words = m->err_host;
  words[1] = 0;
  HIP_TRY(embed(m, src, len, B, S, w.enc, m->err_host + 1, m->err_host + 2, st));
  HIP_TRY(targets(tgt, tgt_len, B, T, m->cfg.tgt_vocab, m->cfg.bos_id, m->cfg.pad_id, w.in_tok, w.want, w.tlen,
                  m->err_host + 1, m->err_host + 3, st));
  HIP_TRY(hipStreamSynchronize(st));
  if (words[1]) {
    if ((rc = name_violation(src, len, B, S, m->cfg.src_vocab, "src", "len", st))) return rc;
    if ((rc = name_violation(tgt, tgt_len, B, T, m->cfg.tgt_vocab, "tgt", "tgt_len", st))) return rc;
    return fail(ONMT_EINVAL, "invalid src, len, tgt or tgt_len");
  }
  mx = words[2];
  const int steps = words[3];
  rc = encode_compute(m, B, S, mx, w.enc, st);
  if (rc) return rc;
  rc = decode_init_compute(m, w.enc, B, 1, w.st[0], st);
  if (rc) return rc;
  HIP_TRY(fill_f32(out_logp, (size_t)B * T, 0.f, st));
  // the recurrence step by step (input feeding makes each step depend on the previous attentional
  // vector); every step's attentional vector is kept for the generator
  const Dims& d = m->d;
  int cur = 0;
  for (int t = 0; t < steps; ++t) {
    State in = w.st[cur], out = w.st[cur ^ 1];
    if (t > 0) {
      in.feed = w.feeds + (size_t)(t - 1) * B * d.H;
      in.feed16 = w.feeds16;
      in.feed16_r0 = (t - 1) * B;
      in.feed16_rows = T * B;
    }
    out.feed = w.feeds + (size_t)t * B * d.H;
    out.feed16 = w.feeds16;
    out.feed16_r0 = t * B;
    out.feed16_rows = T * B;
    rc = decode_compute(m, w.enc, B, S, 1, in, out, w.in_tok + (size_t)t * B, nullptr, 3, nullptr, nullptr, nullptr,
                        nullptr, w.step, st);
    if (rc) return rc;
    cur ^= 1;
  }
  // one generator pass over the steps * B rows: per-tile max and sum of exponentials, and the target's logit
  {
    const int M = steps * B;
    GenParams gp{};
    gp.bias = m->b_s;
    gp.wexp = m->W_s_exp;
    gp.V = d.Vt;
    gp.K = 0;
    gp.ntiles = w.step.ntiles;
    gp.pmax = w.gpmax;
    gp.psum = w.gpsum;
    gp.want = w.want;
    gp.want_logit = w.want_logit;
    time_begin(m, st);
    HIP_TRY(gemm_gen(Split16{w.feeds16, M, d.kb(d.H)}, m->W_s, d.wterms, gp, st));
    time_end(m, st);
    HIP_TRY(score_rows(w.gpmax, w.gpsum, w.step.ntiles, w.want_logit, w.tlen, B, steps, out_logp, T, w.nll, st));
  }
  HIP_TRY(hipMemcpyAsync(out_nll, w.nll, sizeof(double) * B, hipMemcpyDeviceToDevice, st));
  HIP_TRY(hipStreamSynchronize(st));
  if (m->prof) time_collect(m);
  return ONMT_OK;
}

int onmt_profile_enable(onmt_model* m, int every, unsigned kinds) {
  if (!m) return fail(ONMT_EINVAL, "model is NULL");
  if (every < 0) return fail(ONMT_EINVAL, "timing period must be >= 0");
  if (kinds & ~(unsigned)ONMT_KERNEL_ALL) return fail(ONMT_EINVAL, "kernel kind mask 0x%x unknown", kinds);
  m->prof = every;
  m->prof_kinds = kinds;
  for (auto& q : m->prof_seq) q = 0;
  return ONMT_OK;
}

int onmt_profile_read_kernel(onmt_model* m, int kind, int* n, double* ms, int reset) {
  if (!m || !n || !ms) return fail(ONMT_EINVAL, "NULL argument");
  if (kind < 0 || kind >= ONMT_KERNEL_KINDS) return fail(ONMT_EINVAL, "kernel kind %d unknown", kind);
  *n = m->prof_n[kind];
  *ms = m->prof_ms[kind];
  if (reset) {
    m->prof_n[kind] = 0;
    m->prof_ms[kind] = 0.0;
  }
  return ONMT_OK;
}

int onmt_profile_read(onmt_model* m, int* n, double* ms, int reset) {
  return onmt_profile_read_kernel(m, ONMT_KERNEL_GENERATOR, n, ms, reset);
}

}  // extern "C"
