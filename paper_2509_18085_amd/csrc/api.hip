// C ABI of the verification library: argument checks, workspace carving, kernel selection by
// shape, launch order.  No kernel lives here.  Every check runs before the first launch.
#include <cmath>
#include <cstring>

#include <mutex>

#include "kernels.h"

using namespace spiffy;

// Scratch of the allocation-free entry point (spiffy_decode_head_static): every GPU the library runs on holds its own
// copy of this array until the process ends.  In host code the name is only a handle for hipGetSymbolAddress; kernels
// get the device address that call returns.
// Beside the scratch proper it has room for the vocabulary summaries of the heads off the matrix-core path.
constexpr int kTileHeadParts = 512;     // two rounds of one workgroup a CU
constexpr size_t kStaticSummaryBytes = sizeof(TopPartial) * kTileHeadParts * SPIFFY_STATIC_MAX_ROWS;
static __device__ __align__(256) unsigned char scratch[SPIFFY_STATIC_SCRATCH_BYTES + kStaticSummaryBytes];
static_assert(SPIFFY_STATIC_MAX_ROWS % 128 == 0, "rows of a summary array come in groups of 128");

namespace {

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline size_t esize(int dtype) { return dtype == SPIFFY_F32 ? 4 : 2; }

int check_cfg(const spiffy_model_cfg* c) {
  if (!c) return SPIFFY_EINVAL;
  if (c->dtype != SPIFFY_BF16 && c->dtype != SPIFFY_F32) return SPIFFY_EINVAL;
  if (c->d < 8 || c->n_q_heads < 1 || c->n_kv_heads < 1 || c->head_dim < 2 || c->ffn < 8 || c->vocab < 2)
    return SPIFFY_EINVAL;
  if (c->mask_id < 0 || c->mask_id >= c->vocab) return SPIFFY_EINVAL;
  if (!(c->rms_eps >= 0.f) || !(c->rope_base > 0.f)) return SPIFFY_EINVAL;
  if (c->n_q_heads % c->n_kv_heads != 0) return SPIFFY_ESHAPE;
  if (c->head_dim % 8 != 0 || c->head_dim > 256) return SPIFFY_ESHAPE;
  if (c->d % 8 != 0 || c->ffn % 8 != 0) return SPIFFY_ESHAPE;
  return SPIFFY_OK;
}

int check_gb(int32_t G, int32_t B) {
  if (G < 1 || B < 1) return SPIFFY_EINVAL;
  if ((int64_t)G * B > SPIFFY_MAX_ROWS) return SPIFFY_ESHAPE;
  return SPIFFY_OK;
}

bool layer_mfma(const spiffy_model_cfg* c) {
  if (c->dtype != SPIFFY_BF16 || c->head_dim != 128) return false;
  return c->d % 128 == 0 && c->ffn % 64 == 0;
}
bool head_mfma(const spiffy_model_cfg* c) {
  if (c->dtype != SPIFFY_BF16) return false;
  return c->d % 64 == 0;
}

// Limits of the MFMA LM head: per-lane byte offsets into the vocabulary matrix and into the gathered rows are 32-bit,
// and the top-K refinement holds at most 2048 per-chunk summaries of a row (V <= 262144).
bool head_shape_ok(const spiffy_model_cfg* c) {
  if (!head_mfma(c)) return true;
  const size_t lim = (size_t)1 << 32;
  if ((size_t)c->vocab * c->d * 2 >= lim || (size_t)SPIFFY_MAX_ROWS * c->d * 2 >= lim) return false;
  return mfma_lmhead_partials_per_row(c->vocab) <= 2048;
}

// Limit on the block and the cached rows of the shapes without the MFMA attention.  Its kernel keeps neither scores nor
// angles of a whole row and would take more; the limit is what callers of these shapes have been refused so far.
size_t attn_limit_bytes(const spiffy_model_cfg* c, int B, int P) {
  const int hd = c->head_dim;
  const int nchunk = 256 / hd > 0 ? 256 / hd : 1;
  return sizeof(float) * ((size_t)hd + (size_t)B * hd + (size_t)(P + B) + (size_t)nchunk * hd);
}
constexpr size_t kAttnLimitBytes = 150 * 1024;

struct Carve {
  unsigned char* base;
  size_t off;
  explicit Carve(void* p) : base(reinterpret_cast<unsigned char*>(p)), off(0) {}
  void* take(size_t bytes) {
    void* r = base ? base + off : nullptr;
    off += align_up(bytes, 256);
    return r;
  }
};

struct LayerWs {
  void *n, *qkv, *attn, *h, *act;
  void *rope;                    // rotary table: B rows, then S_seq rows
  void *attn_partial, *attn_partial_seq, *splitk;
  void *gat_attn, *gat_x;        // last layer, masked rows only: gathered attention rows and residual rows
  int32_t *rows, *count;         // ... and their row list
  size_t bytes;
};
// P = cached rows (prefix and suffix together).  S_seq > 0: full-sequence step, S_seq true suffix rows ride along
// after the G*B block rows and have an attention scratch of their own (queries over the P + B + S_seq cache rows).
LayerWs carve_layer(const spiffy_model_cfg* c, int G, int B, int P, void* base, int S_seq = 0) {
  const size_t M = (size_t)G * B + S_seq, es = esize(c->dtype);
  const size_t qkv_cols = (size_t)(c->n_q_heads + 2 * c->n_kv_heads) * c->head_dim;
  Carve cv(base);
  LayerWs w;
  w.n = cv.take(M * c->d * es);          // first: the steps' embedding kernel leaves the first layer's input here
  w.qkv = cv.take(M * qkv_cols * es);
  w.attn = cv.take(M * (size_t)c->n_q_heads * c->head_dim * es);
  w.h = cv.take(M * c->d * es);
  w.act = cv.take(M * c->ffn * es);
  w.rope = cv.take(sizeof(float2) * (size_t)(B + S_seq) * (c->head_dim / 2));
  w.rows = (int32_t*)cv.take(sizeof(int32_t) * M);       // in front of everything whose size depends on P: the step's first
  w.count = (int32_t*)cv.take(sizeof(int32_t) * 4);      // kernel fills the table and the list for all layers
  w.attn_partial = cv.take(layer_mfma(c) ? mfma_attn_partial_bytes(G, B, c->n_q_heads, c->head_dim, P + S_seq) : 0);
  w.attn_partial_seq = cv.take(layer_mfma(c) && S_seq ? mfma_attn_partial_bytes(1, S_seq, c->n_q_heads, c->head_dim, P + B + S_seq) : 0);
  w.splitk = cv.take(layer_mfma(c) ? sizeof(float) * 4 * M * c->d : 0);   // up to 4 K slices of [M,d] fp32
  w.gat_attn = cv.take(M * (size_t)c->n_q_heads * c->head_dim * es);
  w.gat_x = cv.take(M * c->d * es);
  w.bytes = cv.off;
  return w;
}

struct HeadWs {
  int32_t *row_idx, *count;
  void* nf;
  TopPartial *part, *part2, *row_top;
  float *logits, *cand_val;           // top-K of a node: with summaries the logits of each position's best chunks, else candidates
  int32_t *chunk_id, *cand_idx;
  int m_cap;
  int n_part;            // MFMA head: summaries of 128 tokens each (the top-K refinement reads them); otherwise 0
  int n_part_tile;       // head of the other shapes: parts of the vocabulary
  size_t tile_summary_bytes, bytes;      // what their summaries take; everything
  size_t static_bytes;   // what SPIFFY_STATIC_SCRATCH_BYTES limits: the head itself and candidate lists of the top-K
};
HeadWs carve_head(const spiffy_model_cfg* c, int G, int B, void* base) {
  const int M = G * B;
  Carve cv(base);
  HeadWs w;
  w.m_cap = (int)align_up((size_t)M, 128);
  w.n_part = head_mfma(c) ? mfma_lmhead_partials_per_row(c->vocab) : 0;
  w.row_idx = (int32_t*)cv.take(sizeof(int32_t) * w.m_cap);
  w.count = (int32_t*)cv.take(sizeof(int32_t) * 4);
  w.nf = cv.take((size_t)w.m_cap * c->d * esize(c->dtype));
  // Other shapes: parts of at least one 64-token tile.  Their number depends on the vocabulary alone: it sets the order in
  // which a row's exponentials are added.
  w.n_part_tile = head_mfma(c) ? 0 : cdiv(c->vocab, 64) < kTileHeadParts ? cdiv(c->vocab, 64) : kTileHeadParts;
  const size_t before = cv.off;
  w.part = (TopPartial*)cv.take(sizeof(TopPartial) * (size_t)(w.n_part + w.n_part_tile) * w.m_cap);
  w.tile_summary_bytes = head_mfma(c) ? 0 : cv.off - before;
  w.part2 = (TopPartial*)cv.take(sizeof(TopPartial) * (size_t)kLmheadCombineSlices * w.m_cap);
  w.row_top = (TopPartial*)cv.take(sizeof(TopPartial) * w.m_cap);
  const size_t lists = sizeof(float) * (size_t)B * SPIFFY_MAX_TOPK * SPIFFY_MAX_TOPK;
  w.static_bytes = cv.off - w.tile_summary_bytes + 2 * align_up(lists, 256);
  w.logits = w.cand_val = nullptr;
  w.chunk_id = w.cand_idx = nullptr;
  if (w.n_part) {
    w.logits = (float*)cv.take(sizeof(float) * (size_t)B * SPIFFY_MAX_TOPK * 128);
    w.chunk_id = (int32_t*)cv.take(sizeof(int32_t) * (size_t)B * SPIFFY_MAX_TOPK);
  } else {
    w.cand_val = (float*)cv.take(lists);
    w.cand_idx = (int32_t*)cv.take(lists);
  }
  w.bytes = cv.off;
  return w;
}

// layer and head scratch alias each other (used one after the other); the step adds a hidden
// buffer and a next-state buffer in front.
struct StepWs {
  void* hidden;
  int32_t* target;
  void* rest;
  size_t rest_bytes, bytes;
};
StepWs carve_step(const spiffy_model_cfg* c, int G, int B, int P, void* base, int S_seq = 0) {
  const size_t M = (size_t)G * B;
  Carve cv(base);
  StepWs w;
  // the layer / head scratch comes first, so that the head's leftovers sit at the start of the workspace whatever
  // G, B, P and S_seq were (spiffy_head_topk finds them there after a step)
  const size_t lb = carve_layer(c, G, B, P, nullptr, S_seq).bytes, hb = carve_head(c, G, B, nullptr).bytes;
  w.rest_bytes = lb > hb ? lb : hb;
  w.rest = cv.take(w.rest_bytes);
  w.hidden = cv.take((M + S_seq) * c->d * esize(c->dtype));
  w.target = (int32_t*)cv.take(sizeof(int32_t) * M);
  w.bytes = cv.off;
  return w;
}

int dev(hipError_t e) { return e == hipSuccess ? SPIFFY_OK : SPIFFY_EDEVICE; }

int check_layer_args(const spiffy_model_cfg* cfg, const spiffy_layer_weights* w, const spiffy_prefix_kv* prefix,
                     int32_t G, int32_t B) {
  if (!w || !prefix) return SPIFFY_EINVAL;
  if (!w->wq || !w->wk || !w->wv || !w->wo || !w->w_gate || !w->w_up || !w->w_down || !w->norm1 || !w->norm2)
    return SPIFFY_EINVAL;
  if (prefix->P < 0 || (prefix->P > 0 && (!prefix->k || !prefix->v))) return SPIFFY_EINVAL;
  if (prefix->capacity != 0 && prefix->capacity < prefix->P) return SPIFFY_EINVAL;
  if (prefix->S < 0 || (prefix->S > 0 && (!prefix->k || !prefix->v))) return SPIFFY_EINVAL;
  if (prefix->S > 0 && (int64_t)prefix->P + B + prefix->S > prefix->capacity) return SPIFFY_ESHAPE;  // suffix rows sit after the block's slot
  const void* ptrs[] = {w->wq, w->wk, w->wv, w->wo, w->w_gate, w->w_up, w->w_down, w->norm1, w->norm2,
                        w->bq, w->bk, w->bv, prefix->k, prefix->v};
  for (const void* p : ptrs)
    if (p && !aligned16(p)) return SPIFFY_EALIGN;
  if (!layer_mfma(cfg) && attn_limit_bytes(cfg, B, prefix->P + prefix->S) > kAttnLimitBytes) return SPIFFY_ESHAPE;
  // the reduction behind the split-K projections keeps a row of d fp32 values in 64 KB of LDS for its RMSNorm
  if (layer_mfma(cfg) && (size_t)cfg->d * sizeof(float) > 64 * 1024) return SPIFFY_ESHAPE;
  return SPIFFY_OK;
}

// Chaining hints used by the whole-step driver: `normed_in` = ws.n already holds RMSNorm-1 of hidden_in
// (written by the previous layer's last kernel); `next_norm1` = gain of the next layer's RMSNorm-1, to be
// produced into ws.n by this layer's last kernel; `rope_ready` = the rotary table is already in place.
enum Projection { QKV_PROJ, OUTPUT_PROJ, GATE_UP_PROJ, DOWN_PROJ };
struct LayerChain {
  bool normed_in = false;
  const void* next_norm1 = nullptr;
  bool rope_ready = false;
  bool normed_out = false;   // set when ws.n holds the next layer's normalised input on return
  bool append_kv = false;    // write the (rotated) K and V rows of state 0 into the cache at rows P .. P+B-1
  int seq_S = 0;             // full-sequence step: this many true suffix rows follow the G*B block rows
  // commit-and-verify step (seq_S == B): the trailing B rows are the finished block BEFORE the one being decoded.
  // prefix->P counts the rows in front of that finished block; its keys / values are written to cache rows
  // P .. P+B-1 and the G states (positions pos0 = that block's + B) attend to P + B cached rows.
  bool tail_is_prev_block = false;
  // Last layer of a step: only masked positions are decoded (Alg. 1 steps 1-4 look at masked positions only), so
  // beyond the attention, where every row still supplies keys and values, only their rows are computed.  rows /
  // count: the device-side list of those rows (ascending) in the layer scratch; the other rows of hidden_out are
  // left as they are.
  bool masked_rows_only = false;
  const int32_t* tokens = nullptr;    // [G,B] block tokens and optional explicit mask, for the row list
  const uint8_t* mask = nullptr;
  bool rows_ready = false;            // the row list is already in the layer scratch
  // The head follows on these rows: their final RMSNorm, row list and count go to its scratch when the last kernel of the
  // layer can do that (head_ready is set then).
  const void* final_norm = nullptr;
  void* head_nf = nullptr;
  HeadRows head = {nullptr, nullptr};
  bool head_ready = false;
  // Launch plans of the projections, made by the pass's first layer (n_ranges = 0 before): a function of the rows and widths,
  // which the layers of a pass share.
  RowsPlan plans[4] = {};
};

// the arguments of the QKV projection that decide which path it and the attention take
GemmArgs qkv_args(const spiffy_model_cfg* cfg, int M) {
  GemmArgs g;
  std::memset(&g, 0, sizeof(g));
  const int qd = cfg->n_q_heads * cfg->head_dim, kvd = cfg->n_kv_heads * cfg->head_dim;
  g.lda = cfg->d; g.M = M; g.K = cfg->d;
  g.Nseg[0] = qd; g.Nseg[1] = kvd; g.Nseg[2] = kvd;
  g.N = qd + 2 * kvd; g.ldc = g.N; g.scale = 1.f;
  return g;
}
bool attn_on_mfma(const spiffy_model_cfg* cfg, int M) { return layer_mfma(cfg) && mfma_gemm_supported(EPI_QKV, qkv_args(cfg, M)); }

// rotary table of a layer's block rows (positions pos0 ..) and of the rows behind them
RopeArgs rope_args(const spiffy_model_cfg* cfg, void* tab, int M, int B, int S_seq, int pos0, int tail_pos0) {
  return RopeArgs{(float2*)tab, B + S_seq, B, cfg->head_dim / 2, pos0, tail_pos0, attn_on_mfma(cfg, M) ? 1 : 0, cfg->rope_base};
}

// A projection of a layer over the rows [0, rows_a) and [rows_a, rows_a + rows_b), as `plan` says.
hipError_t launch_gemm_rows(int epi, GemmArgs g, const RowsPlan& plan, int rows_a, int rows_b, int dtype, hipStream_t st) {
  const size_t es = esize(dtype), ces = epi == EPI_PARTIAL ? sizeof(float) : es;
  g.Mz = g.M = rows_a + rows_b;
  if (plan.n_ranges == 1) return launch_gemm_plan(epi, g, plan.range[0], st);
  GemmArgs a = g;
  a.M = rows_a;
  const hipError_t e = launch_gemm_plan(epi, a, plan.range[0], st);
  if (e != hipSuccess) return e;
  GemmArgs b = g;
  b.M = rows_b;
  b.A = reinterpret_cast<const char*>(g.A) + (size_t)rows_a * g.lda * es;
  b.C = reinterpret_cast<char*>(g.C) + (size_t)rows_a * g.ldc * ces;
  if (g.R) b.R = reinterpret_cast<const char*>(g.R) + (size_t)rows_a * g.ldc * es;
  b.qkv.row0 += rows_a;
  return launch_gemm_plan(epi, b, plan.range[1], st);
}

int run_layer(const spiffy_model_cfg* cfg, const spiffy_layer_weights* w, const spiffy_prefix_kv* prefix,
              const void* hidden_in, int G, int B, int pos0, void* hidden_out, void* workspace, hipStream_t st,
              LayerChain* chain = nullptr) {
  // S_seq > 0 (full-sequence step): rows G*B .. G*B+S_seq-1 of every activation matrix are the true suffix.  It is
  // recomputed like the blocks; its fresh keys / values, and those of the true block (state 0), go to the cache
  // rows behind the prefix, where the blocks find the suffix (as in the dual-cache layout) and the suffix rows
  // find the whole true sequence.
  const int S_seq = chain ? chain->seq_S : 0;
  const bool prev = chain && chain->tail_is_prev_block;
  const int M = G * B + S_seq, d = cfg->d, dt = cfg->dtype;
  const int qd = cfg->n_q_heads * cfg->head_dim, kvd = cfg->n_kv_heads * cfg->head_dim;
  const bool mf = layer_mfma(cfg);
  const LayerWs ws = carve_layer(cfg, G, B, prefix->P + prefix->S, workspace, S_seq);
  int rc;
  auto mfma_rows = [&](Projection which, int epi, const GemmArgs& ga) {
    if (ga.M_dev && ga.M > kMaskedLikeLayerRows) return launch_gemm_plan(epi, ga, plan_gemm_masked(epi, ga.M, ga.N, ga.K, ga.ksplit), st);
    RowsPlan alone = {};
    RowsPlan& plan = chain ? chain->plans[which] : alone;
    if (plan.n_ranges == 0) plan = plan_gemm_rows(epi, G * B, S_seq, ga.N, ga.K, ga.ksplit);
    return launch_gemm_rows(epi, ga, plan, G * B, S_seq, dt, st);
  };
  if (chain) chain->normed_out = false;
  if (!(chain && chain->normed_in) &&
      (rc = dev(launch_rmsnorm(dt, hidden_in, w->norm1, cfg->rms_eps, M, d, nullptr, nullptr, ws.n, st))))
    return rc;

  GemmArgs g = qkv_args(cfg, M);
  g.A = ws.n;
  g.W[0] = w->wq; g.W[1] = w->wk; g.W[2] = w->wv;
  g.bias[0] = w->bq; g.bias[1] = w->bk; g.bias[2] = w->bv;
  g.C = ws.qkv;
  AttnArgs a;
  a.qkv = ws.qkv; a.prefix_k = prefix->k; a.prefix_v = prefix->v; a.out = ws.attn;
  a.G = G; a.B = B; a.Hq = cfg->n_q_heads; a.Hkv = cfg->n_kv_heads; a.hd = cfg->head_dim; a.P = prefix->P;
  a.ldp = prefix->capacity;
  a.S = S_seq ? S_seq : prefix->S;
  if (prev) {                // the finished block has joined the prefix; a cached suffix loses the current block's slot
    a.P = prefix->P + B;
    a.S = prefix->S > B ? prefix->S - B : 0;
  }
  a.own = 1;
  a.pos0 = pos0; a.rope_base = cfg->rope_base;
  const int ldp = prefix->capacity ? prefix->capacity : prefix->P;
  const int tail_pos0 = prev ? pos0 - B : pos0 + B;
  void* const rope_seq = reinterpret_cast<float2*>(ws.rope) + (size_t)B * (cfg->head_dim / 2);
  const bool append = chain && chain->append_kv;
  const bool mfa = attn_on_mfma(cfg, M);
  if (!(chain && chain->rope_ready) &&
      (rc = dev(launch_rope_table(rope_args(cfg, ws.rope, M, B, S_seq, pos0, tail_pos0), st))))
    return rc;
  if (mfa) {
    // queries and keys are rotated, and the rows that extend the cache are stored there, by the projection's epilogue
    QkvArgs& q = g.qkv;
    q.rope = ws.rope; q.rope_rows = B + S_seq;
    q.ck = const_cast<void*>(prefix->k); q.cv = const_cast<void*>(prefix->v); q.ldp = ldp;
    q.rows = G * B; q.B = B; q.magic = (unsigned)((((unsigned long long)1 << 32) + B - 1) / B);
    q.q_scale = 1.4426950408889634f * 0.08838834764831845f;      // log2(e) / sqrt(128)
    q.n_head = append || (S_seq && !prev) ? B : 0;               // the block itself, or the true block (state 0) ..
    q.dst_head = prefix->P;
    q.dst_tail = !S_seq ? -1 : prev ? prefix->P : prefix->P + B; // .. and the suffix behind it; or the finished block
    if ((rc = dev(mfma_rows(QKV_PROJ, EPI_QKV, g)))) return rc;
    a.partial = ws.attn_partial;
  } else {
    if ((rc = dev(launch_gemm_tile(dt, EPI_STORE, g, st)))) return rc;
    a.partial = ws.rope;
    // the true block (state 0: qkv rows 0 .. B-1) and the suffix (qkv rows G*B ..) land next to each other in the cache, at
    // consecutive positions: one launch over the two runs of rows
    if (S_seq && !prev)
      rc = dev(launch_kv_append(dt, ws.qkv, a.Hq, a.Hkv, a.hd, B + S_seq, pos0, cfg->rope_base, const_cast<void*>(prefix->k),
                                const_cast<void*>(prefix->v), prefix->P, ldp, st, B, (G - 1) * B));
    else if (append)
      rc = dev(launch_kv_append(dt, ws.qkv, a.Hq, a.Hkv, a.hd, B, pos0, cfg->rope_base, const_cast<void*>(prefix->k),
                                const_cast<void*>(prefix->v), prefix->P, ldp, st));
    else if (S_seq)    // the finished block in front of the states
      rc = dev(launch_kv_append(dt, reinterpret_cast<const char*>(ws.qkv) + (size_t)G * B * g.N * esize(dt), a.Hq, a.Hkv, a.hd,
                                S_seq, tail_pos0, cfg->rope_base, const_cast<void*>(prefix->k), const_cast<void*>(prefix->v),
                                prefix->P, ldp, st));
    if (rc) return rc;
  }
  if (!(S_seq && mfa) &&      // with rows riding along, the MFMA path runs both groups in one launch below
      (rc = dev(mfa ? launch_attn_mfma(a, st) : launch_attn_tile(dt, a, st))))
    return rc;
  if (S_seq) {      // the suffix rows: queries at positions pos0+B .., keys = cache rows 0 .. P+B+S_seq-1, no block of their own
    const size_t es = esize(dt);
    AttnArgs b = a;
    b.qkv = reinterpret_cast<const char*>(ws.qkv) + (size_t)G * B * g.N * es;
    b.out = reinterpret_cast<char*>(ws.attn) + (size_t)G * B * qd * es;
    b.partial = mfa ? ws.attn_partial_seq : rope_seq;
    b.G = 1; b.B = S_seq; b.P = prefix->P + B + S_seq; b.S = 0; b.own = 0;
    b.pos0 = tail_pos0;
    if (prev) {     // the finished block: one state at the positions before pos0, over the rows in front of it
      b.P = prefix->P; b.S = prefix->S; b.own = 1;
    }
    if (mfa) {       // (b differs from a in row counts and lengths only)
      if ((rc = dev(launch_attn_mfma_pair(a, b, st)))) return rc;
    } else if ((rc = dev(launch_attn_tile(dt, b, st)))) return rc;
  }

  // Masked rows only (last layer): from here on row r of every matrix is row ws.rows[r] of the block rows, r < *ws.count.
  // The row count is known on the device only: the launches cover all M rows and skip what lies beyond it.  A row's
  // arithmetic does not depend on where it sits, so the results are those of the full layer, bit for bit.
  const bool cm = chain && chain->masked_rows_only && !S_seq;
  const int32_t* n_rows = cm ? ws.count : nullptr;
  const void* attn_rows = ws.attn;
  const void* resid = hidden_in;
  std::memset(&g, 0, sizeof(g));
  g.lda = qd; g.M = M; g.M_dev = n_rows; g.K = qd; g.W[0] = w->wo; g.Nseg[0] = d; g.N = d;
  g.C = ws.h; g.ldc = d; g.scale = 1.f;
  const bool o_mfma = mf && mfma_gemm_supported(EPI_RESID, g);
  const int o_slices = o_mfma ? mfma_ksplit(d, qd) : 1;
  const int32_t* src_rows = nullptr;       // the output projection and its reduction read the rows where they are ..
  if (cm) {
    const size_t es = esize(dt);
    if (!chain->rows_ready &&
        (rc = dev(launch_compact_rows(chain->tokens, chain->mask, cfg->mask_id, M, ws.rows, ws.count, st))))
      return rc;
    if (o_slices > 1) {
      src_rows = ws.rows;
    } else {                               // .. or they are gathered first
      if ((rc = dev(launch_gather_rows2(ws.attn, (size_t)qd * es, hidden_in, (size_t)d * es, ws.rows, ws.count, M, ws.gat_attn,
                                        ws.gat_x, st))))
        return rc;
      attn_rows = ws.gat_attn;
      resid = ws.gat_x;
    }
  }

  // output projection + residual (+ RMSNorm-2 fused into the split-K reduction when K is sliced)
  g.A = attn_rows; g.R = resid;
  bool normed = false;
  if (o_mfma) {
    if (o_slices > 1) {
      g.C = ws.splitk; g.ksplit = o_slices; g.a_rows = src_rows;
      if ((rc = dev(mfma_rows(OUTPUT_PROJ, EPI_PARTIAL, g)))) return rc;
      if ((rc = dev(launch_splitk_reduce((const float*)ws.splitk, o_slices, resid, ws.h, w->norm2, cfg->rms_eps, ws.n, M,
                                         d, st, n_rows, nullptr, src_rows))))
        return rc;
      normed = true;
    } else if ((rc = dev(mfma_rows(OUTPUT_PROJ, EPI_RESID, g)))) return rc;
  } else if ((rc = dev(launch_gemm_tile(dt, EPI_RESID, g, st)))) return rc;

  if (!normed && (rc = dev(launch_rmsnorm(dt, ws.h, w->norm2, cfg->rms_eps, M, d, nullptr, n_rows, ws.n, st))))
    return rc;

  std::memset(&g, 0, sizeof(g));
  g.A = ws.n; g.lda = d; g.M = M; g.M_dev = n_rows; g.K = d; g.W[0] = w->w_gate; g.W[1] = w->w_up; g.N = cfg->ffn;
  g.C = ws.act; g.ldc = cfg->ffn; g.scale = 1.f;
  if ((rc = dev(mf && mfma_gemm_supported(EPI_SWIGLU, g) ? mfma_rows(GATE_UP_PROJ, EPI_SWIGLU, g)
                                                          : launch_gemm_tile(dt, EPI_SWIGLU, g, st))))
    return rc;

  // down projection + residual; compacted rows go back to their places in hidden_out (by the reduction when K is
  // sliced, else through ws.gat_x, which is free once the output projection has read it)
  std::memset(&g, 0, sizeof(g));
  g.A = ws.act; g.lda = cfg->ffn; g.M = M; g.M_dev = n_rows; g.K = cfg->ffn; g.W[0] = w->w_down; g.Nseg[0] = d; g.N = d;
  g.C = cm ? ws.gat_x : hidden_out; g.ldc = d; g.R = ws.h; g.scale = 1.f;
  if (mf && mfma_gemm_supported(EPI_RESID, g)) {
    const int ks = mfma_ksplit(d, cfg->ffn);
    if (ks > 1) {
      g.C = ws.splitk; g.ksplit = ks;
      if ((rc = dev(mfma_rows(DOWN_PROJ, EPI_PARTIAL, g)))) return rc;
      if (cm && chain->head_nf) {
        chain->head_ready = true;
        return dev(launch_splitk_reduce((const float*)ws.splitk, ks, ws.h, hidden_out, chain->final_norm, cfg->rms_eps,
                                        chain->head_nf, M, d, st, n_rows, ws.rows, nullptr, &chain->head));
      }
      const void* ng = chain ? chain->next_norm1 : nullptr;
      if (chain && ng) chain->normed_out = true;
      return dev(launch_splitk_reduce((const float*)ws.splitk, ks, ws.h, hidden_out, ng, cfg->rms_eps,
                                      ng ? ws.n : nullptr, M, d, st, n_rows, cm ? ws.rows : nullptr));
    }
    if ((rc = dev(mfma_rows(DOWN_PROJ, EPI_RESID, g)))) return rc;
  } else if ((rc = dev(launch_gemm_tile(dt, EPI_RESID, g, st)))) return rc;
  if (cm) return dev(launch_scatter_rows(ws.gat_x, (size_t)d * esize(dt), ws.rows, ws.count, M, hidden_out, st));
  return SPIFFY_OK;
}

// First kernel of a step: hidden rows of the block tokens (and of the n_tail rows behind them), the first layer's normalised
// input at the start of the layer scratch, the rotary table of all layers and, when the last layer is to compute the masked
// rows only, their list.  The table and the list lie in front of everything whose place depends on a layer's cached rows.
int begin_step(const spiffy_model_cfg* cfg, int n_layers, const spiffy_layer_weights* layers, const void* w_embed,
               const int32_t* tokens, int G, int B, const int32_t* tail_tokens, int n_tail, int pos0, int tail_pos0, void* hid,
               bool list, void* scratch, LayerChain& chain, hipStream_t st) {
  const LayerWs ws = carve_layer(cfg, G, B, 0, scratch, n_tail);
  EmbedArgs e = {};
  e.w = w_embed; e.tok = tokens; e.tok2 = tail_tokens; e.M = G * B; e.M2 = n_tail; e.d = cfg->d; e.V = cfg->vocab;
  e.out = hid; e.n_out = ws.n; e.eps = cfg->rms_eps; e.mask_id = cfg->mask_id;
  if (n_layers > 0) {
    e.gain = layers[0].norm1;
    e.rope = rope_args(cfg, ws.rope, G * B + n_tail, B, n_tail, pos0, tail_pos0);
    if (list) { e.rows = ws.rows; e.count = ws.count; }
  }
  chain.normed_out = chain.rope_ready = true;
  chain.rows_ready = list;
  return dev(launch_embed(cfg->dtype, e, st));
}

int run_head(const spiffy_model_cfg* cfg, const void* hidden, const void* final_norm, const void* w_vocab,
             const int32_t* tokens, const uint8_t* mask, int G, int B, float threshold, float logit_scale,
             int force_one, int32_t* argmax, float* conf, uint8_t* unmask, float* margin, int32_t* target,
             void* workspace, hipStream_t st, bool rows_ready = false) {
  const int M = G * B, dt = cfg->dtype;
  const HeadWs ws = carve_head(cfg, G, B, workspace);
  int rc;
  if (!rows_ready &&
      (rc = dev(launch_masked_rmsnorm(dt, hidden, final_norm, cfg->rms_eps, M, cfg->d, tokens, mask, cfg->mask_id,
                                      ws.row_idx, ws.count, ws.nf, st))))
    return rc;
  int n_part = ws.n_part;
  if (head_mfma(cfg)) {
    GemmArgs g;
    std::memset(&g, 0, sizeof(g));
    g.A = ws.nf; g.lda = cfg->d; g.M = M; g.M_dev = ws.count; g.K = cfg->d;
    g.W[0] = w_vocab; g.Nseg[0] = cfg->vocab; g.N = cfg->vocab;
    g.C = ws.part; g.ldc = ws.m_cap; g.scale = logit_scale;
    if ((rc = dev(launch_gemm_mfma(EPI_LMHEAD, g, st)))) return rc;
  } else {
    n_part = ws.n_part_tile;
    if ((rc = dev(launch_lmhead_tile(dt, ws.nf, w_vocab, cfg->d, cfg->vocab, logit_scale, ws.count, M, ws.m_cap, n_part,
                                     ws.part, st))))
      return rc;
  }
  int n_sums = 1;                                  // 1: merged in row_top; more: slices in part2
  if ((rc = dev(launch_lmhead_combine(ws.part, n_part, ws.m_cap, ws.count, M, ws.part2, ws.row_top, &n_sums, st)))) return rc;
  return dev(launch_head_finalize(ws.part2, n_sums, ws.m_cap, ws.row_top, ws.row_idx, ws.count, tokens, mask, cfg->mask_id, G, B, threshold,
                                  force_one, argmax, conf, unmask, margin, target, st));
}

int check_head_args(const spiffy_model_cfg* cfg, const void* hidden, const void* final_norm, const void* w_vocab,
                    const int32_t* tokens, float threshold, float logit_scale, const int32_t* argmax,
                    const float* conf, const uint8_t* unmask) {
  if (!hidden || !final_norm || !w_vocab || !tokens || !argmax || !conf || !unmask) return SPIFFY_EINVAL;
  if (!(threshold >= 0.f && threshold <= 1.f) || !(logit_scale > 0.f) || !std::isfinite(logit_scale))
    return SPIFFY_EINVAL;
  if (!aligned16(hidden) || !aligned16(final_norm) || !aligned16(w_vocab)) return SPIFFY_EALIGN;
  if ((size_t)cfg->d * sizeof(float) > 64 * 1024 && !head_mfma(cfg)) return SPIFFY_ESHAPE;   // d <= 16384
  return head_shape_ok(cfg) ? SPIFFY_OK : SPIFFY_ESHAPE;
}

int check_accept_args(const int32_t* edges, int32_t E, const int32_t* draft, const int32_t* target, int32_t G,
                      int32_t B, int32_t root, const spiffy_accept_result* res) {
  if (G < 1 || B < 1 || E < 0 || (E > 0 && !edges) || !draft || !target || !res) return SPIFFY_EINVAL;
  if (root < 0 || root >= G) return SPIFFY_EINVAL;
  if (G > SPIFFY_MAX_G) return SPIFFY_ESHAPE;
  return SPIFFY_OK;
}

// arguments of a projection alone, without pointers
GemmArgs gemm_shape(int epilogue, int M, int N, int K) {
  GemmArgs g;
  std::memset(&g, 0, sizeof(g));
  g.M = M; g.N = N; g.K = K; g.lda = K; g.ldc = N; g.scale = 1.f;
  if (epilogue != SPIFFY_GEMM_SWIGLU) g.Nseg[0] = N;
  return g;
}

// a projection alone; layer: in the tiles that a layer's projections take (the matrix-core kernel only)
int gemm_call(int dtype, int epilogue, const void* A, const void* W0, const void* W1, const void* R, void* C, int M, int N, int K,
              void* workspace, size_t workspace_bytes, hipStream_t st, bool layer) {
  if (dtype != SPIFFY_BF16 && dtype != SPIFFY_F32) return SPIFFY_EINVAL;
  if (epilogue < SPIFFY_GEMM_STORE || epilogue > SPIFFY_GEMM_SWIGLU) return SPIFFY_EINVAL;
  if (!A || !W0 || !C || M < 1 || N < 1 || K < 1) return SPIFFY_EINVAL;
  if (epilogue == SPIFFY_GEMM_SWIGLU && !W1) return SPIFFY_EINVAL;
  if (epilogue == SPIFFY_GEMM_RESID && !R) return SPIFFY_EINVAL;
  if (K % 8 != 0 || N % 8 != 0) return SPIFFY_ESHAPE;
  if (!aligned16(A) || !aligned16(W0) || !aligned16(C) || (W1 && !aligned16(W1)) || (R && !aligned16(R)))
    return SPIFFY_EALIGN;
  GemmArgs g = gemm_shape(epilogue, M, N, K);
  g.A = A; g.C = C; g.R = R; g.W[0] = W0;
  if (epilogue == SPIFFY_GEMM_SWIGLU) g.W[1] = W1;
  const bool mf = dtype == SPIFFY_BF16 && mfma_gemm_supported(epilogue, g);
  if (layer && !mf) return SPIFFY_ESHAPE;
  const auto launch = [&](int epi) {
    return dev(layer ? launch_gemm_plan(epi, g, plan_gemm_layer(epi, M, N, K, g.ksplit), st) : launch_gemm_mfma(epi, g, st));
  };
  if (mf && epilogue == SPIFFY_GEMM_RESID) {     // same K slicing as verify_layer when scratch is given
    const int ks = mfma_ksplit(N, K);
    if (ks > 1 && layer && !workspace) return SPIFFY_EINVAL;
    if (ks > 1 && workspace) {
      if (reinterpret_cast<uintptr_t>(workspace) & 255u) return SPIFFY_EALIGN;
      if (workspace_bytes < sizeof(float) * (size_t)ks * M * N) return SPIFFY_EWORKSPACE;
      g.C = workspace; g.ksplit = ks;
      const int rc = launch(EPI_PARTIAL);
      if (rc) return rc;
      return dev(launch_splitk_reduce((const float*)workspace, ks, R, C, nullptr, 0.f, nullptr, M, N, st));
    }
  }
  return mf ? launch(epilogue) : dev(launch_gemm_tile(dtype, epilogue, g, st));
}

void put_plan(const GemmPlan& p, int k_slices, spiffy_gemm_plan_t* plan) {
  std::memset(plan, 0, sizeof(*plan));
  plan->n_launches = p.n_parts;
  plan->k_slices = k_slices;
  for (int i = 0; i < p.n_parts; ++i) {
    plan->launch[i].tile_rows = p.part[i].bm;
    plan->launch[i].tile_cols = p.part[i].bn;
    plan->launch[i].col0 = p.part[i].col0;
    plan->launch[i].n_cols = p.part[i].ncols;
    plan->launch[i].workgroups = p.part[i].workgroups;
  }
}

// Device address of `scratch` on the current device: looked up once per device, with that device current.
int static_scratch_ptr(void** out) {
  static std::mutex mu;
  static void* ptr[64] = {};
  int d = 0;
  if (hipGetDevice(&d) != hipSuccess || d < 0 || d >= 64) return SPIFFY_EDEVICE;
  std::lock_guard<std::mutex> lock(mu);
  if (!ptr[d]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return SPIFFY_EDEVICE;
    ptr[d] = p;
  }
  *out = ptr[d];
  return SPIFFY_OK;
}

}  // namespace

extern "C" {
#pragma GCC visibility push(default)

const char* spiffy_status_str(int s) {
  switch (s) {
    case SPIFFY_OK: return "ok";
    case SPIFFY_EINVAL: return "invalid argument";
    case SPIFFY_ESHAPE: return "unsupported shape";
    case SPIFFY_EALIGN: return "pointer not 16-byte aligned";
    case SPIFFY_EWORKSPACE: return "workspace too small";
    case SPIFFY_EDEVICE: return "device launch failed";
    case SPIFFY_ELIMIT: return "size beyond the limit of the allocation-free entry point";
    default: return "unknown status";
  }
}

int spiffy_uses_mfma(const spiffy_model_cfg* cfg, int32_t B) {
  int rc = check_cfg(cfg);
  if (rc) return rc;
  if (B < 1) return SPIFFY_EINVAL;
  return layer_mfma(cfg) ? 1 : 0;
}

size_t spiffy_workspace_bytes(const spiffy_model_cfg* cfg, int32_t G, int32_t B, int32_t P_max) {
  if (check_cfg(cfg) || check_gb(G, B) || P_max < 0) return 0;
  return carve_step(cfg, G, B, P_max, nullptr).bytes;
}

int spiffy_embed(const spiffy_model_cfg* cfg, const void* w_embed, const int32_t* block_tokens, int32_t G,
                 int32_t B, void* hidden_out, void* stream) {
  int rc;
  if ((rc = check_cfg(cfg)) || (rc = check_gb(G, B))) return rc;
  if (!w_embed || !block_tokens || !hidden_out) return SPIFFY_EINVAL;
  if (!aligned16(w_embed) || !aligned16(hidden_out)) return SPIFFY_EALIGN;
  EmbedArgs e = {};
  e.w = w_embed; e.tok = block_tokens; e.M = G * B; e.d = cfg->d; e.V = cfg->vocab; e.out = hidden_out;
  return dev(launch_embed(cfg->dtype, e, (hipStream_t)stream));
}

int spiffy_verify_layer(const spiffy_model_cfg* cfg, const spiffy_layer_weights* w, const spiffy_prefix_kv* prefix,
                        const void* hidden_in, int32_t G, int32_t B, int32_t pos0, void* hidden_out,
                        void* workspace, size_t workspace_bytes, void* stream) {
  int rc;
  if ((rc = check_cfg(cfg)) || (rc = check_gb(G, B))) return rc;
  if (!hidden_in || !hidden_out || !workspace || pos0 < 0) return SPIFFY_EINVAL;
  if ((rc = check_layer_args(cfg, w, prefix, G, B))) return rc;
  if (!aligned16(hidden_in) || !aligned16(hidden_out) || (reinterpret_cast<uintptr_t>(workspace) & 255u))
    return SPIFFY_EALIGN;
  if (workspace_bytes < carve_layer(cfg, G, B, prefix->P + prefix->S, nullptr).bytes) return SPIFFY_EWORKSPACE;
  return run_layer(cfg, w, prefix, hidden_in, G, B, pos0, hidden_out, workspace, (hipStream_t)stream);
}

int spiffy_verify_layer_last(const spiffy_model_cfg* cfg, const spiffy_layer_weights* w, const spiffy_prefix_kv* prefix,
                             const void* hidden_in, const int32_t* block_tokens, const uint8_t* mask, int32_t G, int32_t B,
                             int32_t pos0, void* hidden_out, void* workspace, size_t workspace_bytes, void* stream) {
  int rc;
  if ((rc = check_cfg(cfg)) || (rc = check_gb(G, B))) return rc;
  if (!hidden_in || !hidden_out || !workspace || !block_tokens || pos0 < 0) return SPIFFY_EINVAL;
  if ((rc = check_layer_args(cfg, w, prefix, G, B))) return rc;
  if (!aligned16(hidden_in) || !aligned16(hidden_out) || (reinterpret_cast<uintptr_t>(workspace) & 255u))
    return SPIFFY_EALIGN;
  if (workspace_bytes < carve_layer(cfg, G, B, prefix->P + prefix->S, nullptr).bytes) return SPIFFY_EWORKSPACE;
  LayerChain chain;
  chain.masked_rows_only = true;
  chain.tokens = block_tokens;
  chain.mask = mask;
  return run_layer(cfg, w, prefix, hidden_in, G, B, pos0, hidden_out, workspace, (hipStream_t)stream, &chain);
}

int spiffy_decode_head(const spiffy_model_cfg* cfg, const void* hidden, const void* final_norm, const void* w_vocab,
                       const int32_t* block_tokens, const uint8_t* mask, int32_t G, int32_t B, float threshold,
                       float logit_scale, int32_t force_one, int32_t* argmax, float* conf, uint8_t* unmask,
                       float* top2_margin, int32_t* target_states, void* workspace, size_t workspace_bytes,
                       void* stream) {
  int rc;
  if ((rc = check_cfg(cfg)) || (rc = check_gb(G, B))) return rc;
  if (!workspace) return SPIFFY_EINVAL;
  if ((rc = check_head_args(cfg, hidden, final_norm, w_vocab, block_tokens, threshold, logit_scale, argmax, conf,
                            unmask)))
    return rc;
  if (reinterpret_cast<uintptr_t>(workspace) & 255u) return SPIFFY_EALIGN;
  if (workspace_bytes < carve_head(cfg, G, B, nullptr).bytes) return SPIFFY_EWORKSPACE;
  return run_head(cfg, hidden, final_norm, w_vocab, block_tokens, mask, G, B, threshold, logit_scale, force_one,
                  argmax, conf, unmask, top2_margin, target_states, workspace, (hipStream_t)stream);
}

int spiffy_decode_head_static(const spiffy_model_cfg* cfg, const void* hidden, const void* final_norm,
                              const void* w_vocab, const int32_t* block_tokens, const uint8_t* mask, int32_t G,
                              int32_t B, float threshold, float logit_scale, int32_t force_one, int32_t* argmax,
                              float* conf, uint8_t* unmask, float* top2_margin, int32_t* target_states, void* stream) {
  int rc;
  if ((rc = check_cfg(cfg)) || (rc = check_gb(G, B))) return rc;
  if ((rc = check_head_args(cfg, hidden, final_norm, w_vocab, block_tokens, threshold, logit_scale, argmax, conf,
                            unmask)))
    return rc;
  if ((int64_t)G * B > SPIFFY_STATIC_MAX_ROWS) return SPIFFY_ELIMIT;
  const HeadWs need = carve_head(cfg, G, B, nullptr);
  if (need.static_bytes > (size_t)SPIFFY_STATIC_SCRATCH_BYTES) return SPIFFY_ELIMIT;
  void* ws = nullptr;
  if ((rc = static_scratch_ptr(&ws))) return rc;
  // every kernel of the head writes what it later reads (row list and count, gathered rows, summaries): nothing in
  // the scratch has to start at zero, and what the previous call left there is never read
  return run_head(cfg, hidden, final_norm, w_vocab, block_tokens, mask, G, B, threshold, logit_scale, force_one,
                  argmax, conf, unmask, top2_margin, target_states, ws, (hipStream_t)stream);
}

int spiffy_gemm(int32_t dtype, int32_t epilogue, const void* A, const void* W0, const void* W1, const void* R,
                void* C, int32_t M, int32_t N, int32_t K, void* workspace, size_t workspace_bytes, void* stream) {
  return gemm_call(dtype, epilogue, A, W0, W1, R, C, M, N, K, workspace, workspace_bytes, (hipStream_t)stream, false);
}

int spiffy_layer_gemm(int32_t epilogue, const void* A, const void* W0, const void* W1, const void* R, void* C, int32_t M,
                      int32_t N, int32_t K, void* workspace, size_t workspace_bytes, void* stream) {
  if (epilogue == SPIFFY_GEMM_STORE) return SPIFFY_EINVAL;
  return gemm_call(SPIFFY_BF16, epilogue, A, W0, W1, R, C, M, N, K, workspace, workspace_bytes, (hipStream_t)stream, true);
}

int spiffy_gemm_plan(int32_t epilogue, int32_t M, int32_t N, int32_t K, int32_t with_workspace,
                     spiffy_gemm_plan_t* plan) {
  if (!plan || epilogue < SPIFFY_GEMM_STORE || epilogue > SPIFFY_GEMM_SWIGLU) return SPIFFY_EINVAL;
  if (M < 1 || N < 1 || K < 1) return SPIFFY_ESHAPE;
  if (!mfma_gemm_supported(epilogue, gemm_shape(epilogue, M, N, K))) return SPIFFY_ESHAPE;
  int epi = epilogue, ks = 1;
  if (epilogue == SPIFFY_GEMM_RESID && with_workspace && mfma_ksplit(N, K) > 1) { epi = EPI_PARTIAL; ks = mfma_ksplit(N, K); }
  put_plan(plan_gemm_mfma(epi, M, N, ks), ks, plan);
  return SPIFFY_OK;
}

int spiffy_layer_gemm_plan(int32_t epilogue, int32_t M, int32_t M_tail, int32_t N, int32_t K, spiffy_gemm_plan_t* plans,
                           int32_t* n_ranges) {
  if (!plans || !n_ranges || epilogue < SPIFFY_GEMM_STORE || epilogue > SPIFFY_GEMM_SWIGLU) return SPIFFY_EINVAL;
  const bool masked = M_tail == SPIFFY_TAIL_MASKED;
  if (masked) M_tail = 0;
  if (M < 1 || M_tail < 0 || M > INT32_MAX - M_tail || N < 1 || K < 1) return SPIFFY_ESHAPE;
  if (!mfma_gemm_supported(epilogue, gemm_shape(epilogue, M + M_tail, N, K))) return SPIFFY_ESHAPE;
  if (epilogue == SPIFFY_GEMM_STORE && N % 128 != 0) return SPIFFY_ESHAPE;       // heads of 128 columns
  int epi = epilogue == SPIFFY_GEMM_STORE ? EPI_QKV : epilogue, ks = 1;
  if (epilogue == SPIFFY_GEMM_RESID && mfma_ksplit(N, K) > 1) { epi = EPI_PARTIAL; ks = mfma_ksplit(N, K); }
  const RowsPlan p = masked ? RowsPlan{1, {plan_gemm_masked(epi, M, N, K, ks)}} : plan_gemm_rows(epi, M, M_tail, N, K, ks);
  *n_ranges = p.n_ranges;
  for (int i = 0; i < p.n_ranges; ++i) {
    if (!plan_has_kernels(epi, p.range[i])) return SPIFFY_EDEVICE;
    put_plan(p.range[i], ks, &plans[i]);
  }
  return SPIFFY_OK;
}

int spiffy_graph_accept(const int32_t* graph_edges, int32_t E, const int32_t* draft_states,
                        const int32_t* target_states, int32_t G, int32_t B, int32_t root,
                        spiffy_accept_result* result, int32_t* accepted_state, void* stream) {
  int rc = check_accept_args(graph_edges, E, draft_states, target_states, G, B, root, result);
  if (rc) return rc;
  return dev(launch_graph_accept(graph_edges, E, draft_states, target_states, G, B, root, result, accepted_state,
                                 (hipStream_t)stream));
}

int spiffy_head_topk(const spiffy_model_cfg* cfg, const void* w_vocab, const int32_t* block_tokens, int32_t G,
                     int32_t B, const spiffy_accept_result* result, int32_t node, int32_t K, float logit_scale,
                     int32_t after_step, int32_t* topk_tokens, float* topk_probs, void* workspace,
                     size_t workspace_bytes, void* stream) {
  int rc;
  if ((rc = check_cfg(cfg)) || (rc = check_gb(G, B))) return rc;
  if (!w_vocab || !block_tokens || !topk_tokens || !topk_probs || !workspace) return SPIFFY_EINVAL;
  if (!(logit_scale > 0.f) || !std::isfinite(logit_scale)) return SPIFFY_EINVAL;
  if (!result && (node < 0 || node >= G)) return SPIFFY_EINVAL;
  if (K < 1 || K > SPIFFY_MAX_TOPK) return SPIFFY_ESHAPE;
  if (cfg->dtype == SPIFFY_BF16 && cfg->d % 8 != 0) return SPIFFY_ESHAPE;
  if (!head_shape_ok(cfg)) return SPIFFY_ESHAPE;
  if (!aligned16(w_vocab)) return SPIFFY_EALIGN;
  if (reinterpret_cast<uintptr_t>(workspace) & 255u) return SPIFFY_EALIGN;
  // a step keeps its layer / head scratch at the start of its workspace, so the head's leftovers are found at the
  // same place after spiffy_decode_head and after a whole step
  (void)after_step;
  void* head_base = workspace;
  if (workspace_bytes < carve_head(cfg, G, B, nullptr).bytes) return SPIFFY_EWORKSPACE;
  const HeadWs ws = carve_head(cfg, G, B, head_base);
  HeadTopkArgs a;
  a.dtype = cfg->dtype; a.nf = ws.nf; a.w_vocab = w_vocab; a.d = cfg->d; a.V = cfg->vocab; a.scale = logit_scale;
  a.part = ws.part; a.n_part = ws.n_part; a.m_cap = ws.m_cap; a.row_top = ws.row_top; a.row_idx = ws.row_idx;
  a.count = ws.count; a.tokens = block_tokens; a.result = result; a.node = node; a.G = G; a.B = B; a.K = K;
  a.logits = ws.logits; a.chunk_id = ws.chunk_id; a.cand_val = ws.cand_val; a.cand_idx = ws.cand_idx; a.out_tokens = topk_tokens; a.out_probs = topk_probs;
  return dev(launch_head_topk(a, (hipStream_t)stream));
}

int spiffy_draft_prune(const int32_t* state, int32_t B, int32_t mask_id, const int32_t* topk_tokens,
                       const float* topk_probs, int32_t K, const int32_t* formula_offsets,
                       const int32_t* formula_pairs, int32_t D, int32_t nnz, const int32_t* edges, int32_t E,
                       int32_t d_star, int32_t* drafts, uint8_t* buildable, float* local, float* score,
                       int32_t* kept, int32_t* states_out, int32_t* edges_out, int32_t* counts, void* stream) {
  if (!state || !topk_tokens || !topk_probs || !formula_offsets || !drafts || !buildable || !local || !score ||
      !kept || !states_out || !counts)
    return SPIFFY_EINVAL;
  if ((nnz > 0 && !formula_pairs) || (E > 0 && (!edges || !edges_out))) return SPIFFY_EINVAL;
  if (B < 1 || B > 4096 || K < 1 || K > 16 || D < 0 || D > SPIFFY_MAX_G - 1 || nnz < 0 || E < 0 || d_star < 0)
    return SPIFFY_ESHAPE;
  DraftPruneArgs a;
  a.state = state; a.topk_tokens = topk_tokens; a.topk_probs = topk_probs;
  a.formula_offsets = formula_offsets; a.formula_pairs = formula_pairs; a.edges = edges;
  a.drafts = drafts; a.buildable = buildable; a.local = local; a.score = score; a.kept = kept;
  a.states_out = states_out; a.edges_out = edges_out; a.counts = counts;
  a.B = B; a.K = K; a.D = D; a.nnz = nnz; a.E = E; a.d_star = d_star; a.mask_id = mask_id;
  return dev(launch_draft_prune(a, (hipStream_t)stream));
}

int spiffy_verify_step(const spiffy_model_cfg* cfg, int32_t n_layers, const spiffy_layer_weights* layers,
                       const spiffy_prefix_kv* prefix, const void* w_embed, const void* final_norm,
                       const void* w_vocab, const int32_t* block_tokens, int32_t G, int32_t B, int32_t pos0,
                       const int32_t* graph_edges, int32_t E, int32_t root, float threshold, float logit_scale,
                       int32_t force_one, void* hidden_out, int32_t* argmax, float* conf, uint8_t* unmask,
                       float* top2_margin, int32_t* target_states, spiffy_accept_result* result,
                       int32_t* accepted_state, void* workspace, size_t workspace_bytes, void* stream) {
  int rc;
  if ((rc = check_cfg(cfg)) || (rc = check_gb(G, B))) return rc;
  if (n_layers < 0 || (n_layers > 0 && (!layers || !prefix)) || !w_embed || !workspace || pos0 < 0)
    return SPIFFY_EINVAL;
  if (!aligned16(w_embed) || (hidden_out && !aligned16(hidden_out)) || (reinterpret_cast<uintptr_t>(workspace) & 255u))
    return SPIFFY_EALIGN;
  int P_max = 0;
  for (int l = 0; l < n_layers; ++l) {
    if ((rc = check_layer_args(cfg, &layers[l], &prefix[l], G, B))) return rc;
    if (prefix[l].P + prefix[l].S > P_max) P_max = prefix[l].P + prefix[l].S;
  }
  if ((rc = check_head_args(cfg, workspace, final_norm, w_vocab, block_tokens, threshold, logit_scale, argmax, conf,
                            unmask)))
    return rc;
  const int32_t* tgt_probe = target_states ? target_states : reinterpret_cast<const int32_t*>(workspace);
  if ((rc = check_accept_args(graph_edges, E, block_tokens, tgt_probe, G, B, root, result))) return rc;
  const StepWs ws = carve_step(cfg, G, B, P_max, workspace);
  if (workspace_bytes < ws.bytes) return SPIFFY_EWORKSPACE;

  hipStream_t st = (hipStream_t)stream;
  void* hid = hidden_out ? hidden_out : ws.hidden;
  int32_t* tgt = target_states ? target_states : ws.target;
  LayerChain chain;
  chain.tokens = block_tokens;
  if ((rc = begin_step(cfg, n_layers, layers, w_embed, block_tokens, G, B, nullptr, 0, pos0, 0, hid, !hidden_out, ws.rest, chain, st)))
    return rc;
  if (!hidden_out) {
    const HeadWs hw = carve_head(cfg, G, B, ws.rest);
    chain.final_norm = final_norm;
    chain.head_nf = hw.nf;
    chain.head = HeadRows{hw.row_idx, hw.count};
  }
  for (int l = 0; l < n_layers; ++l) {
    chain.normed_in = chain.normed_out;
    chain.next_norm1 = (l + 1 < n_layers) ? layers[l + 1].norm1 : nullptr;
    // a caller that does not ask for the hidden states gets the last layer on the masked rows only: the head reads
    // nothing else
    chain.masked_rows_only = !hidden_out && l + 1 == n_layers;
    if ((rc = run_layer(cfg, &layers[l], &prefix[l], hid, G, B, pos0, hid, ws.rest, st, &chain))) return rc;
  }
  if ((rc = run_head(cfg, hid, final_norm, w_vocab, block_tokens, nullptr, G, B, threshold, logit_scale, force_one,
                     argmax, conf, unmask, top2_margin, tgt, ws.rest, st, chain.head_ready)))
    return rc;
  return dev(launch_graph_accept(graph_edges, E, block_tokens, tgt, G, B, root, result, accepted_state, st));
}

size_t spiffy_workspace_bytes_seq(const spiffy_model_cfg* cfg, int32_t G, int32_t B, int32_t S, int32_t P_max) {
  if (check_cfg(cfg) || check_gb(G, B) || P_max < 0 || S < 0 || S > SPIFFY_MAX_SUFFIX) return 0;
  return carve_step(cfg, G, B, P_max, nullptr, S).bytes;
}

int spiffy_verify_step_seq(const spiffy_model_cfg* cfg, int32_t n_layers, const spiffy_layer_weights* layers,
                           const spiffy_prefix_kv* prefix, const void* w_embed, const void* final_norm,
                           const void* w_vocab, const int32_t* block_tokens, const int32_t* suffix_tokens, int32_t G,
                           int32_t B, int32_t S, int32_t pos0, const int32_t* graph_edges, int32_t E, int32_t root,
                           float threshold, float logit_scale, int32_t force_one, void* hidden_out, int32_t* argmax,
                           float* conf, uint8_t* unmask, float* top2_margin, int32_t* target_states,
                           spiffy_accept_result* result, int32_t* accepted_state, void* workspace,
                           size_t workspace_bytes, void* stream) {
  int rc;
  if ((rc = check_cfg(cfg)) || (rc = check_gb(G, B))) return rc;
  if (n_layers < 1 || !layers || !prefix || !w_embed || !workspace || pos0 < 0 || S < 0 || (S > 0 && !suffix_tokens))
    return SPIFFY_EINVAL;
  if (S > SPIFFY_MAX_SUFFIX) return SPIFFY_ESHAPE;
  if (!aligned16(w_embed) || (hidden_out && !aligned16(hidden_out)) || (reinterpret_cast<uintptr_t>(workspace) & 255u))
    return SPIFFY_EALIGN;
  int P_max = 0;
  for (int l = 0; l < n_layers; ++l) {
    if ((rc = check_layer_args(cfg, &layers[l], &prefix[l], G, B))) return rc;
    if (prefix[l].S != 0) return SPIFFY_EINVAL;                       // the suffix is computed here, not cached
    if (S > 0) {
      if (!prefix[l].k || !prefix[l].v) return SPIFFY_EINVAL;         // rows behind the prefix are written
      if ((int64_t)prefix[l].P + B + S > prefix[l].capacity) return SPIFFY_ESHAPE;
      if (!layer_mfma(cfg) && attn_limit_bytes(cfg, S, prefix[l].P + B + S) > kAttnLimitBytes) return SPIFFY_ESHAPE;
    }
    if (prefix[l].P > P_max) P_max = prefix[l].P;
  }
  if ((rc = check_head_args(cfg, workspace, final_norm, w_vocab, block_tokens, threshold, logit_scale, argmax, conf,
                            unmask)))
    return rc;
  const int32_t* tgt_probe = target_states ? target_states : reinterpret_cast<const int32_t*>(workspace);
  if ((rc = check_accept_args(graph_edges, E, block_tokens, tgt_probe, G, B, root, result))) return rc;
  const StepWs ws = carve_step(cfg, G, B, P_max, workspace, S);
  if (workspace_bytes < ws.bytes) return SPIFFY_EWORKSPACE;

  hipStream_t st = (hipStream_t)stream;
  void* hid = hidden_out ? hidden_out : ws.hidden;
  int32_t* tgt = target_states ? target_states : ws.target;
  LayerChain chain;
  if ((rc = begin_step(cfg, n_layers, layers, w_embed, block_tokens, G, B, suffix_tokens, S, pos0, pos0 + B, hid, false, ws.rest, chain, st)))
    return rc;
  chain.seq_S = S;
  for (int l = 0; l < n_layers; ++l) {
    chain.normed_in = chain.normed_out;
    chain.next_norm1 = (l + 1 < n_layers) ? layers[l + 1].norm1 : nullptr;
    if ((rc = run_layer(cfg, &layers[l], &prefix[l], hid, G, B, pos0, hid, ws.rest, st, &chain))) return rc;
  }
  if ((rc = run_head(cfg, hid, final_norm, w_vocab, block_tokens, nullptr, G, B, threshold, logit_scale, force_one,
                     argmax, conf, unmask, top2_margin, tgt, ws.rest, st)))
    return rc;
  return dev(launch_graph_accept(graph_edges, E, block_tokens, tgt, G, B, root, result, accepted_state, st));
}

size_t spiffy_workspace_bytes_commit(const spiffy_model_cfg* cfg, int32_t G, int32_t B, int32_t P_max) {
  if (check_cfg(cfg) || check_gb(G, B) || check_gb(G + 1, B) || P_max < 0) return 0;
  return carve_step(cfg, G, B, P_max, nullptr, B).bytes;
}

int spiffy_verify_step_commit(const spiffy_model_cfg* cfg, int32_t n_layers, const spiffy_layer_weights* layers,
                              const spiffy_prefix_kv* prefix, const void* w_embed, const void* final_norm,
                              const void* w_vocab, const int32_t* prev_block_tokens, const int32_t* block_tokens,
                              int32_t G, int32_t B, int32_t pos0, const int32_t* graph_edges, int32_t E, int32_t root,
                              float threshold, float logit_scale, int32_t force_one, void* hidden_out, int32_t* argmax,
                              float* conf, uint8_t* unmask, float* top2_margin, int32_t* target_states,
                              spiffy_accept_result* result, int32_t* accepted_state, void* workspace,
                              size_t workspace_bytes, void* stream) {
  int rc;
  if ((rc = check_cfg(cfg)) || (rc = check_gb(G, B)) || (rc = check_gb(G + 1, B))) return rc;
  if (n_layers < 1 || !layers || !prefix || !w_embed || !workspace || !prev_block_tokens || pos0 < B) return SPIFFY_EINVAL;
  if (!aligned16(w_embed) || (hidden_out && !aligned16(hidden_out)) || (reinterpret_cast<uintptr_t>(workspace) & 255u))
    return SPIFFY_EALIGN;
  int P_max = 0;
  for (int l = 0; l < n_layers; ++l) {
    if ((rc = check_layer_args(cfg, &layers[l], &prefix[l], G, B))) return rc;
    if (!prefix[l].k || !prefix[l].v) return SPIFFY_EINVAL;            // the finished block's rows are written
    const int cap = prefix[l].capacity ? prefix[l].capacity : prefix[l].P;
    if ((int64_t)prefix[l].P + B > cap) return SPIFFY_ESHAPE;
    if (!layer_mfma(cfg) && attn_limit_bytes(cfg, B, prefix[l].P + B + prefix[l].S) > kAttnLimitBytes) return SPIFFY_ESHAPE;
    if (prefix[l].P + prefix[l].S > P_max) P_max = prefix[l].P + prefix[l].S;
  }
  if ((rc = check_head_args(cfg, workspace, final_norm, w_vocab, block_tokens, threshold, logit_scale, argmax, conf,
                            unmask)))
    return rc;
  const int32_t* tgt_probe = target_states ? target_states : reinterpret_cast<const int32_t*>(workspace);
  if ((rc = check_accept_args(graph_edges, E, block_tokens, tgt_probe, G, B, root, result))) return rc;
  const StepWs ws = carve_step(cfg, G, B, P_max, workspace, B);
  if (workspace_bytes < ws.bytes) return SPIFFY_EWORKSPACE;

  hipStream_t st = (hipStream_t)stream;
  void* hid = hidden_out ? hidden_out : ws.hidden;
  int32_t* tgt = target_states ? target_states : ws.target;
  LayerChain chain;
  if ((rc = begin_step(cfg, n_layers, layers, w_embed, block_tokens, G, B, prev_block_tokens, B, pos0, pos0 - B, hid, false, ws.rest, chain, st)))
    return rc;
  chain.seq_S = B;
  chain.tail_is_prev_block = true;
  for (int l = 0; l < n_layers; ++l) {
    chain.normed_in = chain.normed_out;
    chain.next_norm1 = (l + 1 < n_layers) ? layers[l + 1].norm1 : nullptr;
    if ((rc = run_layer(cfg, &layers[l], &prefix[l], hid, G, B, pos0, hid, ws.rest, st, &chain))) return rc;
  }
  if ((rc = run_head(cfg, hid, final_norm, w_vocab, block_tokens, nullptr, G, B, threshold, logit_scale, force_one,
                     argmax, conf, unmask, top2_margin, tgt, ws.rest, st)))
    return rc;
  return dev(launch_graph_accept(graph_edges, E, block_tokens, tgt, G, B, root, result, accepted_state, st));
}

int spiffy_commit_block(const spiffy_model_cfg* cfg, int32_t n_layers, const spiffy_layer_weights* layers,
                        const spiffy_prefix_kv* prefix, const void* w_embed, const int32_t* block_tokens, int32_t B,
                        int32_t pos0, void* workspace, size_t workspace_bytes, void* stream) {
  int rc;
  if ((rc = check_cfg(cfg)) || (rc = check_gb(1, B))) return rc;
  if (n_layers < 1 || !layers || !prefix || !w_embed || !block_tokens || !workspace || pos0 < 0)
    return SPIFFY_EINVAL;
  if (!aligned16(w_embed)) return SPIFFY_EALIGN;
  if (reinterpret_cast<uintptr_t>(workspace) & 255u) return SPIFFY_EALIGN;
  int P_max = 0;
  for (int l = 0; l < n_layers; ++l) {
    if ((rc = check_layer_args(cfg, &layers[l], &prefix[l], 1, B))) return rc;
    if (!prefix[l].k || !prefix[l].v) return SPIFFY_EINVAL;
    const int cap = prefix[l].capacity ? prefix[l].capacity : prefix[l].P;
    if ((int64_t)prefix[l].P + B > cap) return SPIFFY_ESHAPE;      // no room for the block's rows
    if (prefix[l].P + prefix[l].S > P_max) P_max = prefix[l].P + prefix[l].S;
  }
  const StepWs ws = carve_step(cfg, 1, B, P_max, workspace);
  if (workspace_bytes < ws.bytes) return SPIFFY_EWORKSPACE;
  hipStream_t st = (hipStream_t)stream;
  LayerChain chain;
  if ((rc = begin_step(cfg, n_layers, layers, w_embed, block_tokens, 1, B, nullptr, 0, pos0, 0, ws.hidden, false, ws.rest, chain, st)))
    return rc;
  chain.append_kv = true;
  for (int l = 0; l < n_layers; ++l) {
    chain.normed_in = chain.normed_out;
    chain.next_norm1 = (l + 1 < n_layers) ? layers[l + 1].norm1 : nullptr;
    if ((rc = run_layer(cfg, &layers[l], &prefix[l], ws.hidden, 1, B, pos0, ws.hidden, ws.rest, st, &chain))) return rc;
  }
  return SPIFFY_OK;
}

size_t spiffy_subgraph_search_workspace_bytes(void) { return subgraph_search_workspace_bytes(); }

int spiffy_subgraph_search(const int64_t* count, const int32_t* level, int32_t N, const int32_t* edges, int32_t E,
                           int32_t D, uint64_t* best_mask, int64_t* best_sum, uint64_t* n_connected,
                           int32_t* nodes_out, void* workspace, size_t workspace_bytes, void* stream) {
  if (!count || !level || !best_mask || !best_sum || !n_connected || !workspace || (E > 0 && !edges))
    return SPIFFY_EINVAL;
  if (N < 1 || N > 64 || D < 1 || D > 64 || E < 0) return SPIFFY_ESHAPE;
  // a graph whose sets have to be tried one by one: refuse what would run for minutes
  unsigned long long total = 1;
  if (D > N) {
    total = 0;
  } else {
    const int k = D < N - D ? D : N - D;
    for (int i = 1; i <= k; ++i) {
      total = total * (unsigned long long)(N - k + i) / (unsigned long long)i;     // exact: a product of i consecutive integers
      if (total > SPIFFY_SUBGRAPH_MAX_SETS) return SPIFFY_ESHAPE;
    }
  }
  if (reinterpret_cast<uintptr_t>(workspace) & 255u) return SPIFFY_EALIGN;
  if (workspace_bytes < subgraph_search_workspace_bytes()) return SPIFFY_EWORKSPACE;
  SubgraphArgs a;
  a.count = count; a.level = level; a.edges = edges; a.N = N; a.E = E; a.D = D; a.total_sets = total;
  a.best_mask = best_mask; a.best_sum = best_sum; a.n_connected = n_connected; a.nodes_out = nodes_out;
  a.workspace = workspace;
  return dev(launch_subgraph_search(a, (hipStream_t)stream));
}

#pragma GCC visibility pop
}  // extern "C"
