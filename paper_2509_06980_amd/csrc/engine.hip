// Runtime behind the C boundary: weight store, paged KV pool, trajectory records, and the
// sequencing of kernels for the Generate (decode) and Update (append) steps of the paper's
// rollout loop (Section 2.3.2).  Host code only; kernels live in kernels_*.hip.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <cmath>
#include <functional>
#include <queue>
#include <string>
#include <unordered_map>
#include <unordered_set>
#include <vector>

#include "../../include/rl_rollout.h"
#include "kernels.h"

static thread_local std::string g_err;
static int fail(int code, const std::string& msg) {
  g_err = msg;
  return code;
}
extern "C" const char* rl_last_error(void) { return g_err.c_str(); }
int rl_fail(int code, const char* msg) { return fail(code, msg ? msg : ""); }

#define HIPCHECK(expr)                                                                      \
  do {                                                                                      \
    hipError_t e_ = (expr);                                                                 \
    if (e_ != hipSuccess)                                                                   \
      return fail(RL_E_HIP, std::string(#expr) + ": " + hipGetErrorString(e_));             \
  } while (0)

namespace {

struct Traj {
  int slot = -1;
  int n_cached = 0;  // keys / values of tokens[0 .. n_cached) are in the cache
  std::vector<int32_t> tokens;
  std::vector<uint8_t> mask;
  std::vector<float> logp;
  std::vector<int32_t> pages;
  int shared_lead = 0;  // leading pages that were shared with another trajectory by a fork
  uint64_t seen = 0;    // last call that listed it (duplicate check)
};

struct LayerW {
  void *g_in, *wqkv, *gq, *gk, *wo, *g_post, *wgu, *wdown;
};

template <typename T>
static inline T* dptr(void* p) { return (T*)p; }

}  // namespace

struct rl_model {
  rl_model_config cfg{};
  rl_runtime_config rt{};
  ModelDims md{};
  bool bf16 = false, mfma = false;
  size_t el = 4;
  size_t kv_el = 4;        // bytes per cached key / value element (1: 8-bit cache)
  hipStream_t stream = nullptr;
  std::vector<void*> allocs;  // everything to hipFree
  // weights
  void *embed = nullptr, *lm_head = nullptr, *g_final = nullptr;
  std::vector<LayerW> layers;
  float* rope_cs = nullptr;
  // cache
  std::vector<KvPool> pools;
  size_t page_bytes = 0;  // one page of one layer, K (or V) only
  int32_t* page_table = nullptr;
  // work buffers
  int Mcap = 0, Rl = 0, rows_per_item = 1;
  size_t part_rows = 0;    // rows of the split-K partial-sum buffers qkv and ph
  int attn_slots = 0;      // scratch slots for partial attention results
  bool cascade = false;    // shared-prefix decode attention
  float *h = nullptr, *qkv = nullptr, *ph = nullptr, *gu = nullptr, *logits = nullptr, *attn_scratch = nullptr;
  float* ssq = nullptr;    // sums of squares of the residual stream's rows, [H / 16][up to kResidualRows]
  int pending_parts = 0;   // split-K partial sums of the last down-projection still to be added to h
  void *xa = nullptr, *xo = nullptr, *xm = nullptr, *qb = nullptr;
  int32_t *d_meta = nullptr, *h_meta = nullptr;  // device / pinned staging for per-call integers
  size_t meta_ints = 0;
  // page-table entries (slot, index, page) taken by the running call and not yet on the device: they
  // travel with the metadata of the call's first pass (upload_meta), or by themselves at its end
  std::vector<int32_t> page_upd;
  char** d_pools = nullptr;      // [2][n_layers]: every layer's key pool, then every layer's value pool
  uint64_t calls = 0;
  SamplerScratch ss{};
  int32_t* h_ids = nullptr;
  // several decode steps in one call: per-step ids / log-probs on the device and pinned, and one
  // event per group of staging regions (the host runs up to that many steps ahead of the GPU)
  int32_t *d_hist = nullptr, *h_hist = nullptr;      // per step: n ids, then n log-probs
  std::vector<hipEvent_t> ev_region;
  float *d_lp = nullptr, *h_lp = nullptr;
  int32_t* hd_ids = nullptr;   // device addresses of h_ids and h_lp
  float* hd_lp = nullptr;
  float* d_stripmax = nullptr;   // [Rl, V / 32] maxima of 32-logit strips from the lm-head epilogue
  float *d_zt = nullptr, *d_lp_rows = nullptr, *h_lp_rows = nullptr;   // masked log-prob pass: Mcap rows
  uint8_t* d_mask = nullptr;
  // objective pass: per-row old / reference log-probs, use flags and segments (device + pinned
  // staging, the rewards behind them), per-trajectory advantages and accumulators, the result
  float *d_gaux = nullptr, *h_gaux = nullptr;
  double *d_gadv = nullptr, *d_gacc = nullptr, *d_gout = nullptr;
  // host state
  std::unordered_map<int32_t, Traj> traj;
  std::vector<int> free_slots;
  std::priority_queue<int, std::vector<int>, std::greater<int>> free_pages;
  std::vector<int32_t> refcount;
  int64_t n_free = 0;
  // timing
  int timing_every = 0;
  int64_t decode_steps = 0, attn_launches = 0;
  double attn_ms = 0.0, attn_bytes = 0.0, attn_unique_bytes = 0.0, step_gpu_ms = 0.0, step_wall_ms = 0.0;
  int64_t steps_timed = 0;
  hipEvent_t ev_step[2] = {nullptr, nullptr};
  double acct_kv_bytes = 0.0, acct_kv_unique_bytes = 0.0;   // per layer, summed over accounted decode steps
  int64_t acct_steps = 0;
  std::vector<uint32_t> page_stamp;   // per page: last accounted step that counted it
  uint32_t stamp = 0;
  std::vector<hipEvent_t> ev;

  int dalloc(void** p, size_t bytes, bool zero = false) {
    if (bytes == 0) bytes = 16;
    HIPCHECK(hipMalloc(p, bytes));
    allocs.push_back(*p);
    if (zero) HIPCHECK(hipMemset(*p, 0, bytes));
    return RL_OK;
  }
};

namespace {

int round_up(int a, int b) { return (a + b - 1) / b * b; }

// Offsets (in elements) of the blob's tensors.
struct BlobMap {
  size_t embed, g_final, lm_head;
  struct L { size_t g_in, w_q, w_k, w_v, g_q, g_k, w_o, g_post, w_gate, w_up, w_down; };
  std::vector<L> layers;
  size_t total;
};

BlobMap map_blob(const rl_model_config& c) {
  BlobMap m;
  size_t off = 0;
  size_t H = c.hidden, d = c.head_dim, I = c.intermediate, V = c.vocab;
  size_t qw = (size_t)c.n_q_heads * d, kw = (size_t)c.n_kv_heads * d;
  auto take = [&](size_t n) { size_t o = off; off += n; return o; };
  m.embed = take(V * H);
  for (int l = 0; l < c.n_layers; l++) {
    BlobMap::L x;
    x.g_in = take(H); x.w_q = take(qw * H); x.w_k = take(kw * H); x.w_v = take(kw * H);
    x.g_q = take(d); x.g_k = take(d); x.w_o = take(H * qw); x.g_post = take(H);
    x.w_gate = take(I * H); x.w_up = take(I * H); x.w_down = take(H * I);
    m.layers.push_back(x);
  }
  m.g_final = take(H);
  m.lm_head = c.tie_embeddings ? m.embed : take(V * H);
  m.total = off;
  return m;
}

bool mfma_shape_ok(const rl_model_config& c) {
  int g = c.n_q_heads / c.n_kv_heads;
  bool pow2 = g >= 1 && g <= 16 && (g & (g - 1)) == 0;
  int qw = c.n_q_heads * c.head_dim, kvw = c.n_kv_heads * c.head_dim;
  return c.weight_dtype == 1 && c.head_dim == 128 && pow2 && c.hidden % 64 == 0 &&
         c.intermediate % 64 == 0 && qw % 64 == 0 && (qw + 2 * kvw) % 32 == 0 &&
         c.hidden % 32 == 0 && c.vocab % 32 == 0;
}

// ---- one pass of the decoder over M batch rows ----------------------------------------------
// Row metadata (device): tok, pos, slot.  Leaves the residual stream in m->h.
struct RowMeta {
  const int32_t *tok, *pos, *slot;
  const AttnItem* items;
  int n_items;
  const AttnMerge* merges;
  int n_merges;
  const int32_t* rowlist;   // batch rows of the shared-prefix items
  const AttnItem* pf_items; // mixed pass: prefill items of the appended rows behind the decode rows
  int n_pf_items;
  bool prefill;      // multi-row items (append / recompute) instead of single decode rows
  double kv_bytes;   // keys + values the attention of one layer has to read
  bool time_attn;
};

template <typename TW, typename TA>
void forward_generic(rl_model* m, int M, const RowMeta& r) {
  hipStream_t s = m->stream;
  const ModelDims& md = m->md;
  int H = md.H, qw = md.nq * md.d, kvw = md.nkv * md.d, I = md.I;
  launch_embed<TW>(s, (const TW*)m->embed, r.tok, m->h, M, H);
  for (int l = 0; l < md.L; l++) {
    const LayerW& w = m->layers[l];
    launch_rmsnorm<TW, TA>(s, m->h, (const TW*)w.g_in, (TA*)m->xa, M, H, md.eps);
    launch_gemm_generic<TA, TW>(s, (const TA*)m->xa, (const TW*)w.wqkv, m->qkv, M, qw + 2 * kvw, H, false);
    launch_qkrope<TW, TA, TA>(s, m->qkv, (const TW*)w.gq, (const TW*)w.gk, m->rope_cs, r.pos, r.slot,
                              m->page_table, (TA*)m->qb, m->pools[l], md, M);
    if (r.time_attn) (void)hipEventRecord(m->ev[2 * l], s);
    launch_attention_generic<TA, TA>(s, (const TA*)m->qb, m->pools[l], r.pos, r.slot, m->page_table,
                                     (TA*)m->xo, md, M);
    if (r.time_attn) (void)hipEventRecord(m->ev[2 * l + 1], s);
    launch_gemm_generic<TA, TW>(s, (const TA*)m->xo, (const TW*)w.wo, m->h, M, H, qw, true);
    launch_rmsnorm<TW, TA>(s, m->h, (const TW*)w.g_post, (TA*)m->xa, M, H, md.eps);
    launch_gemm_generic<TA, TW>(s, (const TA*)m->xa, (const TW*)w.wgu, m->gu, M, 2 * I, H, false);
    launch_swiglu<TA>(s, m->gu, (TA*)m->xm, M, I);
    launch_gemm_generic<TA, TW>(s, (const TA*)m->xm, (const TW*)w.wdown, m->h, M, H, I, true);
  }
}

// fp32: the norms, the activation and, for few rows and small heads, QK-norm + RoPE + cache write inside the products.
// False where the blob's layout does not give the products whole 16-byte pieces (forward_generic takes those).
bool forward_fp32(rl_model* m, int M, const RowMeta& r) {
  hipStream_t s = m->stream;
  const ModelDims& md = m->md;
  const int H = md.H, qw = md.nq * md.d, QW = qw + 2 * md.nkv * md.d, I = md.I;
  for (const LayerW& w : m->layers)
    if (!norm_gemm32_takes(m->h, w.g_in, w.wqkv, H) || !norm_gemm32_takes(m->h, w.g_post, w.wgu, H)) return false;
  if (((uintptr_t)m->embed & 15) != 0) return false;
  const bool qkv = norm_qkv32_takes(md, M);
  for (int l = 0; l < md.L; l++) {
    const LayerW& w = m->layers[l];
    const int32_t* tok = l == 0 ? r.tok : nullptr;
    if (qkv) {
      launch_norm_qkv32(s, m->h, (const float*)m->embed, tok, (const float*)w.g_in, (const float*)w.wqkv, (const float*)w.gq,
                        (const float*)w.gk, m->rope_cs, r.pos, r.slot, m->page_table, (float*)m->qb, m->pools[l], md, M);
    } else {
      launch_norm_gemm32(s, m->h, (const float*)m->embed, tok, (const float*)w.g_in, (const float*)w.wqkv, m->qkv, M, QW, H, md.eps, false);
      launch_qkrope<float, float, float>(s, m->qkv, (const float*)w.gq, (const float*)w.gk, m->rope_cs, r.pos, r.slot,
                                         m->page_table, (float*)m->qb, m->pools[l], md, M);
    }
    if (r.time_attn) (void)hipEventRecord(m->ev[2 * l], s);
    launch_attention_generic<float, float>(s, (const float*)m->qb, m->pools[l], r.pos, r.slot, m->page_table, (float*)m->xo, md, M);
    if (r.time_attn) (void)hipEventRecord(m->ev[2 * l + 1], s);
    launch_gemm_generic<float, float>(s, (const float*)m->xo, (const float*)w.wo, m->h, M, H, qw, true);
    launch_norm_gemm32(s, m->h, nullptr, nullptr, (const float*)w.g_post, (const float*)w.wgu, (float*)m->xm, M, I, H, md.eps, true);
    launch_gemm_generic<float, float>(s, (const float*)m->xm, (const float*)w.wdown, m->h, M, H, I, true);
  }
  return true;
}

// Rows of the split-K partial-sum buffers: one pass of `cap` rows, and up to kMaxSplits slices of passes of up
// to 1024 rows.  plan_gemm keeps slices times rows within them.
size_t partial_rows(size_t cap) { return std::max<size_t>(cap, (size_t)kMaxSplits * std::min<size_t>(cap, 1024)); }

// The products of one pass over M rows, the same for every layer.
struct PassPlan {
  GemmPlan q, o, g, d;      // QKV, O, gate-up, down
  bool fused_qkv;           // QK-norm, RoPE and the cache write in the epilogue of QKV
  int eo, ed;               // epilogues of O and down: EPI_ADD or EPI_STORE
  ResidualPlan ro, rd;      // rb > 0: O / down with the residual add and the next norm instead
};
PassPlan plan_pass(const ModelDims& md, int M, size_t part_rows) {
  const int H = md.H, qw = md.nq * md.d, QW = qw + 2 * md.nkv * md.d, I = md.I;
  PassPlan p;
  p.q = plan_gemm(M, QW, H, EPI_STORE, part_rows);
  p.o = plan_gemm(M, H, qw, EPI_STORE, part_rows);
  p.g = plan_gemm(M, 2 * I, H, EPI_SWIGLU, part_rows);
  p.d = plan_gemm(M, H, I, EPI_STORE, part_rows);
  // Norm, RoPE and cache write inside the projection where that is expected to pay.  Per million values of the
  // projection the separate kernel takes 1.6 us (a bit less with the 8-bit cache) and 0.5 us more for every further
  // K-slice that it adds, the epilogue 0.55 us; 4.5 and 3 to 4.5 us come on top.  The remaining constants make up for
  // what the estimates of the two products are off by (128 x 256 tiles: 0.45 us per million values).  Fitted on 8 shapes
  // (1280 to 12288 columns, hidden 512 to 5120), 129 to 8192 rows and both caches: the slower way is taken
  // in 8 of 124 cases, by more than 3 % in two (12288 columns, 1300 rows: 171 against 164 us); with a cost by rows
  // alone it was in 12, by up to 15 % (12288 columns, 300 rows: 80.5 against 70.3 us; 6144 columns of hidden 4096,
  // 3072 rows: 172.2 against 160.7 us).
  const GemmPlan pf = plan_gemm(M, QW, H, EPI_QKV, 0);
  const double mval = 1e-6 * M * QW;
  p.fused_qkv = (pf.kind == GEMM_TILE256 || pf.kind == GEMM_WIDE128) &&
                pf.cost + (pf.kind == GEMM_WIDE128 ? 0.45 : 0.0) * mval <=
                    p.q.cost + 2.0 + (1.0 + 0.65 * (p.q.splits - 1)) * mval;
  if (p.fused_qkv) p.q = pf;
  // the residual add inside the products that leave one partial sum (the norm then reads one array instead
  // of two and writes none back)
  auto adds = [](const GemmPlan& g) { return g.splits == 1 && (g.kind == GEMM_TILE256 || g.kind == GEMM_WIDE128); };
  p.eo = adds(p.o) ? EPI_ADD : EPI_STORE;
  p.ed = adds(p.d) ? EPI_ADD : EPI_STORE;
  // With the residual add and the norm inside where that is expected to be faster than the product and the norm's launch
  // (3.6 us and 0.45 us per 1024 columns; the product's estimate holds the partial sums that the norm reads).  Of the last
  // layer's down the launch stays, without partial sums to read: there the two ways are about equal (hidden 1024 at 64 rows
  // 5.2 + 3.1 against 4.8 + 4.4 us), and one plan serves all layers.
  // Above 128 rows every part on its own, `consumer` the division in gate-up or in the norm / RoPE kernel: the product's
  // estimate is 3 us too high there (its own kernels are told apart by differences), the norm takes its launch and the
  // traffic of its partial sums, its looping form for more than 4096 columns 5 us more.  With the rule of few rows 300 to 512
  // rows of hidden 2048 and more had lost up to 8.5 us a layer (hidden 4096, intermediate 1024, 448 rows: 97 -> 105 us).
  // Fitted on 18 shapes of hidden 512 to 5120, 131 to 512 rows: of the 193 products that took the inside way by the old rule
  // two still do and are slower (by 1.5 and 2 us), six no longer do and would be faster (by at most 1 us).
  auto residual = [&](const GemmPlan& g, int K, double consumer) {
    const ResidualPlan r = plan_residual(M, H, K);
    const double mh = 1e-6 * M * H;
    const bool pays = M <= 128 ? r.cost < g.cost + 3.6 + 4.5e-4 * H
                               : r.cost + consumer + 0.5 < 0.95 * g.cost + 0.4 + 5.2e-4 * H + (0.74 + 0.5 * g.splits) * mh + (H > 4096 ? 5.0 : 0.0);
    return r.rb > 0 && pays ? r : ResidualPlan{0, 0, 0.0};
  };
  const double mh = 1e-6 * M * H;
  p.ro = gate_up_takes_scale(p.g, M, H) ? residual(p.o, qw, 0.75 + 9.1e-4 * H + 0.18 * mh) : ResidualPlan{0, 0, 0.0};
  p.rd = p.fused_qkv ? ResidualPlan{0, 0, 0.0} : residual(p.d, I, 0.88 + 1.3e-4 * H + 0.7 * mh);
  return p;
}

// Leaves the last down-projection as m->pending_parts partial sums in m->ph (added by the next
// add_rmsnorm: the next layer's, or the final norm before the lm-head).
void forward_mfma(rl_model* m, int M, const RowMeta& r) {
  hipStream_t s = m->stream;
  const ModelDims& md = m->md;
  int H = md.H, qw = md.nq * md.d, kvw = md.nkv * md.d, I = md.I, QW = qw + 2 * kvw;
  const PassPlan plan = plan_pass(md, M, m->part_rows);
  float *const co = plan.eo == EPI_ADD ? m->h : m->ph, *const cd = plan.ed == EPI_ADD ? m->h : m->ph;
  // norm, RoPE and the cache write inside the attention: decode rows alone, none of them through a shared-prefix item
  const bool rope_inside = !plan.fused_qkv && !r.prefill && r.n_pf_items == 0 && !m->cascade && attention_takes_rope(r.kv_bytes, md);
  int pend = 0;
  const float *so_q = nullptr, *so_g;       // sums of squares, where the norm's division is left to the consumer
  for (int l = 0; l < md.L; l++) {
    const LayerW& w = m->layers[l];
    // (the last layer's rows with the final gains are read by nobody: the lm-head's own norm gathers the rows it needs from h)
    const bf16_t* g_next = (const bf16_t*)(l + 1 < md.L ? m->layers[l + 1].g_in : m->g_final);
    if (l == 0) launch_embed_rmsnorm(s, (const bf16_t*)m->embed, r.tok, m->h, (const bf16_t*)w.g_in, (bf16_t*)m->xa, M, H, md.eps);
    else if (!so_q) launch_add_rmsnorm(s, m->h, m->ph, pend, (size_t)M * H, (const bf16_t*)w.g_in, (bf16_t*)m->xa, M, H, md.eps);
    RopeArgs rope{};
    if (plan.fused_qkv) {
      const QkvArgs qa{(const bf16_t*)w.gq, (const bf16_t*)w.gk, m->rope_cs, r.pos, r.slot, m->page_table,
                       (bf16_t*)m->qb, m->pools[l].k, m->pools[l].v, md.nq, md.nkv, md.qk_norm,
                       md.max_pages_per_traj, md.eps};
      launch_gemm_qkv(s, (const bf16_t*)m->xa, (const bf16_t*)w.wqkv, M, QW, H, md.kv_fp8 != 0, plan.q, qa);
    } else {
      int sq = launch_gemm_mfma(s, (const bf16_t*)m->xa, (const bf16_t*)w.wqkv, m->qkv, M, QW, H, EPI_STORE, plan.q);
      rope = RopeArgs{m->qkv, sq, (size_t)M * QW, (const bf16_t*)w.gq, (const bf16_t*)w.gk, m->rope_cs, md.nq, md.nkv, md.qk_norm, md.eps,
                      so_q, H / 16, (M + 15) / 16 * 16, H};
      if (!rope_inside) launch_qkrope128(s, rope, r.pos, r.slot, m->page_table, (bf16_t*)m->qb, m->pools[l], md, M);
    }
    if (r.time_attn) (void)hipEventRecord(m->ev[2 * l], s);
    launch_attention_mfma(s, (const bf16_t*)m->qb, m->pools[l], r.items, r.n_items, r.merges, r.n_merges,
                          r.rowlist, m->page_table, (bf16_t*)m->xo, m->attn_scratch, md, r.prefill, rope_inside ? &rope : nullptr);
    if (r.n_pf_items > 0)
      launch_attention_mfma(s, (const bf16_t*)m->qb, m->pools[l], r.pf_items, r.n_pf_items, nullptr, 0,
                            nullptr, m->page_table, (bf16_t*)m->xo, m->attn_scratch, md, true);
    if (r.time_attn) (void)hipEventRecord(m->ev[2 * l + 1], s);
    if (plan.ro.rb > 0) {
      launch_gemm_residual(s, (const bf16_t*)m->xo, (const bf16_t*)w.wo, m->h, (const bf16_t*)w.g_post, (bf16_t*)m->xa, m->ssq, M, H, qw, plan.ro);
      so_g = m->ssq;
    } else {
      int so = launch_gemm_mfma(s, (const bf16_t*)m->xo, (const bf16_t*)w.wo, co, M, H, qw, plan.eo, plan.o);
      launch_add_rmsnorm(s, m->h, m->ph, so, (size_t)M * H, (const bf16_t*)w.g_post, (bf16_t*)m->xa, M, H, md.eps);
      so_g = nullptr;
    }
    launch_gemm_mfma(s, (const bf16_t*)m->xa, (const bf16_t*)w.wgu, m->xm, M, 2 * I, H, EPI_SWIGLU, plan.g, so_g, md.eps);
    if (plan.rd.rb > 0) {
      launch_gemm_residual(s, (const bf16_t*)m->xm, (const bf16_t*)w.wdown, m->h, g_next, (bf16_t*)m->xa, m->ssq, M, H, I, plan.rd);
      so_q = m->ssq;
      pend = 0;
    } else {
      pend = launch_gemm_mfma(s, (const bf16_t*)m->xm, (const bf16_t*)w.wdown, cd, M, H, I, plan.ed, plan.d);
    }
  }
  m->pending_parts = pend;
}

void forward_rows(rl_model* m, int M, const RowMeta& r) {
  if (m->mfma) forward_mfma(m, M, r);
  else if (m->bf16) forward_generic<bf16_t, bf16_t>(m, M, r);
  else if (!forward_fp32(m, M, r)) forward_generic<float, float>(m, M, r);
}

// Where a step that draws leaves the maxima of its logits' strips; null where the sampler would not read them.
float* drawn_maxima(const rl_model* m, bool drawn) {
  return m->mfma && drawn && sampler_reads_maxima(m->logits, (size_t)m->md.V, m->md.V, false) ? m->d_stripmax : nullptr;
}

// final norm + lm-head for rows [r0, r0 + R) of m->h -> m->logits[0 .. R)
// M: rows of the forward pass (stride of its partial sums); norm_rows <= M: leading rows to normalise
// drawn: a token is drawn from every row (on the MFMA path the kernel is then the same for every row count, and the
// logits' per-strip maxima are left in m->d_stripmax where the sampler reads them)
void lm_head_rows(rl_model* m, int M, int r0, int R, bool norm_done, int norm_rows = -1,
                  bool drawn = false) {
  hipStream_t s = m->stream;
  const ModelDims& md = m->md;
  if (norm_rows < 0) norm_rows = M;
  if (m->mfma) {
    if (!norm_done) {
      launch_add_rmsnorm(s, m->h, m->ph, m->pending_parts, (size_t)M * md.H, (const bf16_t*)m->g_final,
                         (bf16_t*)m->xa, norm_rows, md.H, md.eps);
      m->pending_parts = 0;
    }
    // r0 is a multiple of 128: skip whole A tiles
    if (drawn) {
      launch_lm_head_logits(s, (const bf16_t*)m->xa + (size_t)r0 * md.H, (const bf16_t*)m->lm_head,
                            m->logits, R, md.V, md.H, drawn_maxima(m, true));
    } else {
      launch_gemm_mfma(s, (const bf16_t*)m->xa + (size_t)r0 * md.H, (const bf16_t*)m->lm_head, m->logits,
                       R, md.V, md.H, EPI_STORE, plan_gemm(R, md.V, md.H, EPI_STORE, 0));
    }
  } else if (m->bf16) {
    if (!norm_done)
      launch_rmsnorm<bf16_t, bf16_t>(s, m->h, (const bf16_t*)m->g_final, (bf16_t*)m->xa, norm_rows, md.H, md.eps);
    launch_gemm_generic<bf16_t, bf16_t>(s, (const bf16_t*)m->xa + (size_t)r0 * md.H,
                                        (const bf16_t*)m->lm_head, m->logits, R, md.V, md.H, false);
  } else if (!norm_done && r0 == 0 && R == norm_rows && norm_gemm32_takes(m->h, m->g_final, m->lm_head, md.H)) {
    launch_norm_gemm32(s, m->h, nullptr, nullptr, (const float*)m->g_final, (const float*)m->lm_head, m->logits, R, md.V, md.H, md.eps, false);
  } else {
    if (!norm_done)
      launch_rmsnorm<float, float>(s, m->h, (const float*)m->g_final, (float*)m->xa, norm_rows, md.H, md.eps);
    launch_gemm_generic<float, float>(s, (const float*)m->xa + (size_t)r0 * md.H,
                                      (const float*)m->lm_head, m->logits, R, md.V, md.H, false);
  }
}

// ---- per-call metadata staging ----------------------------------------------------------------
// Layout of the integer staging buffer for a pass over M rows:
//   [0,M) tok  [M,2M) pos  [2M,3M) slot  [3M,4M) traj id  [4M,5M) index of the new token
//   [5M,6M) forced / target ids  [6M, ...) attention items (8 ints each), merge records (8 ints
//   each), then the row list of the shared-prefix items
struct Staging {
  std::vector<int32_t> tok, pos, slot, traj, newpos, forced;
  std::vector<AttnItem> items;
  std::vector<AttnMerge> merges;
  std::vector<uint8_t> mask;
  std::vector<int32_t> rowlist;
  void clear() { tok.clear(); pos.clear(); slot.clear(); traj.clear(); newpos.clear(); forced.clear(); items.clear(); merges.clear(); mask.clear(); rowlist.clear(); }
};

struct DevMeta {
  int32_t *tok, *pos, *slot, *traj, *newpos, *forced;
  AttnItem* items;
  AttnMerge* merges;
  int32_t* rowlist;
};

int check_pass(rl_model* m, const Staging& st, int slots_used);
int flush_page_updates(rl_model* m);

// Fills the staging buffer of one pass from offset `at` (in ints) on; *used: ints that have to be copied from there.
int stage_meta(rl_model* m, const Staging& st, DevMeta* dm, size_t at, size_t* used) {
  size_t M = st.tok.size();
  {
    int slots = 0;
    for (const AttnItem& it : st.items) slots = std::max(slots, it.part + 1);
    int crc = check_pass(m, st, slots);
    if (crc) return crc;
  }
  static_assert(sizeof(AttnItem) == 32 && sizeof(AttnMerge) == 32, "metadata records are 8 ints");
  const size_t need = 6 * M + 8 * st.items.size() + 8 * st.merges.size() + st.rowlist.size();
  if (at + need > m->meta_ints) return fail(RL_E_ARG, "internal: metadata staging too small");
  int32_t* h = m->h_meta + at;
  int32_t* d = m->d_meta + at;
  auto put = [&](const std::vector<int32_t>& v, size_t at) {
    if (!v.empty()) memcpy(h + at, v.data(), v.size() * 4);
  };
  put(st.tok, 0); put(st.pos, M); put(st.slot, 2 * M); put(st.traj, 3 * M); put(st.newpos, 4 * M);
  put(st.forced, 5 * M);
  if (!st.items.empty()) memcpy(h + 6 * M, st.items.data(), st.items.size() * sizeof(AttnItem));
  if (!st.merges.empty())
    memcpy(h + 6 * M + 8 * st.items.size(), st.merges.data(), st.merges.size() * sizeof(AttnMerge));
  put(st.rowlist, 6 * M + 8 * st.items.size() + 8 * st.merges.size());
  dm->tok = d; dm->pos = d + M; dm->slot = d + 2 * M;
  dm->traj = d + 3 * M; dm->newpos = d + 4 * M; dm->forced = d + 5 * M;
  dm->items = (AttnItem*)(d + 6 * M);
  dm->merges = (AttnMerge*)(d + 6 * M + 8 * st.items.size());
  dm->rowlist = d + 6 * M + 8 * st.items.size() + 8 * st.merges.size();
  *used = need;
  return RL_OK;
}
int copy_meta(rl_model* m, size_t at, size_t n) {
  HIPCHECK(hipMemcpyAsync(m->d_meta + at, m->h_meta + at, n * 4, hipMemcpyHostToDevice, m->stream));
  return RL_OK;
}

// The metadata of a pass and the pending page-table entries -> device.
int upload_meta(rl_model* m, const Staging& st, DevMeta* dm) {
  size_t need = 0;
  int rc = stage_meta(m, st, dm, 0, &need);
  if (rc) return rc;
  if (!m->page_upd.empty() && need + m->page_upd.size() > m->meta_ints) {
    rc = flush_page_updates(m);            // through the staging buffer, which is then filled again
    if (!rc) rc = stage_meta(m, st, dm, 0, &need);
    if (rc) return rc;
  }
  const size_t n_upd = m->page_upd.size();
  if (n_upd > 0) memcpy(m->h_meta + need, m->page_upd.data(), n_upd * 4);
  rc = copy_meta(m, 0, need + n_upd);
  if (rc) return rc;
  if (n_upd > 0) {
    launch_page_table_update(m->stream, m->page_table, m->d_meta + need, (int)(n_upd / 3), m->md.max_pages_per_traj);
    m->page_upd.clear();
  }
  if (!st.mask.empty())
    HIPCHECK(hipMemcpyAsync(m->d_mask, st.mask.data(), st.mask.size(), hipMemcpyHostToDevice, m->stream));
  return RL_OK;
}

// the page-table entries that no pass has taken along -> device, in batches through the staging buffer
int flush_page_updates(rl_model* m) {
  size_t n = m->page_upd.size() / 3, done = 0;
  size_t cap = m->meta_ints / 3;
  while (done < n) {
    size_t k = std::min(cap, n - done);
    memcpy(m->h_meta, m->page_upd.data() + 3 * done, k * 12);
    HIPCHECK(hipMemcpyAsync(m->d_meta, m->h_meta, k * 12, hipMemcpyHostToDevice, m->stream));
    launch_page_table_update(m->stream, m->page_table, m->d_meta, (int)k, m->md.max_pages_per_traj);
    HIPCHECK(hipStreamSynchronize(m->stream));
    done += k;
  }
  m->page_upd.clear();
  return RL_OK;
}

int take_page(rl_model* m) {
  int p = m->free_pages.top();
  m->free_pages.pop();
  m->refcount[p] = 1;
  m->n_free--;
  return p;
}
void drop_page(rl_model* m, int p) {
  if (--m->refcount[p] == 0) {
    m->free_pages.push(p);
    m->n_free++;
  }
}

int check_ids(const int32_t* ids, int32_t n) {
  if (n < 0 || (n > 0 && !ids)) return fail(RL_E_ARG, "null ids or negative count");
  std::unordered_set<int32_t> seen;
  for (int i = 0; i < n; i++)
    if (ids[i] < 0) return fail(RL_E_ARG, "negative trajectory id");
  for (int i = 0; i < n; i++)
    if (!seen.insert(ids[i]).second) return fail(RL_E_DUP_ID, "duplicate trajectory id");
  return RL_OK;
}

// The listed trajectories, each looked up once.  Unknown or repeated ids take the full check, which
// decides the error code.
int find_trajs(rl_model* m, const int32_t* ids, int32_t n, std::vector<Traj*>* out) {
  if (n < 0 || (n > 0 && !ids)) return fail(RL_E_ARG, "null ids or negative count");
  const uint64_t call = ++m->calls;
  out->resize(n);
  for (int i = 0; i < n; i++) {
    auto it = ids[i] < 0 ? m->traj.end() : m->traj.find(ids[i]);
    if (it == m->traj.end() || it->second.seen == call) {
      int rc = check_ids(ids, n);
      return rc ? rc : RL_E_BAD_TRAJ;
    }
    it->second.seen = call;
    (*out)[i] = &it->second;
  }
  return RL_OK;
}

// attention work items for `cnt` consecutive rows of one trajectory starting at batch row row0
// (chunked prefill: every item covers all pages up to its last row, one part)
void add_items(rl_model* m, Staging& st, int row0, int cnt, int slot, int pos0) {
  int R = m->rows_per_item;
  for (int a = 0; a < cnt; a += R) {
    int nr = std::min(R, cnt - a);
    st.items.push_back(AttnItem{row0 + a, nr, slot, pos0 + a, 0, (pos0 + a + nr - 1) / RL_PAGE + 1, -1, 0});
  }
}

// Decode items: one row per trajectory.  Contexts are cut into parts of about equal page count where
// that pays (see below); a part gets at least 8 pages (ragged batches: 16).
// Shared-prefix ("cascade") mode: trajectories of the step whose leading pages are the same physical
// pages (a forked group) get those pages read once per 16/G members by a gather item; each member
// then covers only its own remainder and a merge record joins the two.
const int kAttnTargetWgs = 1024;
const int kMinSharedPages = 8;
// Sizes of buffers that a model of this many trajectories gets (n_kv_heads 0: not on the MFMA path, no scratch for parts).
const int kDefaultBatchRows = 8192;
int row_capacity(int max_batch_rows, int max_trajectories) {
  return round_up(std::max(max_batch_rows ? max_batch_rows : kDefaultBatchRows, max_trajectories), 128);
}
int attention_slots(int n_kv_heads, int max_trajectories) { return n_kv_heads ? kAttnTargetWgs / n_kv_heads + 3 * max_trajectories + 64 : 0; }
size_t staging_ints(int max_batch_rows, int max_trajectories) { return 32 * (size_t)row_capacity(max_batch_rows, max_trajectories) + 3 * 65536; }
int add_decode_items(rl_model* m, Staging& st, const std::vector<Traj*>& ts) {   // returns scratch slots used
  int n = (int)st.pos.size();
  const int rpb = std::max(1, 16 / (m->md.nq / m->md.nkv));   // member rows per gather item
  // own_lo[i]: first page the row reads by itself; shared part records per row
  std::vector<int> own_lo(n, 0), sfirst(n, 0), snparts(n, 0), srow(n, 0);
  struct Block { std::vector<int> rows; int pages; };
  std::vector<Block> blocks;
  if (m->cascade && m->mfma) {
    std::unordered_map<int32_t, std::vector<int>> by_first;
    for (int i = 0; i < n; i++)
      if (!ts[i]->pages.empty() && m->refcount[ts[i]->pages[0]] > 1) by_first[ts[i]->pages[0]].push_back(i);
    std::vector<int32_t> keys;
    for (auto& kv : by_first) if (kv.second.size() >= 2) keys.push_back(kv.first);
    std::sort(keys.begin(), keys.end());                 // deterministic order of the groups
    for (int32_t k : keys) {
      const std::vector<int>& rows = by_first[k];
      const std::vector<int32_t>& p0 = ts[rows[0]]->pages;
      int common = INT32_MAX;
      for (int i : rows) {
        const std::vector<int32_t>& pi = ts[i]->pages;
        int lim = std::min({st.pos[i] / RL_PAGE, (int)pi.size(), (int)p0.size()});   // pages wholly before the row's position
        int c = 0;
        while (c < lim && pi[c] == p0[c]) c++;
        common = std::min(common, c);
      }
      if (common < kMinSharedPages) continue;
      for (size_t a = 0; a < rows.size(); a += rpb) {
        Block b;
        for (size_t j = a; j < std::min(rows.size(), a + rpb); j++) b.rows.push_back(rows[j]);
        if (b.rows.size() < 2) continue;                 // a lone member reads its pages directly
        b.pages = common;
        for (int i : b.rows) own_lo[i] = common;
        blocks.push_back(std::move(b));
      }
    }
  }
  int64_t total_pages = 0;
  for (int i = 0; i < n; i++) total_pages += st.pos[i] / RL_PAGE + 1 - own_lo[i];
  for (auto& b : blocks) total_pages += b.pages;
  // Contexts of about equal length: the number of parts that a cost estimate finds cheapest.  With W
  // workgroups (one per part and kv head) on 256 CUs, R = ceil(W / 256) of them share a CU and the
  // launch lasts as long as a CU needs for its R parts: per 16-token page and kv head 0.18 us where a
  // workgroup has its CU to itself (0.205 us shared; 8-bit cache 0.135 / 0.12), or the page's share
  // of the bandwidth when all CUs stream (0.31 us, 0.165), plus 8.3 us for the launch (10.7 with the
  // merge) and 3 us for every further part on a CU.  Fitted on the 4B shape at 1 to 48 trajectories
  // and contexts of 200 to 8000 tokens, in each of which it is within a few percent of the best of
  // eight cuts (1 x 800: 17.8 -> 12.2 us against no cut, 4 x 8000: 38.1 -> 31.5 and 16 x 8000: 96.7
  // -> 87.4 against shares for 1024 workgroups).
  int pages_max = 0;
  for (int i = 0; i < n; i++) pages_max = std::max(pages_max, st.pos[i] / RL_PAGE + 1 - own_lo[i]);
  for (auto& b : blocks) pages_max = std::max(pages_max, b.pages);
  const int nkv = m->md.nkv, n_items = n + (int)blocks.size();
  const bool alike = (int64_t)pages_max * n_items * 2 <= total_pages * 3;   // longest <= 1.5 x average
  int chunk;
  if (alike) {
    chunk = std::max(16, pages_max);
    const double t_own = m->md.kv_fp8 ? 0.135 : 0.18, t_shared = m->md.kv_fp8 ? 0.12 : 0.205;
    const double t_all = m->md.kv_fp8 ? 0.165 : 0.31;
    double best = 0.0;
    // parts for at most ~kAttnTargetWgs workgroups, of at least 8 pages
    const int pmax = m->mfma ? std::max(1, std::min(kAttnTargetWgs / (n_items * nkv), pages_max / 8)) : 1;
    for (int p = 1; p <= pmax; p++) {
      const int c = p == 1 ? std::max(16, pages_max) : std::max(8, (pages_max + p - 1) / p);
      int64_t W = 0;
      for (int i = 0; i < n; i++) W += (st.pos[i] / RL_PAGE + 1 - own_lo[i] + c - 1) / c;
      for (auto& b : blocks) W += (b.pages + c - 1) / c;
      W *= nkv;
      const int64_t R = (W + 255) / 256;
      const double t = std::max(R > 1 ? t_shared : t_own, t_all * (double)W / (256.0 * R));
      const double cost = (p == 1 ? 8.3 : 10.7) + 3.0 * (R - 1) + R * c * t;
      if (p == 1 || cost < best) { best = cost; chunk = c; }
    }
  } else {
    // ragged lengths: even shares; with 512 or more (trajectory, kv head) pairs only what is
    // longer than twice the average is cut
    const int target_wgs = (int64_t)n * m->md.nkv >= 512 ? 512 : kAttnTargetWgs;
    chunk = (int)std::max<int64_t>(16, (total_pages * m->md.nkv + target_wgs - 1) / target_wgs);
  }
  int next_part = 0;
  for (auto& b : blocks) {
    int parts = (b.pages + chunk - 1) / chunk;
    int per = (b.pages + parts - 1) / parts;
    int row0 = (int)st.rowlist.size();
    for (size_t j = 0; j < b.rows.size(); j++) {
      int i = b.rows[j];
      st.rowlist.push_back(i);
      sfirst[i] = next_part;
      snparts[i] = parts;
      srow[i] = (int)j;
    }
    for (int k = 0; k < parts; k++)
      st.items.push_back(AttnItem{row0, (int)b.rows.size(), st.slot[b.rows[0]], 0, k * per,
                                  std::min((k + 1) * per, b.pages), next_part++, (b.pages << 8) | 1});
  }
  for (int i = 0; i < n; i++) {
    int np = st.pos[i] / RL_PAGE + 1;
    int own = np - own_lo[i];
    int parts = m->mfma ? (own + chunk - 1) / chunk : 1;
    if (parts <= 1 && snparts[i] == 0) {
      st.items.push_back(AttnItem{i, 1, st.slot[i], st.pos[i], 0, np, -1, ts[i]->shared_lead << 8});
      continue;
    }
    int per = (own + parts - 1) / parts;
    st.merges.push_back(AttnMerge{i, next_part, parts, sfirst[i], snparts[i], srow[i], 0, 0});
    for (int k = 0; k < parts; k++)
      st.items.push_back(AttnItem{i, 1, st.slot[i], st.pos[i], own_lo[i] + k * per,
                                  std::min(own_lo[i] + (k + 1) * per, np), next_part++, ts[i]->shared_lead << 8});
  }
  return next_part;
}

// Host-side bounds of one forward pass, checked before anything is launched: a planning mistake
// must surface as an error code, never as an out-of-bounds access on the GPU.
int check_pass(rl_model* m, const Staging& st, int slots_used) {
  const size_t M = st.tok.size();
  if (M > (size_t)m->Mcap) return fail(RL_E_ARG, "internal: pass exceeds the row capacity");
  if (m->mfma && slots_used > m->attn_slots) return fail(RL_E_ARG, "internal: attention scratch too small");
  if (st.pos.size() != M || st.slot.size() != M) return fail(RL_E_ARG, "internal: row metadata mismatch");
  const int maxp = m->md.max_pages_per_traj;
  for (size_t i = 0; i < M; i++)
    if (st.pos[i] < 0 || st.pos[i] / RL_PAGE >= maxp || st.slot[i] < 0 || st.slot[i] >= m->rt.max_trajectories)
      return fail(RL_E_ARG, "internal: row position / slot out of range");
  for (const AttnItem& it : st.items) {
    const bool gather = it.gather & 1;
    if (it.nrows < 1 || it.pg_lo < 0 || it.pg_hi > maxp || it.pg_lo > it.pg_hi || it.slot < 0 ||
        it.slot >= m->rt.max_trajectories || it.part >= m->attn_slots ||
        (gather ? (size_t)(it.row0 + it.nrows) > st.rowlist.size() : (size_t)(it.row0 + it.nrows) > M))
      return fail(RL_E_ARG, "internal: attention item out of range");
  }
  for (int r : st.rowlist)
    if (r < 0 || (size_t)r >= M) return fail(RL_E_ARG, "internal: row list out of range");
  for (const AttnMerge& mg : st.merges)
    if (mg.row < 0 || (size_t)mg.row >= M || mg.first < 0 || mg.first + mg.nparts > m->attn_slots ||
        mg.sfirst < 0 || mg.sfirst + mg.snparts > m->attn_slots)
      return fail(RL_E_ARG, "internal: merge record out of range");
  return RL_OK;
}

// Chunked prefill of tokens[n_cached .. upto) for the listed trajectories (upto given per traj).
int prefill(rl_model* m, const std::vector<std::pair<Traj*, int>>& work) {
  Staging st;
  int cap = m->rt.max_batch_rows;
  size_t wi = 0;
  int cur = work.empty() ? 0 : work[0].first->n_cached;
  while (wi < work.size()) {
    st.clear();
    while (wi < work.size() && (int)st.tok.size() < cap) {
      Traj* t = work[wi].first;
      int upto = work[wi].second;
      if (cur >= upto) {
        t->n_cached = std::max(t->n_cached, upto);
        wi++;
        if (wi < work.size()) cur = work[wi].first->n_cached;
        continue;
      }
      int take = std::min(upto - cur, cap - (int)st.tok.size());
      add_items(m, st, (int)st.tok.size(), take, t->slot, cur);
      for (int p = cur; p < cur + take; p++) {
        st.tok.push_back(t->tokens[p]);
        st.pos.push_back(p);
        st.slot.push_back(t->slot);
      }
      cur += take;
    }
    int M = (int)st.tok.size();
    if (M == 0) break;
    DevMeta dm;
    int rc = upload_meta(m, st, &dm);
    if (rc) return rc;
    RowMeta r{dm.tok, dm.pos, dm.slot, dm.items, (int)st.items.size(), dm.merges, 0, dm.rowlist, nullptr, 0, true, 0.0, false};
    forward_rows(m, M, r);
    HIPCHECK(hipGetLastError());
    HIPCHECK(hipStreamSynchronize(m->stream));
  }
  return RL_OK;
}

// extra: trajectories whose freshly appended tokens [n_cached, upto) still have to be prefilled.
// Their rows ride behind the decode rows of the same forward pass (the weights are streamed once
// for both); if they do not fit into one pass they are prefilled first, on their own.
// *extra_done tells the caller whether that has happened when the function returns.
int decode_impl(rl_model* m, const int32_t* ids, int32_t n, float temperature, uint64_t seed,
                const int32_t* forced, int32_t* ids_out, float* lp_out,
                const std::vector<std::pair<Traj*, int>>* extra, bool* extra_done) {
  std::vector<Traj*> ts;
  int rc = find_trajs(m, ids, n, &ts);
  if (rc && rc != RL_E_BAD_TRAJ) return rc;
  if (!(temperature >= 0.0f)) return fail(RL_E_ARG, "negative temperature");
  if (n > 0 && !lp_out) return fail(RL_E_ARG, "null output");
  if (n > m->rt.max_trajectories || rc) return fail(RL_E_BAD_TRAJ, "unknown trajectory id");
  for (Traj* t : ts)
    if (t->tokens.empty()) return fail(RL_E_EMPTY, "trajectory has no context");
  if (forced)
    for (int i = 0; i < n; i++)
      if (forced[i] < 0 || forced[i] >= m->cfg.vocab) return fail(RL_E_BAD_TOKEN, "forced token out of range");
  int64_t need = 0;
  for (Traj* t : ts) {
    if ((int)t->tokens.size() + 1 > m->rt.max_context) return fail(RL_E_CTX_OVERFLOW, "context overflow");
    if (t->tokens.size() % RL_PAGE == 0) need++;
  }
  if (need > m->n_free) return fail(RL_E_NOPAGES, "page pool exhausted");
  if (n == 0) return RL_OK;
  // appended rows that ride along: they must fit into this pass together with the decode rows
  int extra_rows = 0;
  if (extra)
    for (auto& w : *extra) extra_rows += std::max(0, w.second - w.first->n_cached);
  if (extra && !extra->empty() && n + extra_rows > m->Mcap) {
    rc = prefill(m, *extra);
    *extra_done = true;
    if (rc) return rc;
    extra = nullptr;
    extra_rows = 0;
  }
  // commit page reservations (call order), then compute
  for (Traj* t : ts)
    if (t->tokens.size() % RL_PAGE == 0) {
      int p = take_page(m);
      m->page_upd.insert(m->page_upd.end(), {t->slot, (int32_t)t->pages.size(), p});
      t->pages.push_back(p);
    }
  Staging st;
  int max_pos = 0;
  double kvb = 0.0;
  for (int i = 0; i < n; i++) {
    Traj* t = ts[i];
    int nt = (int)t->tokens.size();
    st.tok.push_back(t->tokens[nt - 1]);
    st.pos.push_back(nt - 1);
    st.slot.push_back(t->slot);
    st.traj.push_back(ids[i]);
    st.newpos.push_back(nt);
    if (forced) st.forced.push_back(forced[i]);
    max_pos = std::max(max_pos, nt - 1);
    kvb += (double)nt * 2.0 * m->md.nkv * m->md.d * m->kv_el;
  }
  add_decode_items(m, st, ts);
  const int n_dec_items = (int)st.items.size();
  if (extra_rows > 0) {   // prefill rows behind the decode rows, prefill items behind the decode items
    for (auto& w : *extra) {
      Traj* t = w.first;
      int cur = t->n_cached, upto = w.second;
      if (cur >= upto) continue;
      add_items(m, st, (int)st.tok.size(), upto - cur, t->slot, cur);
      for (int p = cur; p < upto; p++) {
        st.tok.push_back(t->tokens[p]);
        st.pos.push_back(p);
        st.slot.push_back(t->slot);
      }
    }
    st.traj.resize(st.tok.size(), 0);
    st.newpos.resize(st.tok.size(), 0);
    if (forced) st.forced.resize(st.tok.size(), 0);
  }
  const int M = (int)st.tok.size();
  DevMeta dm;
  rc = upload_meta(m, st, &dm);
  if (rc) return rc;
  if (extra) {
    for (auto& w : *extra) w.first->n_cached = std::max(w.first->n_cached, w.second);
    *extra_done = true;
  }
  // mixed passes are left out of the kernel timing: its byte counts describe pure decode steps
  bool timed = extra_rows == 0 && m->timing_every > 0 && (m->decode_steps % m->timing_every) == 0;
  m->decode_steps++;
  double kvu = 0.0;
  RowMeta r{dm.tok, dm.pos, dm.slot, dm.items, n_dec_items, dm.merges, (int)st.merges.size(),
            dm.rowlist, dm.items + n_dec_items, (int)st.items.size() - n_dec_items, false, kvb, timed};
  if (timed) (void)hipEventRecord(m->ev_step[0], m->stream);
  forward_rows(m, M, r);
  bool greedy = temperature == 0.0f;
  // sampling needs the row maximum before any weight can be formed: the lm-head epilogue leaves the
  // maximum of every 32-logit strip, so no separate pass over the logits looks for it (the arg-max
  // of a greedy step still takes that pass)
  lm_head_rows(m, M, 0, n, false, n, !greedy);
  float c = sampler_scale(temperature);
  launch_sampler(m->stream, m->logits, (size_t)m->md.V, n, m->md.V, c, greedy ? 1 : 0, nullptr, seed,
                 dm.traj, dm.newpos, forced ? dm.forced : nullptr, nullptr, m->ss, m->hd_ids, m->hd_lp,
                 drawn_maxima(m, !greedy), m->md.V / 32);       // ids and log-probs go straight to the pinned host buffers
  HIPCHECK(hipGetLastError());
  if (timed) (void)hipEventRecord(m->ev_step[1], m->stream);
  if (m->timing_every > 0 && extra_rows == 0) {
    // byte accounting of pure decode steps, done while the GPU works: keys + values per trajectory,
    // and of the distinct pages (pages shared by forked trajectories count once)
    if (m->page_stamp.size() != m->refcount.size()) m->page_stamp.assign(m->refcount.size(), 0);
    m->stamp++;
    const double tokb = 2.0 * m->md.nkv * m->md.d * m->kv_el;
    for (Traj* t : ts) {
      const int nt = (int)t->tokens.size();
      for (int pg = 0; pg * RL_PAGE < nt; pg++) {
        const int page = t->pages[pg];
        if (m->page_stamp[page] == m->stamp) continue;
        m->page_stamp[page] = m->stamp;
        kvu += tokb * std::min(RL_PAGE, nt - pg * RL_PAGE);
      }
    }
    m->acct_kv_bytes += kvb;
    m->acct_kv_unique_bytes += kvu;
    m->acct_steps++;
  }
  HIPCHECK(hipStreamSynchronize(m->stream));
  if (timed) {
    float sms = 0.f;
    if (hipEventElapsedTime(&sms, m->ev_step[0], m->ev_step[1]) == hipSuccess) {
      m->step_gpu_ms += sms;
      m->steps_timed++;
    }
    for (int l = 0; l < m->md.L; l++) {
      float ms = 0.f;
      if (hipEventElapsedTime(&ms, m->ev[2 * l], m->ev[2 * l + 1]) == hipSuccess) {
        m->attn_ms += ms;
        m->attn_launches++;
        m->attn_bytes += kvb;
        m->attn_unique_bytes += kvu;
      }
    }
  }
  for (int i = 0; i < n; i++) {
    Traj* t = ts[i];
    t->n_cached = (int)t->tokens.size();
    t->tokens.push_back(m->h_ids[i]);
    t->mask.push_back(0);
    t->logp.push_back(m->h_lp[i]);
    if (ids_out) ids_out[i] = m->h_ids[i];
    lp_out[i] = m->h_lp[i];
  }
  return RL_OK;
}

// Several decode steps of one list of trajectories in one call.  The result is that of n_steps
// single steps; the difference is in the timing: the token a step samples stays on the device and
// feeds the next step's embedding lookup there, the metadata of the steps is staged in regions of
// the staging buffers, and the host runs up to one region per step ahead of the GPU instead of
// waiting for every step's ids.  Pages for the whole call are reserved up front, in the order the
// single steps would have taken them.
const int kMaxStepsPerChunk = 1024, kStepsPerCopy = 8;

// How the staging buffer is shared out over the steps of such a call.  flush: its page-table entries go over first, on their own and
// waited for, instead of in front of the regions.  group: steps whose metadata goes over in one copy, packed into the front
// of their regions (the first step's alone, with the entries, so that the GPU starts at once); regions: a multiple of it.
// A small fp32 rollout (51 passes) takes 3.17 ms in groups of eight; with a copy and an event per step, a wait for the
// entries and two copies at the end it took 3.50.  Two groups at least, so that one is filled while the GPU works on the other's
// steps; and where the entries would leave room for fewer regions than that takes they go first, which costs tens of us a call
// whose steps have hundreds of rows.
struct StagingPlan { bool flush; int regions, group; };
size_t staging_region_ints(int n, int attn_slots) { return 7 * (size_t)n + 8 * (size_t)(2 * n + attn_slots + 8); }
StagingPlan plan_staging(size_t meta_ints, size_t region_ints, size_t entry_ints) {
  auto fit = [&](size_t taken) { return taken >= meta_ints ? 0 : (int)std::min<size_t>((meta_ints - taken) / region_ints, 64); };
  StagingPlan p{};
  p.flush = entry_ints > meta_ints / 4 || fit(entry_ints) < std::min(fit(0), 2 * kStepsPerCopy);
  p.regions = fit(p.flush ? 0 : entry_ints);
  p.group = std::max(1, std::min(kStepsPerCopy, p.regions / 2));
  p.regions -= p.regions % p.group;
  return p;
}

int decode_multi(rl_model* m, const int32_t* ids, int32_t n, int32_t n_steps, float temperature,
                 uint64_t seed, int32_t* ids_out, float* lp_out) {
  std::vector<Traj*> ts;
  int rc = find_trajs(m, ids, n, &ts);
  if (rc && rc != RL_E_BAD_TRAJ) return rc;
  if (n_steps < 0) return fail(RL_E_ARG, "negative step count");
  if (!(temperature >= 0.0f)) return fail(RL_E_ARG, "negative temperature");
  if (n > 0 && n_steps > 0 && (!ids_out || !lp_out)) return fail(RL_E_ARG, "null output");
  if (n > m->rt.max_trajectories || rc) return fail(RL_E_BAD_TRAJ, "unknown trajectory id");
  for (Traj* t : ts)
    if (t->tokens.empty()) return fail(RL_E_EMPTY, "trajectory has no context");
  int64_t need = 0;
  for (Traj* t : ts) {
    const int64_t after = (int64_t)t->tokens.size() + n_steps;
    if (after > m->rt.max_context) return fail(RL_E_CTX_OVERFLOW, "context overflow");
    need += (after + RL_PAGE - 1) / RL_PAGE - (int64_t)t->pages.size();
  }
  if (need > m->n_free) return fail(RL_E_NOPAGES, "page pool exhausted");
  if (n == 0 || n_steps == 0) return RL_OK;
  // one staging region per step, behind the page-table entries of the call; the host may run as many steps ahead as there are regions
  const size_t region_ints = staging_region_ints(n, m->attn_slots);
  const StagingPlan plan = plan_staging(m->meta_ints, region_ints, m->page_upd.size() + 3 * (size_t)need);
  if (plan.regions < 1) return fail(RL_E_ARG, "internal: metadata staging too small");
  {
    std::vector<size_t> len0(n);
    for (int i = 0; i < n; i++) len0[i] = ts[i]->tokens.size();
    for (int sidx = 0; sidx < n_steps; sidx++)
      for (int i = 0; i < n; i++)
        if ((len0[i] + sidx) % RL_PAGE == 0) {
          Traj* t = ts[i];
          int p = take_page(m);
          m->page_upd.insert(m->page_upd.end(), {t->slot, (int32_t)t->pages.size(), p});
          t->pages.push_back(p);
        }
  }
  if (plan.flush) {
    rc = flush_page_updates(m);
    if (rc) return rc;
  }
  const size_t n_upd = m->page_upd.size(), regions_at = n_upd;
  const int group = plan.group, n_regions = plan.regions;
  while ((int)m->ev_region.size() < n_regions / group) {
    hipEvent_t e = nullptr;
    HIPCHECK(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    m->ev_region.push_back(e);
  }
  const bool greedy = temperature == 0.0f;
  const float c = sampler_scale(temperature);
  const double tokb = 2.0 * m->md.nkv * m->md.d * m->kv_el;
  Staging st;
  for (int s0 = 0; s0 < n_steps; s0 += kMaxStepsPerChunk) {
    const int C = std::min(kMaxStepsPerChunk, n_steps - s0);
    std::vector<int> len0(n);
    for (int i = 0; i < n; i++) len0[i] = (int)ts[i]->tokens.size();
    struct StepMeta { DevMeta dm; int n_items, n_merges; double kvb; };
    std::vector<StepMeta> staged;          // of the steps from first_staged on
    int first_staged = 0;
    for (int sc = 0; sc < C; sc++) {
      const int region = sc % n_regions;
      if (sc == first_staged + (int)staged.size()) {
        staged.clear();
        first_staged = sc;
        const int k = std::min(sc == 0 ? 1 : group - sc % group, C - sc);
        // the steps that used this group's regions before are over when the last of them is
        if (sc >= n_regions) HIPCHECK(hipEventSynchronize(m->ev_region[region / group]));
        const size_t at = regions_at + (size_t)region * region_ints;
        size_t filled = 0;
        for (int j = sc; j < sc + k; j++) {
          st.clear();
          double kvb = 0.0;
          for (int i = 0; i < n; i++) {
            const int nt = len0[i] + j;               // context length at this step
            st.tok.push_back(j == 0 ? ts[i]->tokens[nt - 1] : 0);    // later steps: the id sampled on the device
            st.pos.push_back(nt - 1);
            st.slot.push_back(ts[i]->slot);
            st.traj.push_back(ids[i]);
            st.newpos.push_back(nt);
            kvb += (double)nt * tokb;
          }
          add_decode_items(m, st, ts);
          StepMeta sm{{}, (int)st.items.size(), (int)st.merges.size(), kvb};
          size_t used = 0;
          if (6 * (size_t)n + 8 * st.items.size() + 8 * st.merges.size() + st.rowlist.size() > region_ints)
            return fail(RL_E_ARG, "internal: staging region too small");
          rc = stage_meta(m, st, &sm.dm, at + filled, &used);
          if (rc) return rc;
          filled += used;
          staged.push_back(sm);
        }
        const bool entries = !m->page_upd.empty();
        if (entries) memcpy(m->h_meta, m->page_upd.data(), n_upd * 4);
        rc = entries ? copy_meta(m, 0, at + filled) : copy_meta(m, at, filled);
        if (rc) return rc;
        if (entries) {
          launch_page_table_update(m->stream, m->page_table, m->d_meta, (int)(n_upd / 3), m->md.max_pages_per_traj);
          m->page_upd.clear();
        }
      }
      const DevMeta& dm = staged[sc - first_staged].dm;
      const int n_items = staged[sc - first_staged].n_items, n_merges = staged[sc - first_staged].n_merges;
      const double kvb = staged[sc - first_staged].kvb;
      const bool timed = m->timing_every > 0 && (m->decode_steps % m->timing_every) == 0;
      m->decode_steps++;
      const int32_t* tok = sc == 0 ? dm.tok : m->d_hist + (size_t)(sc - 1) * 2 * n;
      RowMeta r{tok, dm.pos, dm.slot, dm.items, n_items, dm.merges, n_merges,
                dm.rowlist, nullptr, 0, false, kvb, timed};
      if (timed) (void)hipEventRecord(m->ev_step[0], m->stream);
      forward_rows(m, n, r);
      lm_head_rows(m, n, 0, n, false, n, !greedy);
      launch_sampler(m->stream, m->logits, (size_t)m->md.V, n, m->md.V, c, greedy ? 1 : 0, nullptr, seed,
                     dm.traj, dm.newpos, nullptr, nullptr, m->ss, m->d_hist + (size_t)sc * 2 * n,
                     (float*)(m->d_hist + (size_t)(2 * sc + 1) * n), drawn_maxima(m, !greedy), m->md.V / 32);
      HIPCHECK(hipGetLastError());
      if (timed) (void)hipEventRecord(m->ev_step[1], m->stream);
      if ((region + 1) % group == 0) HIPCHECK(hipEventRecord(m->ev_region[region / group], m->stream));
      double kvu = 0.0;
      if (m->timing_every > 0) {    // byte accounting, while the GPU works (as in the single step)
        if (m->page_stamp.size() != m->refcount.size()) m->page_stamp.assign(m->refcount.size(), 0);
        m->stamp++;
        for (int i = 0; i < n; i++) {
          const int nt = len0[i] + sc;
          for (int pg = 0; pg * RL_PAGE < nt; pg++) {
            const int page = ts[i]->pages[pg];
            if (m->page_stamp[page] == m->stamp) continue;
            m->page_stamp[page] = m->stamp;
            kvu += tokb * std::min(RL_PAGE, nt - pg * RL_PAGE);
          }
        }
        m->acct_kv_bytes += kvb;
        m->acct_kv_unique_bytes += kvu;
        m->acct_steps++;
      }
      if (timed) {    // a timed step is waited for: its events are read before they are reused
        HIPCHECK(hipStreamSynchronize(m->stream));
        float sms = 0.f;
        if (hipEventElapsedTime(&sms, m->ev_step[0], m->ev_step[1]) == hipSuccess) {
          m->step_gpu_ms += sms;
          m->steps_timed++;
        }
        for (int l = 0; l < m->md.L; l++) {
          float ms = 0.f;
          if (hipEventElapsedTime(&ms, m->ev[2 * l], m->ev[2 * l + 1]) == hipSuccess) {
            m->attn_ms += ms;
            m->attn_launches++;
            m->attn_bytes += kvb;
            m->attn_unique_bytes += kvu;
          }
        }
      }
    }
    HIPCHECK(hipMemcpyAsync(m->h_hist, m->d_hist, (size_t)C * 2 * n * 4, hipMemcpyDeviceToHost, m->stream));
    HIPCHECK(hipStreamSynchronize(m->stream));
    for (int sc = 0; sc < C; sc++)
      for (int i = 0; i < n; i++) {
        Traj* t = ts[i];
        const int32_t id = m->h_hist[(size_t)sc * 2 * n + i];
        float lp;
        memcpy(&lp, m->h_hist + (size_t)(2 * sc + 1) * n + i, 4);
        t->tokens.push_back(id);
        t->mask.push_back(0);
        t->logp.push_back(lp);
        ids_out[(size_t)(s0 + sc) * n + i] = id;
        lp_out[(size_t)(s0 + sc) * n + i] = lp;
      }
    for (Traj* t : ts) t->n_cached = (int)t->tokens.size() - 1;
  }
  return RL_OK;
}

int decode_common(rl_model* m, const int32_t* ids, int32_t n, float temperature, uint64_t seed,
                  const int32_t* forced, int32_t* ids_out, float* lp_out,
                  const std::vector<std::pair<Traj*, int>>* extra = nullptr) {
  bool extra_done = false;
  int rc = decode_impl(m, ids, n, temperature, seed, forced, ids_out, lp_out, extra, &extra_done);
  if (extra && !extra->empty() && !extra_done) {
    // the decode part failed validation (or was empty): the append part still takes effect
    std::string msg = g_err;
    int prc = prefill(m, *extra);
    if (rc == RL_OK) rc = prc; else g_err = msg;
  }
  if (!m->page_upd.empty()) {
    std::string msg = g_err;
    int urc = flush_page_updates(m);
    if (rc == RL_OK) rc = urc; else g_err = msg;
  }
  return rc;
}

}  // namespace

// =============================================================================================
extern "C" int rl_model_load(const rl_runtime_config* rt, const void* weights, size_t nbytes,
                             rl_model** out) {
  if (!rt || !weights || !out || nbytes < 64) return fail(RL_E_ARG, "null argument or short blob");
  const unsigned char* b = (const unsigned char*)weights;
  uint32_t version;
  memcpy(&version, b + 4, 4);
  if (memcmp(b, "RLW1", 4) != 0 || version != 1) return fail(RL_E_ARG, "bad blob magic / version");
  rl_model_config c;
  memcpy(&c, b + 8, sizeof(c));
  if (c.n_layers <= 0 || c.hidden <= 0 || c.n_q_heads <= 0 || c.n_kv_heads <= 0 || c.head_dim <= 0 ||
      c.intermediate <= 0 || c.vocab <= 0 || c.n_q_heads % c.n_kv_heads != 0 || c.head_dim % 2 != 0 ||
      (c.weight_dtype != 0 && c.weight_dtype != 1))
    return fail(RL_E_ARG, "bad model config");
  if (c.head_dim > 128) return fail(RL_E_ARG, "head_dim above 128 is not supported");
  if (c.weight_dtype == 1 && (c.hidden % 16 != 0 || c.intermediate % 16 != 0))
    return fail(RL_E_ARG, "bf16 models need hidden and intermediate to be multiples of 16");
  if (rt->page_tokens != RL_PAGE || rt->max_context <= 0 || rt->max_trajectories <= 0 ||
      rt->kv_pool_pages < 0 || rt->kv_pool_pages > 0x7fffffff || rt->max_batch_rows < 0)
    return fail(RL_E_ARG, "bad runtime config");
  BlobMap bm = map_blob(c);
  size_t el = c.weight_dtype == 1 ? 2 : 4;
  if (nbytes != 64 + bm.total * el) return fail(RL_E_ARG, "blob size does not match its header");

  rl_model* m = new rl_model();
  m->cfg = c;
  m->rt = *rt;
  if (m->rt.max_batch_rows == 0) m->rt.max_batch_rows = kDefaultBatchRows;
  m->bf16 = c.weight_dtype == 1;
  m->el = el;
  m->mfma = m->bf16 && mfma_shape_ok(c) && !(rt->flags & RL_FLAG_GENERIC_KERNELS);
  m->cascade = (rt->flags & RL_FLAG_SHARED_PREFIX_ATTENTION) != 0;
  const bool kv_fp8 = (rt->flags & RL_FLAG_FP8_KV_CACHE) != 0;
  if (kv_fp8 && !m->mfma) {
    delete m;
    return fail(RL_E_ARG, "the 8-bit cache needs a bf16 model on the MFMA kernels (head_dim 128)");
  }
  m->kv_el = kv_fp8 ? 1 : el;
  int max_pages = (rt->max_context + RL_PAGE - 1) / RL_PAGE;
  m->md = ModelDims{c.n_layers, c.hidden, c.n_q_heads, c.n_kv_heads, c.head_dim, c.intermediate,
                    c.vocab, c.rms_eps, c.qk_norm, max_pages, kv_fp8 ? 1 : 0};
  // prefill items: 4 waves of kPrefillColumns columns
  m->rows_per_item = m->mfma ? 4 * (kPrefillColumns / (c.n_q_heads / c.n_kv_heads)) : 1;
  int rc = RL_OK;
#define TRY(x) do { rc = (x); if (rc) { rl_model_free(m); return rc; } } while (0)
#define HIPTRY(x) do { hipError_t e_ = (x); if (e_ != hipSuccess) { fail(RL_E_HIP, std::string(#x) + ": " + hipGetErrorString(e_)); rl_model_free(m); return RL_E_HIP; } } while (0)
  HIPTRY(hipStreamCreate(&m->stream));
  HIPTRY((hipError_t)sampler_noalloc_prepare());
  // ---- weights ----
  int H = c.hidden, d = c.head_dim, I = c.intermediate, V = c.vocab;
  int qw = c.n_q_heads * d, kvw = c.n_kv_heads * d;
  char* raw = nullptr;  // device copy of the tensor area
  HIPTRY(hipMalloc((void**)&raw, bm.total * el));
  hipError_t ce = hipMemcpy(raw, b + 64, bm.total * el, hipMemcpyHostToDevice);
  if (ce != hipSuccess) { (void)hipFree(raw); fail(RL_E_HIP, "weight upload failed"); rl_model_free(m); return RL_E_HIP; }
  auto at = [&](size_t off) { return (void*)(raw + off * el); };
  m->layers.resize(c.n_layers);
  if (!m->mfma) {
    m->allocs.push_back(raw);  // keep the blob image, point into it
    m->embed = at(bm.embed); m->g_final = at(bm.g_final); m->lm_head = at(bm.lm_head);
    for (int l = 0; l < c.n_layers; l++) {
      const BlobMap::L& x = bm.layers[l];
      m->layers[l] = LayerW{at(x.g_in), at(x.w_q), at(x.g_q), at(x.g_k), at(x.w_o), at(x.g_post),
                            at(x.w_gate), at(x.w_down)};
    }
  } else {
    auto fin = [&](int code) { (void)hipFree(raw); return code; };
    auto keep = [&](void** dst, size_t off, size_t n) -> int {
      int r2 = m->dalloc(dst, n * 2);
      if (r2) return r2;
      if (hipMemcpyAsync(*dst, at(off), n * 2, hipMemcpyDeviceToDevice, m->stream) != hipSuccess)
        return fail(RL_E_HIP, "device copy failed");
      return RL_OK;
    };
    auto pack = [&](void** dst, size_t off, size_t off_u, int N, int K, bool il) -> int {
      int r2 = m->dalloc(dst, (size_t)N * K * 2);
      if (r2) return r2;
      launch_repack_weight(m->stream, (const bf16_t*)at(off), (const bf16_t*)at(off_u), (bf16_t*)*dst, N, K, il);
      return RL_OK;
    };
    int r2 = keep(&m->embed, bm.embed, (size_t)V * H);
    if (!r2) r2 = keep(&m->g_final, bm.g_final, H);
    if (!r2) r2 = pack(&m->lm_head, bm.lm_head, 0, V, H, false);
    for (int l = 0; l < c.n_layers && !r2; l++) {
      const BlobMap::L& x = bm.layers[l];
      LayerW& w = m->layers[l];
      r2 = keep(&w.g_in, x.g_in, H);
      if (!r2) r2 = keep(&w.gq, x.g_q, d);
      if (!r2) r2 = keep(&w.gk, x.g_k, d);
      if (!r2) r2 = keep(&w.g_post, x.g_post, H);
      if (!r2) r2 = pack(&w.wqkv, x.w_q, 0, qw + 2 * kvw, H, false);
      if (!r2) r2 = pack(&w.wo, x.w_o, 0, H, qw, false);
      if (!r2) r2 = pack(&w.wgu, x.w_gate, x.w_up, 2 * I, H, true);
      if (!r2) r2 = pack(&w.wdown, x.w_down, 0, H, I, false);
    }
    if (!r2 && (hipStreamSynchronize(m->stream) != hipSuccess || hipGetLastError() != hipSuccess))
      r2 = fail(RL_E_HIP, "weight repack failed");
    fin(0);
    if (r2) { rl_model_free(m); return r2; }
  }
  // ---- RoPE table: cos/sin(pos * theta^(-2i/d)), computed in double ----
  {
    int half = d / 2;
    std::vector<float> cs((size_t)rt->max_context * half * 2);
    for (int i = 0; i < half; i++) {
      double inv = pow((double)c.rope_theta, -2.0 * i / d);
      for (int p = 0; p < rt->max_context; p++) {
        double a = (double)p * inv;
        cs[((size_t)p * half + i) * 2] = (float)cos(a);
        cs[((size_t)p * half + i) * 2 + 1] = (float)sin(a);
      }
    }
    TRY(m->dalloc((void**)&m->rope_cs, cs.size() * 4));
    HIPTRY(hipMemcpy(m->rope_cs, cs.data(), cs.size() * 4, hipMemcpyHostToDevice));
  }
  // ---- KV pool ----
  m->page_bytes = (size_t)c.n_kv_heads * RL_PAGE * d * m->kv_el;
  if (m->rt.kv_pool_pages == 0) {
    // automatic size: a page for every token of every trajectory at max_context, capped by 85 % of
    // the device memory that is free now (the work buffers below come out of the rest)
    size_t free_b = 0, total_b = 0;
    HIPTRY(hipMemGetInfo(&free_b, &total_b));
    const double per_page = 2.0 * (double)m->page_bytes * c.n_layers;
    const int64_t want = (int64_t)rt->max_trajectories * max_pages;
    const int64_t fit = (int64_t)(0.85 * (double)free_b / per_page);
    m->rt.kv_pool_pages = std::min<int64_t>(std::min(want, fit), 0x7fffffff);
    if (m->rt.kv_pool_pages <= 0) {
      fail(RL_E_HIP, "no device memory left for the KV page pool");
      rl_model_free(m);
      return RL_E_HIP;
    }
  }
  const int64_t pool_pages = m->rt.kv_pool_pages;
  m->pools.resize(c.n_layers);
  for (int l = 0; l < c.n_layers; l++) {
    TRY(m->dalloc(&m->pools[l].k, m->page_bytes * pool_pages, true));
    TRY(m->dalloc(&m->pools[l].v, m->page_bytes * pool_pages, true));
  }
  TRY(m->dalloc((void**)&m->page_table, (size_t)rt->max_trajectories * max_pages * 4, true));
  m->refcount.assign(pool_pages, 0);
  for (int p = 0; p < pool_pages; p++) m->free_pages.push(p);
  m->n_free = pool_pages;
  for (int s = rt->max_trajectories - 1; s >= 0; s--) m->free_slots.push_back(s);
  // ---- work buffers ----
  m->Mcap = row_capacity(m->rt.max_batch_rows, rt->max_trajectories);
  m->Rl = round_up(std::max(rt->max_trajectories, 256), 128);
  size_t Mc = m->Mcap;
  size_t ael = m->bf16 ? 2 : 4;
  TRY(m->dalloc((void**)&m->h, Mc * H * 4, true));
  const size_t prow = m->mfma ? partial_rows(Mc) : Mc;
  m->part_rows = prow;
  TRY(m->dalloc((void**)&m->qkv, prow * (qw + 2 * kvw) * 4, true));
  if (m->mfma) TRY(m->dalloc((void**)&m->ph, prow * H * 4, true));
  if (m->mfma) TRY(m->dalloc((void**)&m->ssq, (size_t)kResidualRows * (H / 16) * 4));
  TRY(m->dalloc(&m->xa, Mc * H * ael, true));
  TRY(m->dalloc(&m->xo, Mc * qw * ael, true));
  TRY(m->dalloc(&m->xm, Mc * I * ael, true));
  TRY(m->dalloc(&m->qb, Mc * qw * ael, true));
  if (!m->mfma) TRY(m->dalloc((void**)&m->gu, Mc * 2 * I * 4, true));
  TRY(m->dalloc((void**)&m->logits, (size_t)m->Rl * V * 4));
  if (m->mfma) {
    m->attn_slots = attention_slots(c.n_kv_heads, rt->max_trajectories);
    TRY(m->dalloc((void**)&m->attn_scratch,   // one slot per part of a cut decode row
                  (size_t)m->attn_slots * c.n_kv_heads * 16 * 130 * 4));
  }
  int nseg = sampler_nseg(V);
  TRY(m->dalloc((void**)&m->ss.segmax, (size_t)m->Rl * nseg * 4));
  TRY(m->dalloc((void**)&m->ss.segarg, (size_t)m->Rl * nseg * 4));
  TRY(m->dalloc((void**)&m->ss.segw, (size_t)m->Rl * nseg * 8));
  TRY(m->dalloc((void**)&m->ss.sege, (size_t)m->Rl * nseg * 4));
  if (m->mfma) TRY(m->dalloc((void**)&m->d_stripmax, (size_t)m->Rl * (V / 32) * 4));
  TRY(m->dalloc((void**)&m->d_hist, (size_t)kMaxStepsPerChunk * m->Rl * 8));
  HIPTRY(hipHostMalloc((void**)&m->h_hist, (size_t)kMaxStepsPerChunk * m->Rl * 8));
  TRY(m->dalloc((void**)&m->d_lp, (size_t)m->Rl * 4));
  TRY(m->dalloc((void**)&m->d_mask, Mc));
  TRY(m->dalloc((void**)&m->d_zt, Mc * 4));
  TRY(m->dalloc((void**)&m->d_lp_rows, Mc * 4));
  {
    size_t T = (size_t)rt->max_trajectories;
    TRY(m->dalloc((void**)&m->d_gaux, (3 * Mc + 4 * T + 4) * 4));
    TRY(m->dalloc((void**)&m->d_gadv, T * 8));
    TRY(m->dalloc((void**)&m->d_gacc, 3 * T * 8));
    TRY(m->dalloc((void**)&m->d_gout, 3 * 8));
    HIPTRY(hipHostMalloc((void**)&m->h_gaux, (3 * Mc + 4 * T + 4) * 4));
  }
  m->meta_ints = staging_ints(m->rt.max_batch_rows, rt->max_trajectories);
  TRY(m->dalloc((void**)&m->d_meta, m->meta_ints * 4));
  HIPTRY(hipHostMalloc((void**)&m->h_meta, m->meta_ints * 4));
  HIPTRY(hipHostMalloc((void**)&m->h_ids, (size_t)m->Rl * 4));
  HIPTRY(hipHostMalloc((void**)&m->h_lp, (size_t)m->Rl * 4));
  HIPTRY(hipHostMalloc((void**)&m->h_lp_rows, Mc * 4));
  HIPTRY(hipHostGetDevicePointer((void**)&m->hd_ids, m->h_ids, 0));
  HIPTRY(hipHostGetDevicePointer((void**)&m->hd_lp, m->h_lp, 0));
  {
    std::vector<char*> base;
    for (int l = 0; l < c.n_layers; l++) base.push_back((char*)m->pools[l].k);
    for (int l = 0; l < c.n_layers; l++) base.push_back((char*)m->pools[l].v);
    TRY(m->dalloc((void**)&m->d_pools, base.size() * sizeof(char*)));
    HIPTRY(hipMemcpy(m->d_pools, base.data(), base.size() * sizeof(char*), hipMemcpyHostToDevice));
  }
  m->ev.resize(2 * c.n_layers);
  for (auto& e : m->ev) HIPTRY(hipEventCreate(&e));
  HIPTRY(hipEventCreate(&m->ev_step[0]));
  HIPTRY(hipEventCreate(&m->ev_step[1]));
  HIPTRY(hipDeviceSynchronize());
#undef TRY
#undef HIPTRY
  *out = m;
  return RL_OK;
}

extern "C" void rl_model_free(rl_model* m) {
  if (!m) return;
  if (m->stream) (void)hipStreamSynchronize(m->stream);
  for (void* p : m->allocs) (void)hipFree(p);
  if (m->h_meta) (void)hipHostFree(m->h_meta);
  if (m->h_ids) (void)hipHostFree(m->h_ids);
  if (m->h_hist) (void)hipHostFree(m->h_hist);
  for (auto e : m->ev_region) if (e) (void)hipEventDestroy(e);
  if (m->h_lp) (void)hipHostFree(m->h_lp);
  if (m->h_lp_rows) (void)hipHostFree(m->h_lp_rows);
  if (m->h_gaux) (void)hipHostFree(m->h_gaux);
  for (auto e : m->ev) if (e) (void)hipEventDestroy(e);
  for (auto e : m->ev_step) if (e) (void)hipEventDestroy(e);
  if (m->stream) (void)hipStreamDestroy(m->stream);
  delete m;
}

extern "C" int rl_model_get_config(const rl_model* m, rl_model_config* out) {
  if (!m || !out) return fail(RL_E_ARG, "null argument");
  *out = m->cfg;
  return RL_OK;
}

// Host part of an append: validation, token / mask bookkeeping, page reservation and page-table
// update.  On success *work lists the trajectories whose new tokens still need their keys / values.
static int append_host(rl_model* m, const int32_t* traj_ids, int32_t n, const int32_t* tokens,
                       const int32_t* lens, std::vector<std::pair<Traj*, int>>* work_out) {
  if (!m) return fail(RL_E_ARG, "null model");
  int rc = check_ids(traj_ids, n);
  if (rc) return rc;
  if (n > 0 && !lens) return fail(RL_E_ARG, "null lens");
  int64_t total = 0;
  for (int i = 0; i < n; i++) {
    if (lens[i] < 0) return fail(RL_E_ARG, "negative length");
    total += lens[i];
  }
  if (total > 0 && !tokens) return fail(RL_E_ARG, "null tokens");
  for (int64_t i = 0; i < total; i++)
    if (tokens[i] < 0 || tokens[i] >= m->cfg.vocab) return fail(RL_E_BAD_TOKEN, "token id out of range");
  int64_t need = 0;
  int n_new = 0;
  for (int i = 0; i < n; i++) {
    auto it = m->traj.find(traj_ids[i]);
    int64_t cur = it == m->traj.end() ? 0 : (int64_t)it->second.tokens.size();
    if (it == m->traj.end()) n_new++;
    if (cur + lens[i] > m->rt.max_context) return fail(RL_E_CTX_OVERFLOW, "context overflow");
    need += (cur + lens[i] + RL_PAGE - 1) / RL_PAGE - (cur + RL_PAGE - 1) / RL_PAGE;
  }
  if ((int64_t)m->traj.size() + n_new > m->rt.max_trajectories)
    return fail(RL_E_TOO_MANY, "too many trajectories");
  if (need > m->n_free) return fail(RL_E_NOPAGES, "page pool exhausted");
  // commit
  std::vector<std::pair<Traj*, int>> work;
  int64_t off = 0;
  for (int i = 0; i < n; i++) {
    Traj& t = m->traj[traj_ids[i]];
    if (t.slot < 0) {
      t.slot = m->free_slots.back();
      m->free_slots.pop_back();
    }
    size_t after = t.tokens.size() + lens[i];
    while (t.pages.size() * RL_PAGE < after) {
      int p = take_page(m);
      m->page_upd.insert(m->page_upd.end(), {t.slot, (int32_t)t.pages.size(), p});
      t.pages.push_back(p);
    }
    t.tokens.insert(t.tokens.end(), tokens + off, tokens + off + lens[i]);
    t.mask.insert(t.mask.end(), lens[i], (uint8_t)1);
    t.logp.insert(t.logp.end(), lens[i], 0.0f);
    off += lens[i];
  }
  for (int i = 0; i < n; i++) {   // after all insertions: map references are stable now
    Traj& t = m->traj[traj_ids[i]];
    if (!t.tokens.empty()) work.push_back({&t, (int)t.tokens.size() - 1});
  }
  *work_out = std::move(work);
  return RL_OK;
}

extern "C" int rl_append_observation(rl_model* m, const int32_t* traj_ids, int32_t n,
                                     const int32_t* tokens, const int32_t* lens) {
  std::vector<std::pair<Traj*, int>> work;
  int rc = append_host(m, traj_ids, n, tokens, lens, &work);
  if (rc) return rc;
  rc = prefill(m, work);
  const int urc = flush_page_updates(m);      // nothing left unless no token needed a pass
  return rc ? rc : urc;
}

extern "C" int rl_decode_step_with_appends(rl_model* m, const int32_t* app_ids, int32_t n_app,
                                           const int32_t* app_tokens, const int32_t* app_lens,
                                           const int32_t* ids, int32_t n, float temperature,
                                           uint64_t rng_seed, int32_t* token_ids_out,
                                           float* logprobs_out) {
  if (!m) return fail(RL_E_ARG, "null model");
  if (n > 0 && !token_ids_out) return fail(RL_E_ARG, "null output");
  std::vector<std::pair<Traj*, int>> work;
  int rc = append_host(m, app_ids, n_app, app_tokens, app_lens, &work);
  if (rc) return rc;
  return decode_common(m, ids, n, temperature, rng_seed, nullptr, token_ids_out, logprobs_out, &work);
}

extern "C" int rl_decode_step_forced_with_appends(rl_model* m, const int32_t* app_ids, int32_t n_app,
                                                  const int32_t* app_tokens, const int32_t* app_lens,
                                                  const int32_t* ids, int32_t n, float temperature,
                                                  const int32_t* forced_token_ids, float* logprobs_out) {
  if (!m) return fail(RL_E_ARG, "null model");
  if (n > 0 && !forced_token_ids) return fail(RL_E_ARG, "null forced ids");
  std::vector<std::pair<Traj*, int>> work;
  int rc = append_host(m, app_ids, n_app, app_tokens, app_lens, &work);
  if (rc) return rc;
  return decode_common(m, ids, n, temperature, 0, forced_token_ids, nullptr, logprobs_out, &work);
}

extern "C" int rl_decode_step(rl_model* m, const int32_t* ids, int32_t n, float temperature,
                              uint64_t rng_seed, int32_t* token_ids_out, float* logprobs_out) {
  if (!m) return fail(RL_E_ARG, "null model");
  if (n > 0 && !token_ids_out) return fail(RL_E_ARG, "null output");
  return decode_common(m, ids, n, temperature, rng_seed, nullptr, token_ids_out, logprobs_out);
}

extern "C" int rl_decode_steps(rl_model* m, const int32_t* ids, int32_t n, int32_t n_steps,
                               float temperature, uint64_t rng_seed, int32_t* token_ids_out,
                               float* logprobs_out) {
  if (!m) return fail(RL_E_ARG, "null model");
  return decode_multi(m, ids, n, n_steps, temperature, rng_seed, token_ids_out, logprobs_out);
}

extern "C" int rl_decode_step_forced(rl_model* m, const int32_t* ids, int32_t n, float temperature,
                                     const int32_t* forced_token_ids, float* logprobs_out) {
  if (!m) return fail(RL_E_ARG, "null model");
  if (n > 0 && !forced_token_ids) return fail(RL_E_ARG, "null forced ids");
  return decode_common(m, ids, n, temperature, 0, forced_token_ids, nullptr, logprobs_out);
}

extern "C" int rl_release(rl_model* m, const int32_t* ids, int32_t n) {
  if (!m) return fail(RL_E_ARG, "null model");
  int rc = check_ids(ids, n);
  if (rc) return rc;
  for (int i = 0; i < n; i++)
    if (!m->traj.count(ids[i])) return fail(RL_E_BAD_TRAJ, "unknown trajectory id");
  for (int i = 0; i < n; i++) {
    Traj& t = m->traj[ids[i]];
    for (int p : t.pages) drop_page(m, p);
    m->free_slots.push_back(t.slot);
    m->traj.erase(ids[i]);
  }
  return RL_OK;
}

extern "C" int rl_fork(rl_model* m, int32_t src, const int32_t* dst_ids, int32_t n) {
  if (!m) return fail(RL_E_ARG, "null model");
  int rc = check_ids(dst_ids, n);
  if (rc) return rc;
  auto sit = m->traj.find(src);
  if (sit == m->traj.end()) return fail(RL_E_BAD_TRAJ, "unknown source trajectory");
  for (int i = 0; i < n; i++)
    if (dst_ids[i] == src || m->traj.count(dst_ids[i])) return fail(RL_E_DUP_ID, "destination id already exists");
  int nt = (int)sit->second.tokens.size();
  int n_shared = nt > 0 ? (nt - 1) / RL_PAGE : 0;   // pages entirely before the last token
  int n_own = (int)sit->second.pages.size() - n_shared;
  if ((int64_t)m->traj.size() + n > m->rt.max_trajectories) return fail(RL_E_TOO_MANY, "too many trajectories");
  if ((int64_t)n_own * n > m->n_free) return fail(RL_E_NOPAGES, "page pool exhausted");
  std::vector<int32_t>& upd = m->page_upd;
  std::vector<int32_t> pairs;
  m->traj.reserve(m->traj.size() + n);
  for (int i = 0; i < n; i++) {
    Traj t = m->traj.find(src)->second;   // copy of tokens / mask / logp / n_cached
    t.slot = m->free_slots.back();
    m->free_slots.pop_back();
    for (int k = 0; k < n_shared; k++) m->refcount[t.pages[k]]++;
    t.shared_lead = std::max(t.shared_lead, n_shared);
    for (int k = n_shared; k < n_shared + n_own; k++) {
      int p = take_page(m);
      pairs.push_back(t.pages[k]);
      pairs.push_back(p);
      t.pages[k] = p;
    }
    for (size_t k = 0; k < t.pages.size(); k++) upd.insert(upd.end(), {t.slot, (int32_t)k, t.pages[k]});
    m->traj[dst_ids[i]] = std::move(t);
  }
  if (n > 0) {
    Traj& st = m->traj.find(src)->second;
    st.shared_lead = std::max(st.shared_lead, n_shared);
  }
  // page-table entries and page copies travel in one transfer, all layers' copies in one launch
  size_t nu = upd.size() / 3, np = pairs.size() / 2;
  if (3 * nu + 2 * np > m->meta_ints) {
    rc = flush_page_updates(m);
    if (rc) return rc;
    nu = 0;
  }
  for (size_t done = 0; nu > 0 || done < np;) {
    const size_t k = std::min((m->meta_ints - 3 * nu) / 2, np - done);
    if (nu) memcpy(m->h_meta, upd.data(), nu * 12);
    if (k) memcpy(m->h_meta + 3 * nu, pairs.data() + 2 * done, k * 8);
    HIPCHECK(hipMemcpyAsync(m->d_meta, m->h_meta, nu * 12 + k * 8, hipMemcpyHostToDevice, m->stream));
    launch_page_table_update(m->stream, m->page_table, m->d_meta, (int)nu, m->md.max_pages_per_traj);
    launch_copy_pages(m->stream, m->d_pools, m->md.L, m->d_meta + 3 * nu, (int)k, m->page_bytes);
    HIPCHECK(hipGetLastError());
    HIPCHECK(hipStreamSynchronize(m->stream));
    done += k;
    nu = 0;
    upd.clear();
  }
  return RL_OK;
}

extern "C" int rl_traj_info(rl_model* m, int32_t id, int32_t* n_tokens, int32_t* n_pages) {
  if (!m) return fail(RL_E_ARG, "null model");
  auto it = m->traj.find(id);
  if (it == m->traj.end()) return fail(RL_E_BAD_TRAJ, "unknown trajectory id");
  if (n_tokens) *n_tokens = (int32_t)it->second.tokens.size();
  if (n_pages) *n_pages = (int32_t)it->second.pages.size();
  return RL_OK;
}

extern "C" int rl_traj_read(rl_model* m, int32_t id, int32_t* tokens, uint8_t* obs_mask,
                            float* logprobs, int32_t* pages) {
  if (!m) return fail(RL_E_ARG, "null model");
  auto it = m->traj.find(id);
  if (it == m->traj.end()) return fail(RL_E_BAD_TRAJ, "unknown trajectory id");
  const Traj& t = it->second;
  if (tokens && !t.tokens.empty()) memcpy(tokens, t.tokens.data(), t.tokens.size() * 4);
  if (obs_mask && !t.mask.empty()) memcpy(obs_mask, t.mask.data(), t.mask.size());
  if (logprobs && !t.logp.empty()) memcpy(logprobs, t.logp.data(), t.logp.size() * 4);
  if (pages && !t.pages.empty()) memcpy(pages, t.pages.data(), t.pages.size() * 4);
  return RL_OK;
}

extern "C" int64_t rl_free_pages(const rl_model* m) { return m ? m->n_free : -1; }

extern "C" int rl_debug_logits(rl_model* m, int32_t id, float* logits_out) {
  if (!m || !logits_out) return fail(RL_E_ARG, "null argument");
  auto it = m->traj.find(id);
  if (it == m->traj.end()) return fail(RL_E_BAD_TRAJ, "unknown trajectory id");
  Traj& t = it->second;
  if (t.tokens.empty()) return fail(RL_E_EMPTY, "trajectory has no context");
  int nt = (int)t.tokens.size();
  Staging st;
  st.tok.push_back(t.tokens[nt - 1]);
  st.pos.push_back(nt - 1);
  st.slot.push_back(t.slot);
  add_decode_items(m, st, std::vector<Traj*>{&t});
  DevMeta dm;
  int rc = upload_meta(m, st, &dm);
  if (rc) return rc;
  RowMeta r{dm.tok, dm.pos, dm.slot, dm.items, (int)st.items.size(), dm.merges, (int)st.merges.size(),
            dm.rowlist, nullptr, 0, false, 0.0, false};
  forward_rows(m, 1, r);   // rewrites the key / value of position nt-1 with the same values
  lm_head_rows(m, 1, 0, 1, false);
  HIPCHECK(hipGetLastError());
  HIPCHECK(hipMemcpyAsync(logits_out, m->logits, (size_t)m->md.V * 4, hipMemcpyDeviceToHost, m->stream));
  HIPCHECK(hipStreamSynchronize(m->stream));
  return RL_OK;
}

namespace {

// What the objective pass adds to the teacher-forced pass: the log-probs of the tokens under the
// old and the reference policy, one value per token of every listed trajectory, concatenated.
struct ObjectiveCall {
  const float* old_lp;   // null: the log-probs recorded when the tokens were sampled
  const float* ref_lp;   // null: no KL term
  double clip_eps, beta;
};

// Teacher-forced pass over whole trajectories.  out != null: the log-prob of every sampled token
// goes to out (0 elsewhere).  obj != null: every sampled token's term of the objective is added to
// the accumulators of its trajectory (cleared beforehand by the advantages kernel).
int teacher_forced_pass(rl_model* m, const int32_t* ids, int32_t n, float temperature, float* out,
                        const ObjectiveCall* obj) {
  int rc = RL_OK;
  float c = sampler_scale(temperature);
  // flat list of rows: (trajectory, position p) for p in [0, n_tokens - 1); row p predicts token p+1
  struct Seg { Traj* t; size_t out_off; };
  std::vector<Seg> segs;
  size_t off = 0;
  for (int i = 0; i < n; i++) {
    Traj& t = m->traj[ids[i]];
    segs.push_back({&t, off});
    if (out)
      for (size_t k = 0; k < t.tokens.size(); k++) out[off + k] = 0.0f;
    off += t.tokens.size();
  }
  const size_t Mc = (size_t)m->Mcap;
  float* g_old = m->h_gaux;
  float* g_ref = m->h_gaux + Mc;
  int32_t* g_use = (int32_t*)(m->h_gaux + 2 * Mc);
  int32_t* g_seg = (int32_t*)(m->h_gaux + 3 * Mc);
  // rows of this block of the pass -> terms of the objective (rows k in [0, K): log-prob in
  // d_lp_rows[k], token dest[k] of trajectory number dtraj[k])
  auto objective_rows = [&](int K, const std::vector<size_t>& dest, const std::vector<int>& dtraj,
                            const std::vector<uint8_t>* mask) -> int {
    if (K == 0) return RL_OK;
    int nseg = 0;
    for (int k = 0; k < K; k++) {
      size_t at = dest[k];
      const Traj* t = segs[dtraj[k]].t;
      g_old[k] = obj->old_lp ? obj->old_lp[at] : t->logp[at - segs[dtraj[k]].out_off];
      g_ref[k] = obj->ref_lp ? obj->ref_lp[at] : 0.0f;
      g_use[k] = mask ? ((*mask)[k] == 0) : 1;
      if (k == 0 || dtraj[k] != dtraj[k - 1]) {
        if (nseg) g_seg[3 * nseg - 1] = k;
        g_seg[3 * nseg] = dtraj[k];
        g_seg[3 * nseg + 1] = k;
        nseg++;
      }
    }
    g_seg[3 * nseg - 1] = K;
    float* d = m->d_gaux;
    HIPCHECK(hipMemcpyAsync(d, m->h_gaux, (3 * Mc + 3 * (size_t)nseg) * 4, hipMemcpyHostToDevice, m->stream));
    launch_grpo_terms(m->stream, m->d_lp_rows, d, obj->ref_lp ? d + Mc : nullptr, (const int32_t*)(d + 2 * Mc),
                      (const int32_t*)(d + 3 * Mc), nseg, m->d_gadv, obj->clip_eps, obj->beta, m->d_gacc);
    HIPCHECK(hipGetLastError());
    return RL_OK;
  };
  Staging st;
  std::vector<size_t> dest;   // output index of each row's log-prob
  std::vector<int> dtraj;     // number (in call order) of each row's trajectory
  size_t si = 0;
  int cur = 0;
  int cap = m->Mcap;
  while (si < segs.size()) {
    st.clear();
    dest.clear();
    dtraj.clear();
    while (si < segs.size() && (int)st.tok.size() < cap) {
      Traj* t = segs[si].t;
      int upto = (int)t->tokens.size() - 1;
      if (cur >= upto) { si++; cur = 0; continue; }
      int take = std::min(upto - cur, cap - (int)st.tok.size());
      add_items(m, st, (int)st.tok.size(), take, t->slot, cur);
      for (int p = cur; p < cur + take; p++) {
        st.tok.push_back(t->tokens[p]);
        st.pos.push_back(p);
        st.slot.push_back(t->slot);
        st.forced.push_back(t->tokens[p + 1]);
        st.mask.push_back(t->mask[p + 1]);
        dest.push_back(segs[si].out_off + p + 1);
        dtraj.push_back((int)si);
      }
      cur += take;
    }
    int M = (int)st.tok.size();
    if (M == 0) break;
    st.traj.assign(M, 0);
    st.newpos.assign(M, 0);
    // rows whose target token was sampled by the policy (mask 0): only they need the lm-head.
    // Their row numbers and targets travel in the two metadata arrays this pass does not use.
    int nsel = 0;
    if (m->mfma)
      for (int k = 0; k < M; k++)
        if (st.mask[k] == 0) {
          st.traj[nsel] = k;
          st.newpos[nsel] = st.forced[k];
          dest[nsel] = dest[k];
          dtraj[nsel] = dtraj[k];
          nsel++;
        }
    DevMeta dm;
    rc = upload_meta(m, st, &dm);
    if (rc) return rc;
    RowMeta r{dm.tok, dm.pos, dm.slot, dm.items, (int)st.items.size(), dm.merges, 0, dm.rowlist, nullptr, 0, true, 0.0, false};
    forward_rows(m, M, r);
    if (m->mfma) {
      // fused pass: gather + final norm, lm-head with the log-softmax reduced in its epilogue (the
      // logits are never stored; the logits buffer serves as scratch for the per-strip statistics)
      const ModelDims& md = m->md;
      size_t per_row = (size_t)(md.V / 32) * 8;
      int rows_cap = (int)std::min<size_t>((size_t)m->Mcap, (size_t)m->Rl * md.V * 4 / per_row);
      for (int c0 = 0; c0 < nsel; c0 += rows_cap) {
        int R = std::min(rows_cap, nsel - c0);
        launch_add_rmsnorm(m->stream, m->h, m->ph, m->pending_parts, (size_t)M * md.H,
                           (const bf16_t*)m->g_final, (bf16_t*)m->xa, R, md.H, md.eps, dm.traj + c0);
        launch_lm_head_logprob(m->stream, (const bf16_t*)m->xa, (const bf16_t*)m->lm_head, R, md.V, md.H,
                               dm.newpos + c0, c, m->logits, m->d_zt, m->d_lp_rows + c0);
      }
      m->pending_parts = 0;
      HIPCHECK(hipGetLastError());
      if (obj && (rc = objective_rows(nsel, dest, dtraj, nullptr))) return rc;
      if (out && nsel > 0)
        HIPCHECK(hipMemcpyAsync(m->h_lp_rows, m->d_lp_rows, (size_t)nsel * 4, hipMemcpyDeviceToHost, m->stream));
      HIPCHECK(hipStreamSynchronize(m->stream));
      if (out)
        for (int k = 0; k < nsel; k++) out[dest[k]] = m->h_lp_rows[k];
      continue;
    }
    for (int r0 = 0; r0 < M; r0 += m->Rl) {
      int R = std::min(m->Rl, M - r0);
      lm_head_rows(m, M, r0, R, r0 > 0);
      launch_sampler(m->stream, m->logits, (size_t)m->md.V, R, m->md.V, c, 0, nullptr, 0, nullptr,
                     nullptr, dm.forced + r0, m->d_mask + r0, m->ss, nullptr, m->d_lp);
      HIPCHECK(hipGetLastError());
      if (obj)
        HIPCHECK(hipMemcpyAsync(m->d_lp_rows + r0, m->d_lp, (size_t)R * 4, hipMemcpyDeviceToDevice, m->stream));
      if (out) HIPCHECK(hipMemcpyAsync(m->h_lp, m->d_lp, (size_t)R * 4, hipMemcpyDeviceToHost, m->stream));
      HIPCHECK(hipStreamSynchronize(m->stream));
      if (out)
        for (int k = 0; k < R; k++) out[dest[r0 + k]] = m->h_lp[k];
    }
    if (obj) {
      if ((rc = objective_rows(M, dest, dtraj, &st.mask))) return rc;
      HIPCHECK(hipStreamSynchronize(m->stream));
    }
  }
  return RL_OK;
}

}  // namespace

extern "C" int rl_recompute_logprobs(rl_model* m, const int32_t* ids, int32_t n, float temperature,
                                     float* out) {
  if (!m) return fail(RL_E_ARG, "null model");
  int rc = check_ids(ids, n);
  if (rc) return rc;
  if (!(temperature >= 0.0f) || (n > 0 && !out)) return fail(RL_E_ARG, "bad temperature or null output");
  for (int i = 0; i < n; i++)
    if (!m->traj.count(ids[i])) return fail(RL_E_BAD_TRAJ, "unknown trajectory id");
  return teacher_forced_pass(m, ids, n, temperature, out, nullptr);
}

extern "C" int rl_grpo_objective(rl_model* m, const int32_t* ids, int32_t n, int32_t group_size,
                                 const float* rewards, const float* old_logprobs,
                                 const float* ref_logprobs, float temperature, double clip_eps,
                                 double beta, double eps_std, int32_t std_ddof, double* objective_out,
                                 double* kl_out, int64_t* n_tokens_out, double* advantages_out) {
  if (!m) return fail(RL_E_ARG, "null model");
  int rc = check_ids(ids, n);
  if (rc) return rc;
  if (n <= 0 || !rewards || !objective_out) return fail(RL_E_ARG, "no trajectories, or null rewards or output");
  if (group_size <= 0 || n % group_size != 0) return fail(RL_E_ARG, "trajectories must form whole groups");
  if (std_ddof != 0 && !(std_ddof == 1 && group_size >= 2))
    return fail(RL_E_ARG, "std_ddof must be 0, or 1 with groups of at least two");
  if (!(temperature >= 0.0f) || !(clip_eps >= 0.0) || !(eps_std >= 0.0) || !(beta >= 0.0) ||
      !std::isfinite(clip_eps) || !std::isfinite(beta) || !std::isfinite(eps_std))
    return fail(RL_E_ARG, "bad temperature, clip_eps, beta or eps_std");
  for (int i = 0; i < n; i++) {
    if (!m->traj.count(ids[i])) return fail(RL_E_BAD_TRAJ, "unknown trajectory id");
    if (!std::isfinite(rewards[i])) return fail(RL_E_ARG, "reward is not finite");
  }
  const size_t Mc = (size_t)m->Mcap, T = (size_t)m->rt.max_trajectories;
  float* h_rew = m->h_gaux + 3 * Mc + 3 * T + 3;   // behind the per-block staging: not reused during the pass
  float* d_rew = m->d_gaux + 3 * Mc + 3 * T + 3;
  memcpy(h_rew, rewards, (size_t)n * 4);
  HIPCHECK(hipMemcpyAsync(d_rew, h_rew, (size_t)n * 4, hipMemcpyHostToDevice, m->stream));
  launch_grpo_advantages(m->stream, d_rew, n, group_size, eps_std, std_ddof, m->d_gadv, m->d_gacc);
  HIPCHECK(hipGetLastError());
  ObjectiveCall oc{old_logprobs, ref_logprobs, clip_eps, beta};
  rc = teacher_forced_pass(m, ids, n, temperature, nullptr, &oc);
  if (rc) return rc;
  launch_grpo_finish(m->stream, m->d_gacc, n, m->d_gout);
  HIPCHECK(hipGetLastError());
  double res[3];
  HIPCHECK(hipMemcpyAsync(res, m->d_gout, sizeof(res), hipMemcpyDeviceToHost, m->stream));
  if (advantages_out)
    HIPCHECK(hipMemcpyAsync(advantages_out, m->d_gadv, (size_t)n * 8, hipMemcpyDeviceToHost, m->stream));
  HIPCHECK(hipStreamSynchronize(m->stream));
  *objective_out = res[0];
  if (kl_out) *kl_out = res[1];
  if (n_tokens_out) *n_tokens_out = (int64_t)res[2];
  return RL_OK;
}

extern "C" int rl_sample_from_logits(const float* logits, int32_t rows, int32_t vocab,
                                     float temperature, const uint32_t* u32, int32_t* ids_out,
                                     float* logprobs_out) {
  if (!logits || !u32 || !ids_out || !logprobs_out || rows <= 0 || vocab <= 0 || !(temperature >= 0.0f))
    return fail(RL_E_ARG, "bad argument");
  int nseg = sampler_nseg(vocab);
  size_t zb = (size_t)rows * vocab * 4;
  char* buf = nullptr;
  size_t seg_n = (size_t)rows * nseg;
  size_t total = zb + seg_n * (4 + 4 + 8 + 4) + (size_t)rows * 12 + 64;
  HIPCHECK(hipMalloc((void**)&buf, total));
  float* dz = (float*)buf;
  SamplerScratch sc;
  sc.segw = (uint64_t*)(buf + ((zb + 7) / 8) * 8);
  sc.segmax = (float*)(sc.segw + seg_n);
  sc.segarg = (int32_t*)(sc.segmax + seg_n);
  sc.sege = (float*)(sc.segarg + seg_n);
  uint32_t* du = (uint32_t*)(sc.sege + seg_n);
  int32_t* dids = (int32_t*)(du + rows);
  float* dlp = (float*)(dids + rows);
  int rc = RL_OK;
  bool greedy = temperature == 0.0f;
  float c = sampler_scale(temperature);
  hipError_t e = hipMemcpy(dz, logits, zb, hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(du, u32, (size_t)rows * 4, hipMemcpyHostToDevice);
  if (e == hipSuccess) {
    launch_sampler(nullptr, dz, (size_t)vocab, rows, vocab, c, greedy ? 1 : 0, du, 0, nullptr, nullptr,
                   nullptr, nullptr, sc, dids, dlp);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipDeviceSynchronize();
  if (e == hipSuccess) e = hipMemcpy(ids_out, dids, (size_t)rows * 4, hipMemcpyDeviceToHost);
  if (e == hipSuccess) e = hipMemcpy(logprobs_out, dlp, (size_t)rows * 4, hipMemcpyDeviceToHost);
  if (e != hipSuccess) rc = fail(RL_E_HIP, hipGetErrorString(e));
  (void)hipFree(buf);
  return rc;
}

namespace {
int debug_plan(const rl_model_config* c, int32_t rows, int32_t max_rows, const int32_t* out, ModelDims* md, PassPlan* p) {
  if (!c || !out || rows <= 0 || max_rows < rows) return fail(RL_E_ARG, "bad argument");
  if (c->n_layers <= 0 || c->hidden <= 0 || c->n_q_heads <= 0 || c->n_kv_heads <= 0 || c->intermediate <= 0 ||
      c->vocab <= 0 || c->n_q_heads % c->n_kv_heads != 0 || !mfma_shape_ok(*c))
    return fail(RL_E_ARG, "not a shape of the MFMA kernels");
  *md = ModelDims{c->n_layers, c->hidden, c->n_q_heads, c->n_kv_heads, c->head_dim, c->intermediate,
                  c->vocab, c->rms_eps, c->qk_norm, 1, 0};
  *p = plan_pass(*md, rows, partial_rows((size_t)round_up(max_rows, 128)));
  return RL_OK;
}
}  // namespace

extern "C" int rl_debug_residual_plan(const rl_model_config* c, int32_t rows, int32_t max_rows, int32_t* out) {
  ModelDims md;
  PassPlan p;
  const int rc = debug_plan(c, rows, max_rows, out, &md, &p);
  if (rc) return rc;
  out[0] = p.ro.rb; out[1] = p.ro.cb; out[2] = p.rd.rb; out[3] = p.rd.cb;
  return RL_OK;
}

extern "C" int rl_debug_pass_plan(const rl_model_config* c, int32_t rows, int32_t max_rows, int32_t* out) {
  ModelDims md;
  PassPlan p;
  const int rc = debug_plan(c, rows, max_rows, out, &md, &p);
  if (rc) return rc;
  auto put = [&](int at, const GemmPlan& g, int epilogue) {
    out[4 * at] = g.kind; out[4 * at + 1] = g.width; out[4 * at + 2] = g.splits; out[4 * at + 3] = epilogue;
  };
  put(0, p.q, p.fused_qkv ? EPI_QKV : EPI_STORE);
  put(1, p.o, p.eo);
  put(2, p.g, EPI_SWIGLU);
  put(3, p.d, p.ed);
  put(4, plan_gemm(rows, md.V, md.H, EPI_LSE, 0), EPI_LSE);
  put(5, plan_gemm(rows, md.V, md.H, EPI_STORE, 0), EPI_STORE);
  return RL_OK;
}

extern "C" int rl_debug_staging_plan(int32_t n, int32_t n_kv_heads, int32_t max_trajectories, int32_t max_batch_rows, int32_t new_pages,
                                     int32_t* out) {
  if (!out || n <= 0 || n > max_trajectories || n_kv_heads < 0 || max_batch_rows < 0 || new_pages < 0) return fail(RL_E_ARG, "bad argument");
  const StagingPlan p = plan_staging(staging_ints(max_batch_rows, max_trajectories), staging_region_ints(n, attention_slots(n_kv_heads, max_trajectories)),
                                     3 * (size_t)new_pages);
  out[0] = p.flush; out[1] = p.regions; out[2] = p.group;
  return RL_OK;
}

extern "C" int rl_debug_many_row_loads(int32_t rows, int32_t n, int32_t k, int32_t kernel, int32_t width, int32_t slices,
                                       int32_t epilogue, int64_t* out) {
  const bool t256 = kernel == GEMM_TILE256;
  if (!out || rows <= 0 || n <= 0 || n % 32 != 0 || k <= 0 || k % 64 != 0 || (!t256 && kernel != GEMM_WIDE128) ||
      (width != 4 && !(t256 && width == 5)) || slices < 1 || slices > kMaxSplits || (int64_t)n * k * 2 >= 0x7fff0000)
    return fail(RL_E_ARG, "bad argument");
  debug_many_row_loads(rows, n, k, t256 ? 4 : 2, width, slices, epilogue, out);
  return RL_OK;
}

extern "C" int rl_timing_enable(rl_model* m, int32_t every) {
  if (!m || every < 0) return fail(RL_E_ARG, "bad argument");
  m->timing_every = every;
  return RL_OK;
}

// Plain streaming read for calibrating benchmarks: every thread keeps eight 16-byte loads in flight.
__global__ __launch_bounds__(256) void stream_read_kernel(const u32x4* __restrict__ p, size_t n,
                                                          unsigned* __restrict__ sink) {
  u32x4 a = {0u, 0u, 0u, 0u};
  const size_t stride = (size_t)gridDim.x * 256 * 8;
  for (size_t i = (size_t)blockIdx.x * 256 * 8 + threadIdx.x; i + 7 * 256 < n; i += stride) {
    u32x4 x[8];
#pragma unroll
    for (int u = 0; u < 8; u++) x[u] = __builtin_nontemporal_load(p + i + u * 256);
#pragma unroll
    for (int u = 0; u < 8; u++) a ^= x[u];
  }
  if ((a[0] ^ a[1] ^ a[2] ^ a[3]) == 0x9e3779b9u) *sink = 1;   // keeps the loads alive
}

extern "C" int rl_measure_stream_read(size_t bytes, int32_t iters, double* gb_per_s) {
  if (!gb_per_s || iters <= 0 || bytes < (1u << 24)) return fail(RL_E_ARG, "bad argument");
  void* buf = nullptr;
  unsigned* sink = nullptr;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  int rc = RL_OK;
  size_t n = bytes / 16 / (256 * 8) * (256 * 8);   // whole groups of 8 loads per workgroup
  auto run = [&]() -> int {
    HIPCHECK(hipMalloc(&buf, bytes));
    HIPCHECK(hipMalloc((void**)&sink, 4));
    HIPCHECK(hipMemset(buf, 1, bytes));
    HIPCHECK(hipEventCreate(&e0));
    HIPCHECK(hipEventCreate(&e1));
    stream_read_kernel<<<512, 256>>>((const u32x4*)buf, n, sink);
    HIPCHECK(hipDeviceSynchronize());
    HIPCHECK(hipEventRecord(e0, nullptr));
    for (int i = 0; i < iters; i++) stream_read_kernel<<<512, 256>>>((const u32x4*)buf, n, sink);
    HIPCHECK(hipEventRecord(e1, nullptr));
    HIPCHECK(hipEventSynchronize(e1));
    HIPCHECK(hipGetLastError());
    float ms = 0.f;
    HIPCHECK(hipEventElapsedTime(&ms, e0, e1));
    *gb_per_s = (double)n * 16.0 * iters / (ms * 1e-3) / 1e9;
    return RL_OK;
  };
  rc = run();
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  if (buf) (void)hipFree(buf);
  if (sink) (void)hipFree(sink);
  return rc;
}

extern "C" int rl_timing_read_steps(rl_model* m, double* step_gpu_ms, int64_t* steps, int reset) {
  if (!m) return fail(RL_E_ARG, "null model");
  if (step_gpu_ms) *step_gpu_ms = m->step_gpu_ms;
  if (steps) *steps = m->steps_timed;
  if (reset) { m->step_gpu_ms = 0.0; m->steps_timed = 0; }
  return RL_OK;
}

extern "C" int rl_timing_read_decode_bytes(rl_model* m, double* kv_bytes, double* kv_unique_bytes,
                                           int64_t* steps, int reset) {
  if (!m) return fail(RL_E_ARG, "null model");
  if (kv_bytes) *kv_bytes = m->acct_kv_bytes;
  if (kv_unique_bytes) *kv_unique_bytes = m->acct_kv_unique_bytes;
  if (steps) *steps = m->acct_steps;
  if (reset) { m->acct_kv_bytes = 0.0; m->acct_kv_unique_bytes = 0.0; m->acct_steps = 0; }
  return RL_OK;
}

extern "C" int rl_timing_read(rl_model* m, double* attn_ms, int64_t* attn_launches,
                              double* attn_kv_bytes, double* attn_kv_unique_bytes, int reset) {
  if (!m) return fail(RL_E_ARG, "null model");
  if (attn_ms) *attn_ms = m->attn_ms;
  if (attn_launches) *attn_launches = m->attn_launches;
  if (attn_kv_bytes) *attn_kv_bytes = m->attn_bytes;
  if (attn_kv_unique_bytes) *attn_kv_unique_bytes = m->attn_unique_bytes;
  if (reset) { m->attn_ms = 0.0; m->attn_launches = 0; m->attn_bytes = 0.0; m->attn_unique_bytes = 0.0; }
  return RL_OK;
}
