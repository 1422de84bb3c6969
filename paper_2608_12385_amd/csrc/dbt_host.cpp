// Host side of the decode library: argument checking, workspace layout, the
// page allocator of the single primary KV cache, and the order in which the
// kernels of prefill, boundary and continuation steps are enqueued
// (Sec. 4.4 of the Decode-Branch Transformer paper).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <functional>
#include <numeric>
#include <new>
#include <queue>
#include <string>
#include <vector>

#include "../../include/dbt.h"
#include "host_internal.h"
#include "kernels.h"

using namespace dbt;

namespace {

thread_local std::string g_err;

dbt_status fail(dbt_status s, const char *fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return s;
}

#define HIPCHK(expr)                                                                         \
  do {                                                                                       \
    hipError_t e_ = (expr);                                                                  \
    if (e_ != hipSuccess) return fail(DBT_ERR_HIP, "%s: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

constexpr int kPage = 16;
// Decode attention reads a sequence of P pages in ceil(P / target) equal
// splits, one workgroup of eight waves each.  A model with few (sequence, KV
// head) pairs (max_batch x n_kv below 256) takes the target that makes its
// longest caches one round of workgroups, within 24 pages (two or three page
// pairs for each wave; the workgroup's start costs as much) and the 1024 page
// ids the kernel holds; one with more pairs, which reads whole sequences when
// the batch fills the chip, 86 pages for its smaller calls.  The target is
// fixed when the model is created, so a row's result depends only on its own
// query and cache.
// Whole steps by target: 24 layers, 16 sequences of 300-1500 positions, 4 KV
// heads: 16 pages 1607 us, 24 (the rule) 1421, 32 1441, 48 1479, 64 1522; a share
// of one KV head, 13 sequences of 150-4096: 84 us at 16 and 24, 86 at 48, 95 at 128.
// The rule cannot know how full a model is.  One 8B-shape layer, 8 sequences of
// at most 8192 positions (target 128), 1 x 8000 positions: 119.7 us (64 pages
// 111.8; four-wave workgroups of 64 pages, the form before, 116.4), 8 x 1025-2048:
// 120.9 (131.6; 133.6), 8 x 8150: 148.7 (144.9; 146.1); every other partly filled
// model that was timed gains over that form as well.
// fp32 splits are 64 pages long.
constexpr int kSplitTargetBf16 = 86, kSplitMinBf16 = 24, kSplitMaxBf16 = 1024, kSplitTargetF32 = 64;
constexpr int kMixChunk = 4096;
// Prompts are prefilled in packed passes of up to max(max_prompt, kPackRows)
// rows, so that each weight is read once for many short prompts and the tiled
// projections fill the chip: a W_O of 2048 columns has 8 x 32 tiles at 8192
// rows, one for each compute unit.  24 prompts of 17-300 positions through two
// layers of width 2048: 7.74 ms one by one, 1.13 ms packed.
constexpr int kPackRows = 8192;
// Average rows per expert from which a prompt pass runs the experts' products
// as 128-row tiles instead of streaming each expert's weights past 32 rows at
// a time.  64 experts of 1408, whole pass of one layer: 19 rows each 571 us
// tiled and 537 streamed, 31 rows 614 and 682.
constexpr int kExpertTileRows = 24;

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }
int round16(int x) { return (x + 15) / 16 * 16; }
// Decode branches (App. C.1 for more than one); 0 reads as one branch.
int n_branches(const dbt_config &c) { return c.n_branches > 1 ? c.n_branches : 1; }

// Offsets (bytes) of every workspace buffer.
struct Layout {
  int Bp_max = 0, R_max = 0, pack_rows = 0, max_in = 0, nqkv = 0, f = 0;
  GemmConfig g_qkv{1, 1, 1}, g_o{1, 1, 1}, g_gu{1, 1, 1}, g_d{1, 1, 1}, g_lm{1, 1, 1};
  int split_target = 0, max_splits = 0, nch = 0, nstat = 0;
  bool moe = false;
  // Decode gate/up on the fused SwiGLU kernel: fixed per model (from the
  // largest stacked call), so every call of a step sums each output element
  // in the same order whatever paths it carries.
  bool glu = false;
  int fe = 0, fs = 0, amax = 0;
  GemmConfig g_sgu{1, 1, 1}, g_sd{1, 1, 1};
  size_t moe_idx = 0, moe_logits = 0, moe_tiles = 0, moe_ntiles = 0, moe_w = 0, moe_aslot = 0, moe_counts = 0, moe_offsets = 0, moe_arow = 0, moe_h = 0,
         moe_y = 0, ret_idx = 0;
  size_t prow = 0, ptiles = 0;  // prompt passes: row map, attention tiles
  size_t part = 0;  // floats at P
  size_t rope = 0, pos = 0, S = 0, Xn = 0, Xh = 0, Q = 0, O = 0, P = 0, apart = 0, astat = 0,
         logits = 0, mstats = 0, xss = 0, ret_q = 0, ret_h = 0, ret_m = 0, ret_a = 0, btok = 0, slast = 0,
         // [0, state_total): state; [state_total, step_total): step buffers; [step_total, total): prompt passes
         state_total = 0, step_total = 0, total = 0;
};

dbt_status check_config(const dbt_config *c) {
  if (!c) return fail(DBT_ERR_ARG, "config is NULL");
  if (c->n_layers <= 0 || c->d_model <= 0 || c->n_q_heads <= 0 || c->n_kv_heads <= 0 ||
      c->head_dim <= 0 || c->vocab < 0 || c->max_batch <= 0 || c->max_pos <= 0 || c->max_prompt < 0)
    return fail(DBT_ERR_ARG, "sizes must be positive");
  if (c->dtype != DBT_F32 && c->dtype != DBT_BF16) return fail(DBT_ERR_ARG, "dtype must be DBT_F32 or DBT_BF16");
  if (c->n_q_heads % c->n_kv_heads) return fail(DBT_ERR_SHAPE, "n_q_heads %% n_kv_heads != 0");
  if (c->head_dim % 4) return fail(DBT_ERR_SHAPE, "head_dim must be a multiple of 4");
  if (c->d_model % 4) return fail(DBT_ERR_SHAPE, "d_model must be a multiple of 4");
  if (c->d_model > 32768) return fail(DBT_ERR_UNSUPPORTED, "d_model above 32768");
  if (c->max_prompt > c->max_pos) return fail(DBT_ERR_SHAPE, "max_prompt > max_pos");
  if (c->n_experts > 0) {
    if (c->dtype != DBT_BF16) return fail(DBT_ERR_UNSUPPORTED, "MoE layers run in bf16 only");
    if (c->n_experts > 256 || c->d_model > 4096 || c->d_model % 512)
      return fail(DBT_ERR_UNSUPPORTED, "MoE needs n_experts <= 256 and d_model a multiple of 512 up to 4096");
    if (c->top_k1 < 1 || c->top_k1 > 8 || c->top_k2 < 1 || c->top_k2 > 8 || c->top_k1 > c->n_experts ||
        c->top_k2 > c->n_experts)
      return fail(DBT_ERR_ARG, "top_k1/top_k2 must be in [1, min(8, n_experts)]");
    if (c->replay && c->top_k2 != c->top_k1) return fail(DBT_ERR_ARG, "router replay needs top_k2 == top_k1");
    if (c->compute_matched != 0 && c->compute_matched != 1) return fail(DBT_ERR_ARG, "compute_matched must be 0 or 1");
    if (c->d_ff_expert <= 0 || c->d_ff_expert % 128 || c->d_ff_shared < 0 || c->d_ff_shared % 128)
      return fail(DBT_ERR_UNSUPPORTED, "expert widths must be multiples of 128");
  } else if (c->d_ff <= 0) {
    return fail(DBT_ERR_ARG, "d_ff must be positive");
  } else if (c->compute_matched) {
    return fail(DBT_ERR_UNSUPPORTED, "the compute-matched variant (App. B.3) is an MoE variant");
  }
  if (c->has_embeddings && c->vocab <= 0) return fail(DBT_ERR_SHAPE, "token inputs need a vocabulary");
  if (c->max_prompt > 0 && !c->has_embeddings) return fail(DBT_ERR_SHAPE, "prefill needs token inputs");
  if (!(c->rms_eps >= 0.f) || !(c->rope_theta > 0.f)) return fail(DBT_ERR_ARG, "bad rms_eps/rope_theta");
  if (c->n_branches < 0 || c->n_branches > 3) return fail(DBT_ERR_ARG, "n_branches must be in [0, 3]");
  if (c->n_branches > 1 && c->n_experts > 0)
    return fail(DBT_ERR_UNSUPPORTED, "more than one decode branch runs with dense MLPs only");
  const int G = c->n_q_heads / c->n_kv_heads, P = 1 + n_branches(*c);
  if (P * G > 16) return fail(DBT_ERR_UNSUPPORTED, "(1 + n_branches) * query heads per KV head exceeds 16");
  if (c->head_dim > 128) return fail(DBT_ERR_UNSUPPORTED, "head_dim > 128");
  if (c->dtype == DBT_BF16) {
    const int dq = c->n_q_heads * c->head_dim, dkv = c->n_kv_heads * c->head_dim;
    if (c->head_dim != 128) return fail(DBT_ERR_UNSUPPORTED, "bf16 attention needs head_dim 128");
    if (c->d_model % 128 || dq % 128 || (c->n_experts == 0 && c->d_ff % 128))
      return fail(DBT_ERR_UNSUPPORTED, "bf16 projections need d_model, n_q*d_h, d_ff multiples of 128");
    if (dkv % 64 || c->vocab % 64) return fail(DBT_ERR_UNSUPPORTED, "bf16 projections need n_kv*d_h, vocab multiples of 64");
  }
  return DBT_OK;
}

// Reduction splits of a streaming projection over M prompt rows (fewer than
// the tiled projection needs): the decode splits, fewer where the second
// block of 128 rows doubles the workgroups.
int prompt_splits(const GemmConfig &g, int M) { return std::max(1, g.S / ((M + 127) / 128)); }

// fp32 output elements a projection N x K of a prompt pass of up to `rows`
// rows can need: plain outputs, the slabs of a short pass, or those of a tiled
// one (at least 1024 elements of the reduction each; kTileSlabs bounds all of
// them together).  fused: the tiled kernel's epilogue writes no fp32 output.
size_t prompt_part(const GemmConfig &g, int N, int K, int dtype, int rows, bool fused) {
  const size_t one = (size_t)rows * N;
  if (dtype != DBT_BF16) return one;
  const size_t slabs = (size_t)std::max(g.S, 2) * std::min(rows, 128) * N;
  if (rows < kTileRows) return std::max(slabs, one);
  if (fused && (long long)N * K < (1LL << 31) && (long long)rows * K < (1LL << 31)) return slabs;
  return std::max({slabs, one, K >= 2048 ? std::min<size_t>(kTileSlabs, one * std::min(4, K / 1024)) : 0});
}

// The workspace of a model: the state, the buffers of a call over stacked
// sequences, and the buffers of the packed prompt passes.
Layout make_layout(const dbt_config *c) {
  Layout L;
  const int d = c->d_model, dq = c->n_q_heads * c->head_dim, dkv = c->n_kv_heads * c->head_dim;
  L.moe = c->n_experts > 0;
  L.fe = c->d_ff_expert;
  L.fs = L.moe ? c->d_ff_shared : 0;
  L.f = L.moe ? std::max(L.fs, 128) : c->d_ff;
  L.Bp_max = round16(c->max_batch);
  L.R_max = (1 + n_branches(*c)) * L.Bp_max;
  L.max_in = std::max(std::max(d, dq), L.f);
  L.nqkv = dq + 2 * dkv;
  L.g_qkv = gemm_config(L.nqkv, d, c->dtype, std::gcd(dq, dkv), L.R_max);
  L.g_o = gemm_config(d, dq, c->dtype, d, L.R_max);
  L.g_gu = gemm_config(2 * L.f, d, c->dtype, L.f, L.R_max);
  L.g_d = gemm_config(d, L.f, c->dtype, d, L.R_max);
  L.g_lm = gemm_config(std::max(c->vocab, 1), d, c->dtype, std::max(c->vocab, 1), L.R_max);
  L.g_lm.S = 1;  // the logits are written in place (one slab)
  L.glu = !L.moe && gemm_glu_ok(L.f, L.R_max, 1 + n_branches(*c), c->dtype);
  if (L.moe && L.fs > 0) {
    L.g_sgu = gemm_config(2 * L.fs, d, c->dtype, L.fs, L.R_max);
    L.g_sd = gemm_config(d, L.fs, c->dtype, d, L.R_max);
  }
  const int maxpages = (c->max_pos + kPage - 1) / kPage;
  if (c->dtype == DBT_BF16) {
    const int pairs = c->max_batch * c->n_kv_heads;
    const int want = (kComputeUnits + pairs - 1) / pairs;  // splits per pair
    L.split_target = pairs >= kComputeUnits ? std::min(std::max(maxpages, kSplitMinBf16), kSplitTargetBf16)
                                  : std::clamp((maxpages + want - 1) / want, kSplitMinBf16, kSplitMaxBf16);
  } else {
    L.split_target = kSplitTargetF32;
  }
  L.max_splits = (maxpages + L.split_target - 1) / L.split_target;
  L.nch = c->vocab > 0 ? (c->vocab + kMixChunk - 1) / kMixChunk : 0;
  L.pack_rows = c->max_prompt > 0
                    ? (int)std::max<long long>(c->max_prompt, std::min<long long>((long long)c->max_batch * c->max_prompt, kPackRows))
                    : 0;
  size_t part = std::max({(size_t)L.g_qkv.S * L.R_max * L.nqkv, (size_t)L.g_o.S * L.R_max * d,
                          (size_t)L.g_gu.S * L.R_max * 2 * L.f, (size_t)L.g_d.S * L.R_max * d});
  if (L.moe) part = std::max({part, (size_t)L.g_sgu.S * L.R_max * 2 * L.f, (size_t)L.g_sd.S * L.R_max * d});
  L.part = part;
  size_t o = 0;
  auto take = [&](size_t bytes) { size_t at = o; o += align256(bytes); return at; };
  // State kept between calls: the RoPE table, positions, the primary
  // intermediates retained for a later branch evaluation, the boundary's
  // token and residual.
  L.rope = take((size_t)c->max_pos * (c->head_dim / 2) * 2 * sizeof(float));
  L.pos = take((size_t)c->max_batch * sizeof(int));
  L.ret_q = take((size_t)c->n_layers * L.Bp_max * dq * 4);
  L.ret_h = take((size_t)c->n_layers * L.Bp_max * L.f * 4);
  L.ret_m = take((size_t)c->n_layers * L.Bp_max * d * 4);
  L.ret_a = take(c->compute_matched ? (size_t)c->n_layers * L.Bp_max * d * 4 : 0);
  if (L.moe) L.ret_idx = take((size_t)c->n_layers * L.Bp_max * 8 * 4);
  L.btok = take((size_t)c->max_batch * 4);
  L.slast = take((size_t)L.Bp_max * d * 4);
  // Step buffers: written and read within one call (every element a call
  // reads is written earlier in the same call, apart from padding rows whose
  // results are never used), so any memory of this size can hold them.
  o = align256(o);
  L.state_total = o;
  L.S = take((size_t)L.R_max * d * 4);
  L.Xn = take((size_t)L.R_max * L.max_in * 4);
  L.Xh = take((size_t)L.R_max * L.f * 4);
  L.Q = take((size_t)L.R_max * dq * 4);
  L.O = take((size_t)L.R_max * dq * 4);
  L.P = take(part * 4);
  L.apart = take((size_t)c->max_batch * c->n_kv_heads * L.max_splits * 16 * c->head_dim * 4);
  L.astat = take((size_t)c->max_batch * c->n_kv_heads * L.max_splits * 16 * 2 * 4);
  L.logits = take((size_t)L.R_max * std::max(c->vocab, 1) * 4);
  L.nstat = gemm_stats_tiles(std::max(c->vocab, 1), L.g_lm, c->dtype);
  if (L.nstat == 0) L.nstat = std::max(L.nch, 1);
  L.mstats = take((size_t)L.R_max * L.nstat * 3 * 4);
  L.xss = take((size_t)std::max(L.g_qkv.S, 1) * L.R_max * 4);
  if (L.moe) {
    L.amax = L.R_max * 8;
    L.moe_idx = take((size_t)L.R_max * 8 * 4);
    if (c->n_experts > kRouteOne) L.moe_logits = take((size_t)L.R_max * 256 * 4);
    L.moe_w = take((size_t)L.R_max * 8 * 4);
    L.moe_aslot = take((size_t)L.R_max * 8 * 4);
    L.moe_counts = take((size_t)c->n_experts * 4);
    L.moe_offsets = take((size_t)(c->n_experts + 1) * 4);
    L.moe_arow = take((size_t)L.amax * 4);
    L.moe_h = take((size_t)L.amax * L.fe * 2);
    L.moe_y = take((size_t)L.amax * d * 4);
  }
  L.step_total = L.total = o;
  return L;
}

// The same buffers for the packed prompt passes, behind those of L.
Layout make_prompt_layout(const dbt_config *c, const Layout &step) {
  Layout L = step;
  const int d = c->d_model, dq = c->n_q_heads * c->head_dim, R = L.pack_rows;
  const size_t es = c->dtype == DBT_BF16 ? 2 : 4;
  if (R == 0) return L;
  size_t o = step.total;
  auto take = [&](size_t bytes) { size_t at = o; o += align256(bytes); return at; };
  L.prow = take((size_t)R * sizeof(PromptRow));
  L.ptiles = take((size_t)R * sizeof(PromptTile));
  L.S = take((size_t)R * d * 4);
  L.Xn = take((size_t)R * d * es);
  L.Xh = take((size_t)R * L.f * es);
  L.Q = take((size_t)R * dq * 4);
  L.O = take((size_t)R * dq * es);
  size_t part = std::max(prompt_part(L.g_qkv, L.nqkv, d, c->dtype, R, true), prompt_part(L.g_o, d, dq, c->dtype, R, false));
  if (L.moe)
    part = std::max({part, prompt_part(L.g_sgu, 2 * L.fs, d, c->dtype, R, true), prompt_part(L.g_sd, d, L.fs, c->dtype, R, false)});
  else
    part = std::max({part, prompt_part(L.g_gu, 2 * L.f, d, c->dtype, R, true), prompt_part(L.g_d, d, L.f, c->dtype, R, false)});
  L.part = part;
  L.P = take(part * 4);
  if (L.moe) {
    L.amax = R * c->top_k1;  // (the primary alone)
    L.moe_idx = take((size_t)R * 8 * 4);
    L.moe_tiles = take((size_t)(L.pack_rows * c->top_k1 / kTileExpert + c->n_experts + 1) * sizeof(int2));
    L.moe_ntiles = take(4);
    if (c->n_experts > kRouteOne) L.moe_logits = take((size_t)R * 256 * 4);
    L.moe_w = take((size_t)R * 8 * 4);
    L.moe_aslot = take((size_t)R * 8 * 4);
    L.moe_arow = take((size_t)L.amax * 4);
    L.moe_h = take((size_t)L.amax * L.fe * 2);
    L.moe_y = take((size_t)L.amax * d * 4);
  }
  L.total = o;
  return L;
}

}  // namespace

struct StageTimer {
  bool on = false;
  std::vector<std::pair<hipEvent_t, hipEvent_t>> ev;
  size_t used = 0;
};

struct dbt_model {
  StageTimer timers[DBT_STAGE_COUNT];
  // Second stream for the MoE shared expert, which runs beside the routing
  // chain (created by the first MoE layer of a call that may create it;
  // default priority), and the events of its fork and join.
  hipStream_t side = nullptr;
  hipEvent_t ev_fork = nullptr, ev_join = nullptr;
  bool no_fork = false;  // the current call creates no stream (allocation-free entry point)
  ~dbt_model() {
    for (auto &t : timers)
      for (auto &e : t.ev) {
        (void)hipEventDestroy(e.first);
        (void)hipEventDestroy(e.second);
      }
    if (ev_fork) (void)hipEventDestroy(ev_fork);
    if (ev_join) (void)hipEventDestroy(ev_join);
    if (side) (void)hipStreamDestroy(side);
  }
  dbt_config cfg;
  dbt_weights w;
  std::vector<dbt_layer_weights> layers;
  char *ws = nullptr;
  Layout L, Lp;  // Lp: the buffers of the packed prompt passes
  std::vector<float> rope_host;
  bool dev_ready = false;
  // boundary state: set by dbt_prefill(run_boundary = 0)
  const dbt_kv *bnd_kv = nullptr;
  int bnd_batch = 0;
  // Step buffers of the current call: the workspace's own step region, or
  // memory a call supplies for them (see decode_step_in).
  char *step = nullptr;
  char *p(size_t off) const {
    return off >= L.state_total && off < L.step_total ? step + (off - L.state_total) : ws + off;
  }
  template <typename T> T *at(size_t off) const { return (T *)p(off); }
};

struct dbt_kv {
  dbt_model *m;
  char *k, *v;
  int num_pages;
  int *page_table;
  int mpps;
  std::priority_queue<int, std::vector<int>, std::greater<int>> free_pages;
  std::vector<std::vector<int>> table;
  std::vector<int> len;
  struct Upd { int b, slot, page; };
  std::vector<Upd> pending;

  // whether the next position of sequence b is on a page it does not hold (a
  // failed step leaves the pages it took for the next one)
  bool needs_page(int b) const { return (size_t)len[b] == table[b].size() * kPage; }

  int take_page() {
    const int p = free_pages.top();
    free_pages.pop();
    return p;
  }
};

namespace {

size_t esize(const dbt_config &c) { return c.dtype == DBT_BF16 ? 2 : 4; }

// Records an event pair around the launches made during its lifetime when
// timing is enabled for the stage (a measurement aid; failures are ignored).
class Timed {
 public:
  Timed(dbt_model *m, int stage, hipStream_t st) : st_(st) {
    StageTimer &t = m->timers[stage];
    if (!t.on) return;
    if (t.used == t.ev.size()) {
      hipEvent_t a, b;
      if (hipEventCreate(&a) != hipSuccess) return;
      if (hipEventCreate(&b) != hipSuccess) { (void)hipEventDestroy(a); return; }
      t.ev.emplace_back(a, b);
    }
    pair_ = &t.ev[t.used++];
    (void)hipEventRecord(pair_->first, st_);
  }
  ~Timed() {
    if (pair_) (void)hipEventRecord(pair_->second, st_);
  }

 private:
  hipStream_t st_;
  std::pair<hipEvent_t, hipEvent_t> *pair_ = nullptr;
};

// K/V pages of one layer.
KVRef kv_layer(const dbt_kv *kv, int l) {
  const dbt_config &c = kv->m->cfg;
  KVRef r;
  const size_t per_layer = (size_t)kv->num_pages * c.n_kv_heads * kPage * c.head_dim * esize(c);
  r.k = kv->k + per_layer * l;
  r.v = kv->v + per_layer * l;
  r.page_table = kv->page_table;
  r.mpps = kv->mpps;
  r.n_kv = c.n_kv_heads;
  r.d_h = c.head_dim;
  return r;
}

dbt_status ensure_device(dbt_model *m, hipStream_t st) {
  if (m->dev_ready) return DBT_OK;
  HIPCHK(hipMemsetAsync(m->ws, 0, m->L.state_total, st));  // (step buffers need no clearing)
  HIPCHK(hipMemcpyAsync(m->p(m->L.rope), m->rope_host.data(), m->rope_host.size() * sizeof(float),
                        hipMemcpyHostToDevice, st));
  m->dev_ready = true;
  return DBT_OK;
}

// Enqueue pending page-table entries and (optionally) per-sequence positions:
// runs of consecutive pages (new sequences) as one launch of up to kPageRuns
// runs, single entries with the positions.  With `fold` the last block of
// those is returned there instead of launched, for the caller to pass to the
// step's first kernel.
dbt_status flush(dbt_kv *kv, const int *h_pos, int npos, hipStream_t st, StepBegin *fold = nullptr) {
  dbt_model *m = kv->m;
  if (fold) {
    fold->n_pos = fold->n_pt = 0;
    fold->b0 = 0;
  }
  // The list itself is left as it is until everything is enqueued (with `fold`:
  // until the step is, see step_done): after a failure the next call sends it
  // again.
  const std::vector<dbt_kv::Upd> &up = kv->pending;
  auto run_end = [&](size_t i) {  // end of the run of consecutive pages from entry i
    size_t e = i + 1;
    while (e < up.size() && up[e].b == up[i].b && up[e].slot == up[i].slot + (int)(e - i) &&
           up[e].page == up[i].page + (int)(e - i))
      ++e;
    return e;
  };
  PageRuns pr;
  pr.n = 0;
  size_t singles = 0;
  for (size_t i = 0, e; i < up.size(); i = e) {
    e = run_end(i);
    if (e == i + 1) {
      ++singles;
      continue;
    }
    pr.b[pr.n] = up[i].b;
    pr.slot[pr.n] = up[i].slot;
    pr.page[pr.n] = up[i].page;
    pr.count[pr.n] = (int)(e - i);
    if (++pr.n == kPageRuns) {
      HIPCHK(launch_page_runs(pr, kv->page_table, kv->mpps, st));
      pr.n = 0;
    }
  }
  HIPCHK(launch_page_runs(pr, kv->page_table, kv->mpps, st));
  size_t ip = 0;  // entries looked at
  int ipos = 0;
  while (singles > 0 || ipos < npos) {
    StepBegin sb;
    std::memset(&sb, 0, sizeof sb);
    sb.b0 = ipos;
    sb.n_pos = std::min(64, npos - ipos);
    for (int i = 0; i < sb.n_pos; ++i) sb.pos[i] = h_pos[ipos + i];
    ipos += sb.n_pos;
    while (sb.n_pt < 64 && singles > 0) {
      const size_t e = run_end(ip);
      if (e == ip + 1) {
        sb.pt_b[sb.n_pt] = up[ip].b;
        sb.pt_slot[sb.n_pt] = up[ip].slot;
        sb.pt_page[sb.n_pt++] = up[ip].page;
        --singles;
      }
      ip = e;
    }
    if (fold && singles == 0 && ipos >= npos) {
      *fold = sb;
      return DBT_OK;
    }
    HIPCHK(launch_step_begin(sb, m->at<int>(m->L.pos), kv->page_table, kv->mpps, st));
  }
  kv->pending.clear();
  return DBT_OK;
}

// One layer for the active rows.  rows_layout: rows of the partial slabs.
struct LayerCall {
  Rows rows;
  int mode;
  bool retain;
  bool prefill;
  PromptAttn tiles;  // prefill: the pass's attention tiles (list, count, positions per tile)
  int rows_layout;   // prefill: rows of the pass; decode: (1 + n_branches)*Bp
  bool last_norm;    // apply the next norm after the layer
  const dbt_step_out *out;  // routing outputs (MoE), may be NULL
  // layer 0 reads its rows straight from the step inputs (XNorm; no norm
  // kernel before it) when set; sb is then applied by its QKV projection
  const HIn *hin;
  const StepBegin *sb;
  HOut ho;  // where the last layer leaves the states (see HOut)
};

// Whether the decode attention of B sequences, the longest of maxlen positions
// after the append, reads each (sequence, KV head) in one workgroup: bf16 where
// the batch fills the chip (and the kernel holds the page ids), fp32 where no
// sequence needs a second split.
bool attn_single(const dbt_model *m, int B, int maxlen) {
  const dbt_config &cf = m->cfg;
  const int npages = (maxlen + kPage - 1) / kPage;
  if (cf.dtype != DBT_BF16) return npages <= m->L.split_target;
  return B * cf.n_kv_heads >= kComputeUnits && npages <= kSplitMaxBf16;
}

// Whether the first layer of a layer-only model takes its rows straight from
// the step inputs (XNorm) for a decode step of B sequences.  Decided from
// the model and batch only, so the grouped, primary-only and two-pass steps
// (and a branch pass) all use the same arithmetic for a row.
bool input_fold(const dbt_model *m, int B) {
  const dbt_config &cf = m->cfg;
  if (cf.has_embeddings || cf.dtype != DBT_BF16 || cf.d_model % 128) return false;
  // the largest call of a step: every path's rows, or the primary's alone
  // when only it attends (compute-matched)
  const int Bp = round16(B), M = (cf.compute_matched ? 1 : 1 + n_branches(cf)) * Bp;
  return gemm_xnorm_ok(m->L.g_qkv, M);
}

// MoE MLP of layer l for the active rows: route, dispatch, touched experts,
// shared expert (with the b coupling), combine (with the c coupling).
dbt_status run_moe_mlp(dbt_model *m, int l, const LayerCall &c, hipStream_t st) {
  const dbt_config &cf = m->cfg;
  const Layout &L = c.prefill ? m->Lp : m->L;
  const PromptRow *map = c.prefill ? m->at<PromptRow>(L.prow) : nullptr;
  const dbt_layer_weights &W = m->layers[l];
  const int d = cf.d_model, fs = L.fs;
  const size_t es = esize(cf);
  float *P = m->at<float>(L.P), *S = m->at<float>(L.S);
  const size_t rq = (size_t)l * L.Bp_max;
  float *ret_h = m->at<float>(L.ret_h) + rq * L.f;
  float *ret_m = m->at<float>(L.ret_m) + rq * d;
  int *ret_idx = m->at<int>(L.ret_idx) + rq * 8;
  const int k2 = cf.replay ? cf.top_k1 : cf.top_k2;
  MoeRoute ro{};
  ro.Sbar = S;
  ro.g = W.mlp_norm;
  ro.eps = cf.rms_eps;
  ro.d = d;
  ro.Wr = W.router;
  ro.E = cf.n_experts;
  ro.k1 = cf.top_k1;
  ro.k2 = k2;
  ro.replay = cf.replay;
  ro.rows = c.rows;
  ro.mode = c.mode;
  ro.logits = m->at<float>(L.moe_logits);
  ro.idx = m->at<int>(L.moe_idx);
  ro.wts = m->at<float>(L.moe_w);
  ro.idx1_in = ret_idx;
  if (c.out && !c.prefill) {
    const size_t B = c.rows.B;
    ro.out_idx1 = c.out->route_idx1 ? c.out->route_idx1 + (size_t)l * B * cf.top_k1 : nullptr;
    ro.out_w1 = c.out->route_w1 ? c.out->route_w1 + (size_t)l * B * cf.top_k1 : nullptr;
    ro.out_idx2 = c.out->route_idx2 ? c.out->route_idx2 + (size_t)l * B * k2 : nullptr;
    ro.out_w2 = c.out->route_w2 ? c.out->route_w2 + (size_t)l * B * k2 : nullptr;
    const size_t E = cf.n_experts;
    ro.out_lg1 = c.out->route_logits1 ? c.out->route_logits1 + (size_t)l * B * E : nullptr;
    ro.out_lg2 = c.out->route_logits2 ? c.out->route_logits2 + (size_t)l * B * E : nullptr;
  }
  ro.ret_idx = c.retain ? ret_idx : nullptr;
  ro.ret_map = map;
  // The shared expert needs only the normed rows: it runs on a second stream
  // beside the routing chain (router, top-k, dispatch: short kernels that
  // leave most compute units idle) and the routed experts; the combine waits
  // for both.  Neither side writes what the other reads (shared: P, Xh;
  // routed: the MoE buffers).
  struct Fork {
    dbt_model *m;
    hipStream_t st;
    bool on;
    ~Fork() {
      if (!on) return;
      (void)hipEventRecord(m->ev_join, m->side);
      (void)hipStreamWaitEvent(st, m->ev_join, 0);
    }
  } fork{m, st, false};
  hipStream_t sst = st;
  const bool has_shared = fs > 0 && !(cf.compute_matched && c.mode == MODE_BRANCH);
  if (has_shared && !m->no_fork) {
    if (!m->side) {
      HIPCHK(hipStreamCreateWithFlags(&m->side, hipStreamNonBlocking));
      // device-scope release: the hand-off is between two queues of one GPU
      // (a system-scope release would also write the caches back for the host)
      HIPCHK(hipEventCreateWithFlags(&m->ev_fork, hipEventDisableTiming | hipEventReleaseToDevice));
      HIPCHK(hipEventCreateWithFlags(&m->ev_join, hipEventDisableTiming | hipEventReleaseToDevice));
    }
    HIPCHK(hipEventRecord(m->ev_fork, st));
    HIPCHK(hipStreamWaitEvent(m->side, m->ev_fork, 0));
    sst = m->side;
    fork.on = true;
  }
  // shared expert: dense SwiGLU of width fs with the b coupling on its
  // intermediate; compute-matched variant (App. B.3): primary rows only
  const bool cm = cf.compute_matched != 0;
  const Rows srows = cm ? Rows{c.rows.B, c.rows.Bp, 0, 1} : c.rows;
  const int smode = cm ? (int)MODE_PRIMARY : c.mode;
  const int sxrow0 = srows.p0 * srows.Bp, sM = srows.np * srows.Bp;
  long long stride = (long long)c.rows_layout * d;
  int S_sh = 0;
  if (fs > 0 && !(cm && c.mode == MODE_BRANCH)) {
    GemmConfig g_sgu = L.g_sgu, g_sd = L.g_sd;
    if (c.prefill) {  // as in run_layer
      g_sgu.S = sM < kTileRows ? prompt_splits(g_sgu, sM) : 1;
      g_sd.S = sM < kTileRows ? prompt_splits(g_sd, sM) : 1;
    }
    WSegs gu{{W.s_gate, W.s_up, nullptr}, {fs, fs, 0}};
    long long st_gu = (long long)c.rows_layout * 2 * fs;
    const Retain keep{c.retain && !cm ? ret_h : nullptr, map};
    TileGemm tg{}, td{};
    tg.w[0] = (const uint16_t *)W.s_gate;
    tg.w[1] = (const uint16_t *)W.s_up;
    tg.rows[0] = tg.rows[1] = tg.N = fs;
    tg.K = d;
    tg.X = (const uint16_t *)(m->p(L.Xn) + (size_t)sxrow0 * d * es);
    tg.ldx = d;
    tg.M = sM;
    tg.H = (uint16_t *)(m->p(L.Xh) + (size_t)sxrow0 * fs * es);
    tg.ldh = fs;
    tg.ret = keep;
    if (c.prefill && gemm_tile_args_ok(tg, true)) {
      HIPCHK(launch_gemm_tile(tg, true, sst));
    } else {
      if ((size_t)g_sgu.S * (size_t)st_gu > L.part) return fail(DBT_ERR_STATE, "internal: shared-expert slabs");
      HIPCHK(launch_gemm(gu, 2 * fs, d, cf.dtype, m->p(L.Xn) + (size_t)sxrow0 * d * es, d, sM,
                         P + (size_t)sxrow0 * 2 * fs, 2 * fs, st_gu, g_sgu, sst));
      HIPCHK(launch_swiglu_finish(P, st_gu, g_sgu.S, 2 * fs, fs, smode, srows, W.b, ret_h, keep, cf.dtype,
                                  m->p(L.Xh), fs, sst));
    }
    WSegs sd{{W.s_down, nullptr, nullptr}, {d, 0, 0}};
    td.w[0] = (const uint16_t *)W.s_down;
    td.rows[0] = td.N = d;
    td.K = fs;
    td.X = tg.H;
    td.ldx = fs;
    td.M = sM;
    td.Y = P + (size_t)sxrow0 * d;
    td.ldy = d;
    if (c.prefill && gemm_tile_args_ok(td, false)) {
      td.splits = g_sd.S = gemm_tile_splits(d, fs, sM);
      td.y_stride = stride;
    }
    if ((size_t)g_sd.S * (size_t)stride > L.part) return fail(DBT_ERR_STATE, "internal: shared-expert slabs");
    if (td.splits) {
      HIPCHK(launch_gemm_tile(td, false, sst));
    } else {
      HIPCHK(launch_gemm(sd, d, fs, cf.dtype, m->p(L.Xh) + (size_t)sxrow0 * fs * es, fs, sM, P + (size_t)sxrow0 * d,
                         d, stride, g_sd, sst));
    }
    S_sh = g_sd.S;
  }
  HIPCHK(launch_moe_route(ro, st));
  MoeDispatch di{};
  di.idx = ro.idx;
  di.rows = c.rows;
  di.k1 = cf.top_k1;
  di.k2 = k2;
  di.E = cf.n_experts;
  di.counts = m->at<int>(L.moe_counts);
  di.offsets = m->at<int>(L.moe_offsets);
  di.arow = m->at<int>(L.moe_arow);
  di.aslot = m->at<int>(L.moe_aslot);
  const int max_rows = c.rows.np * c.rows.B;
  // The experts' products of a prompt pass with enough rows per expert on the
  // tiled kernel (see kExpertTileRows).
  TileGemm xg{}, xd{};
  if (c.prefill && (long long)max_rows * cf.top_k1 >= (long long)kExpertTileRows * cf.n_experts) {
    di.tiles = m->at<int2>(L.moe_tiles);
    di.ntiles = m->at<int>(L.moe_ntiles);
    xg.w[0] = (const uint16_t *)W.x_gate;
    xg.w[1] = (const uint16_t *)W.x_up;
    xg.rows[0] = xg.rows[1] = xg.N = L.fe;
    xg.K = d;
    xg.X = (const uint16_t *)m->p(L.Xn);
    xg.ldx = d;
    xg.M = max_rows;
    xg.H = (uint16_t *)m->p(L.moe_h);
    xg.ldh = L.fe;
    xg.tiles = di.tiles;
    xg.ntiles = di.ntiles;
    xg.counts = di.counts;
    xg.offsets = di.offsets;
    xg.arow = di.arow;
    xg.max_tiles = max_rows * cf.top_k1 / kTileExpert + std::min(cf.n_experts, max_rows * cf.top_k1);
    xd = xg;
    xd.w[0] = (const uint16_t *)W.x_down;
    xd.rows[0] = xd.N = d;
    xd.K = L.fe;
    xd.X = xg.H;
    xd.ldx = L.fe;
    xd.M = max_rows * cf.top_k1;
    xd.H = nullptr;
    xd.Y = m->at<float>(L.moe_y);
    xd.ldy = d;
    xd.arow = nullptr;
  }
  const bool tiled = di.tiles && gemm_tile_experts_ok(xg) && gemm_tile_experts_ok(xd);
  HIPCHK(launch_moe_dispatch(di, st));
  if (tiled) {
    Timed tm(m, DBT_STAGE_GATEUP, st);
    HIPCHK(launch_gemm_tile_experts(xg, true, st));
  } else {
    Timed tm(m, DBT_STAGE_GATEUP, st);
    MoeGemm g{};
    g.X = m->p(L.Xn);
    g.ldx = d;
    g.W0 = W.x_gate;
    g.W1 = W.x_up;
    g.E = cf.n_experts;
    g.N = L.fe;
    g.K = d;
    g.counts = di.counts;
    g.offsets = di.offsets;
    g.arow = di.arow;
    g.Y = m->p(L.moe_h);
    g.ldy = L.fe;
    HIPCHK(launch_moe_gemm(g, true, max_rows, st));
  }
  if (tiled) {
    Timed tm(m, DBT_STAGE_DOWN, st);
    HIPCHK(launch_gemm_tile_experts(xd, false, st));
  } else {
    Timed tm(m, DBT_STAGE_DOWN, st);
    MoeGemm g{};
    g.X = m->p(L.moe_h);
    g.ldx = L.fe;
    g.W0 = W.x_down;
    g.E = cf.n_experts;
    g.N = d;
    g.K = L.fe;
    g.counts = di.counts;
    g.offsets = di.offsets;
    g.arow = di.arow;
    g.Y = m->p(L.moe_y);
    g.ldy = d;
    HIPCHK(launch_moe_gemm(g, false, max_rows, st));
  }
  if (fork.on) {
    HIPCHK(hipEventRecord(m->ev_join, m->side));
    HIPCHK(hipStreamWaitEvent(st, m->ev_join, 0));
    fork.on = false;
  }
  const float *g_next = nullptr;
  if (l + 1 < cf.n_layers) g_next = m->layers[l + 1].attn_norm;
  else if (cf.vocab > 0 && c.last_norm) g_next = m->w.final_norm;
  MoeCombine cb{};
  cb.rows = c.rows;
  cb.mode = c.mode;
  cb.d = d;
  cb.k1 = cf.top_k1;
  cb.k2 = k2;
  cb.idx = ro.idx;
  cb.wts = ro.wts;
  cb.aslot = di.aslot;
  cb.Yexp = m->at<float>(L.moe_y);
  cb.part = P;
  cb.stride = stride;
  cb.S_sh = S_sh;
  cb.c = W.c;
  cb.M1_in = ret_m;  // compute-matched: the kept G1
  cb.ret = Retain{c.retain ? ret_m : nullptr, map};
  cb.gG = cm ? W.g_shared_copy : nullptr;
  cb.S = S;
  if (l + 1 == cf.n_layers) cb.ho = c.ho;
  cb.g_next = g_next;
  cb.eps = cf.rms_eps;
  cb.Xn = m->p(L.Xn);
  cb.ldx = d;
  HIPCHK(launch_moe_combine(cb, cf.dtype, st));
  return DBT_OK;
}

dbt_status run_layer(dbt_model *m, dbt_kv *kv, int l, const LayerCall &c, hipStream_t st) {
  const dbt_config &cf = m->cfg;
  const Layout &L = c.prefill ? m->Lp : m->L;
  const PromptRow *map = c.prefill ? m->at<PromptRow>(L.prow) : nullptr;
  const dbt_layer_weights &W = m->layers[l];
  const int d = cf.d_model, dq = cf.n_q_heads * cf.head_dim, dkv = cf.n_kv_heads * cf.head_dim, f = L.f;
  const size_t es = esize(cf);
  const int xrow0 = c.rows.p0 * c.rows.Bp;
  const int M = c.rows.np * c.rows.Bp;
  char *Xn = m->p(L.Xn), *Xh = m->p(L.Xh), *O = m->p(L.O);
  float *P = m->at<float>(L.P), *S = m->at<float>(L.S), *Q = m->at<float>(L.Q);
  // prompt-wide rows: no reduction split (plenty of row tiles), but for a
  // short pass, which the streaming kernel runs like a step
  auto cfg = [&](GemmConfig g) {
    if (c.prefill) g.S = M < kTileRows && cf.dtype == DBT_BF16 ? prompt_splits(g, M) : 1;
    return g;
  };
  // A projection of the active rows: the tiled kernel over a pass of prompts
  // (256 rows and more), the weight-streaming kernel otherwise.
  // S: its reduction splits.
  auto project = [&](const WSegs &segs, int N, int K, const char *X, int ldx, int rows_M, float *Y, int ldy,
                     long long y_stride, const GemmConfig &g, int &S) -> hipError_t {
    TileGemm tg{};
    for (int i = 0; i < 3; ++i) {
      tg.w[i] = (const uint16_t *)segs.w[i];
      tg.rows[i] = segs.rows[i];
    }
    tg.N = N;
    tg.K = K;
    tg.X = (const uint16_t *)X;
    tg.ldx = ldx;
    tg.M = rows_M;
    tg.Y = Y;
    tg.ldy = ldy;
    S = g.S;
    if (c.prefill && cf.dtype == DBT_BF16 && gemm_tile_args_ok(tg, false)) {
      tg.splits = S = gemm_tile_splits(N, K, rows_M);
      tg.y_stride = y_stride;
    }
    if ((size_t)S * (size_t)y_stride > L.part) return hipErrorInvalidValue;  // (y_stride: the rows of every path)
    if (tg.splits) return launch_gemm_tile(tg, false, st);
    return launch_gemm(segs, N, K, cf.dtype, X, ldx, rows_M, Y, ldy, y_stride, g, st);
  };
  const GemmConfig g_qkv = cfg(L.g_qkv), g_o = cfg(L.g_o), g_gu = cfg(L.g_gu), g_d = cfg(L.g_d);
  const int S_gu = g_gu.S;
  int S_qkv = g_qkv.S, S_o = 1, S_d = 1;
  KVRef kvl = kv_layer(kv, l);
  const size_t rq = (size_t)l * L.Bp_max;
  float *ret_q = m->at<float>(L.ret_q) + rq * dq;
  float *ret_h = m->at<float>(L.ret_h) + rq * f;
  float *ret_m = m->at<float>(L.ret_m) + rq * d;
  // Compute-matched variant (App. B.3): attention runs on the primary rows
  // only and the branch takes g_A * A1 in the residual step.
  const bool cm = cf.compute_matched != 0;
  float *ret_a = cm ? m->at<float>(L.ret_a) + rq * d : nullptr;
  const HIn hin0 = l == 0 && c.hin ? *c.hin : HIn{};
  if (cm && c.mode == MODE_BRANCH) {
    if (hin0.h1 && c.sb) HIPCHK(launch_step_begin(*c.sb, m->at<int>(L.pos), kv->page_table, kv->mpps, st));
    HIPCHK(launch_resid_norm(P, 0, 0, d, S, W.mlp_norm, cf.rms_eps, d, cf.dtype, c.rows, Xn, d, st,
                             GatedCopy{W.g_attn_copy, ret_a, Retain{}}, hin0));
    return run_moe_mlp(m, l, c, st);
  }
  const Rows arows = cm ? Rows{c.rows.B, c.rows.Bp, 0, 1} : c.rows;
  const int amode = cm ? (int)MODE_PRIMARY : c.mode;
  const int axrow0 = arows.p0 * arows.Bp, aM = arows.np * arows.Bp;

  // 1. stacked QKV projection (branch rows need only W_Q)
  WSegs qkv{};
  int nq;
  if (amode == MODE_BRANCH) {
    qkv = WSegs{{W.wq, nullptr, nullptr}, {dq, 0, 0}};
    nq = dq;
  } else {
    qkv = WSegs{{W.wq, W.wk, W.wv}, {dq, dkv, dkv}};
    nq = L.nqkv;
  }
  long long stride = (long long)c.rows_layout * nq;
  // A whole prompt: the tiled projection applies the rotary embedding and
  // writes Q and the cache itself (no fp32 Q/K/V slab, no finish kernel).
  TileGemm tq{};
  if (c.prefill && amode == MODE_PRIMARY && cf.dtype == DBT_BF16) {
    for (int i = 0; i < 3; ++i) {
      tq.w[i] = (const uint16_t *)qkv.w[i];
      tq.rows[i] = qkv.rows[i];
    }
    tq.N = nq;
    tq.K = d;
    tq.X = (const uint16_t *)(Xn + (size_t)axrow0 * d * es);
    tq.ldx = d;
    tq.M = aM;
    tq.rope = m->at<float2>(L.rope);
    tq.Qout = Q;
    tq.kv = kvl;
    tq.prompt = map;
    tq.ret = Retain{c.retain && !cm ? ret_q : nullptr, map};
  }
  const bool qkv_fused = tq.rope && gemm_tile_args_ok(tq, false);
  // Decode on the bf16 cache: the attention kernel finishes the queries and
  // appends the cache entry itself.
  int maxlen = 0;
  if (!c.prefill)
    for (int b = 0; b < c.rows.B; ++b) maxlen = std::max(maxlen, kv->len[b] + 1);  // (the boundary: one too many)
  const bool finish_in_attn = !c.prefill && cf.dtype == DBT_BF16;
  const bool xin = l == 0 && c.hin && c.hin->h1;
  if (xin && (c.prefill || !finish_in_attn || cf.dtype != DBT_BF16 || !gemm_xnorm_ok(g_qkv, aM)))
    return fail(DBT_ERR_STATE, "internal: first-layer input fold on an unsupported call");
  if (qkv_fused) {
    Timed tm(m, DBT_STAGE_QKV, st);
    HIPCHK(launch_gemm_tile(tq, false, st));
  } else if (xin) {
    XNorm xn{};
    xn.h = *c.hin;
    xn.rows = arows;
    xn.g = W.attn_norm;
    xn.ss = m->at<float>(L.xss);
    xn.ss_ld = L.R_max;
    if (c.sb) {
      xn.sb = *c.sb;
      xn.pos_arr = m->at<int>(L.pos);
      xn.page_table = kv->page_table;
      xn.mpps = kv->mpps;
    }
    Timed tm(m, DBT_STAGE_QKV, st);
    HIPCHK(launch_gemm_xnorm(qkv, nq, d, xn, aM, P + (size_t)axrow0 * nq, nq, stride, g_qkv, st));
  } else {
    Timed tm(m, DBT_STAGE_QKV, st);
    HIPCHK(project(qkv, nq, d, Xn + (size_t)axrow0 * d * es, d, aM, P + (size_t)axrow0 * nq, nq, stride, g_qkv, S_qkv));
  }
  QKVFinish qf{};
  qf.part = P;
  qf.split_stride = stride;
  qf.S = S_qkv;
  qf.ldp = nq;
  qf.n_q = cf.n_q_heads;
  qf.n_kv = cf.n_kv_heads;
  qf.d_h = cf.head_dim;
  qf.rows = arows;
  qf.mode = amode;
  qf.rope = m->at<float2>(L.rope);
  qf.pos_arr = c.prefill ? nullptr : m->at<int>(L.pos);
  qf.prompt = map;
  qf.a = W.a;
  qf.Q = Q;
  qf.Q1_in = ret_q;
  qf.ret = Retain{c.retain && !cm ? ret_q : nullptr, map};
  qf.kv = kvl;
  qf.dtype = cf.dtype;
  if (xin) {
    qf.ss = m->at<float>(L.xss);
    qf.ss_ld = L.R_max;
    qf.ss_S = S_qkv;
    qf.d_model = d;
    qf.eps = cf.rms_eps;
  }
  if (!qkv_fused && !finish_in_attn) HIPCHK(launch_qkv_finish(qf, st));

  // 2. attention over the primary cache
  if (c.prefill) {
    PromptAttn pa = c.tiles;
    pa.Q = Q;
    pa.ldq = dq;
    pa.kv = kvl;
    pa.n_q = cf.n_q_heads;
    pa.dtype = cf.dtype;
    pa.O = O;
    pa.ldo = dq;
    HIPCHK(launch_attn_prefill(pa, st));
  } else {
    AttnArgs aa{};
    aa.Q = Q;
    aa.kv = kvl;
    aa.pos_arr = m->at<int>(L.pos);
    aa.rows = arows;
    aa.n_q = cf.n_q_heads;
    aa.pages_per_split = L.split_target;
    aa.max_splits = L.max_splits;
    aa.opart = m->at<float>(L.apart);
    aa.ostat = m->at<float>(L.astat);
    aa.dtype = cf.dtype;
    // When the batch fills the chip (B x n_kv >= 256 workgroups), each
    // (sequence, KV head) is read by one eight-wave workgroup and no partials
    // are merged.  The choice depends on the batch, never on the branch.
    aa.single = attn_single(m, c.rows.B, maxlen);
    aa.fin = qf;
    aa.O = O;
    aa.ldo = dq;
    {
      Timed tm(m, DBT_STAGE_ATTN, st);
      HIPCHK(launch_attn_decode(aa, st));
    }
    // (a sequence of one split is written by the kernel itself)
    if (!aa.single && (maxlen + kPage - 1) / kPage > L.split_target) HIPCHK(launch_attn_combine(aa, O, dq, st));
  }

  // 3. output projection + residual + MLP norm
  WSegs wo{{W.wo, nullptr, nullptr}, {d, 0, 0}};
  stride = (long long)c.rows_layout * d;
  {
    Timed tm(m, DBT_STAGE_WO, st);
    HIPCHK(project(wo, d, dq, O + (size_t)axrow0 * dq * es, dq, aM, P + (size_t)axrow0 * d, d, stride, g_o, S_o));
  }
  const GatedCopy gca = cm ? GatedCopy{W.g_attn_copy, ret_a, Retain{c.retain ? ret_a : nullptr, map}}
                           : GatedCopy{};
  HIPCHK(launch_resid_norm(P, stride, S_o, d, S, W.mlp_norm, cf.rms_eps, d, cf.dtype, c.rows, Xn, d, st, gca, hin0));

  if (L.moe) return run_moe_mlp(m, l, c, st);

  // 4. gate/up + SwiGLU + b coupling (fused into the projection's epilogue
  // when the tiles fill the chip)
  const Retain ret_h_keep{c.retain ? ret_h : nullptr, map};
  TileGemm tg{};
  if (c.prefill && c.mode == MODE_PRIMARY && c.rows.np == 1 && cf.dtype == DBT_BF16) {
    tg.w[0] = (const uint16_t *)W.w_gate;
    tg.w[1] = (const uint16_t *)W.w_up;
    tg.rows[0] = tg.rows[1] = f;
    tg.N = f;
    tg.K = d;
    tg.X = (const uint16_t *)(Xn + (size_t)xrow0 * d * es);
    tg.ldx = d;
    tg.M = M;
    tg.H = (uint16_t *)(Xh + (size_t)xrow0 * f * es);
    tg.ldh = f;
    tg.ret = ret_h_keep;
  }
  if (tg.w[0] && gemm_tile_args_ok(tg, true)) {
    Timed tm(m, DBT_STAGE_GATEUP, st);
    HIPCHK(launch_gemm_tile(tg, true, st));
  } else if (c.prefill ? gemm_glu_ok(f, M, c.rows.np, cf.dtype) : L.glu) {
    const GluEpi ep{c.rows, c.mode, f, W.b, ret_h, ret_h_keep, (uint16_t *)Xh, f};
    Timed tm(m, DBT_STAGE_GATEUP, st);
    HIPCHK(launch_gemm_glu((const uint16_t *)W.w_gate, (const uint16_t *)W.w_up, f, d, Xn + (size_t)xrow0 * d * es,
                           d, M, ep, st));
  } else {
    WSegs gu{{W.w_gate, W.w_up, nullptr}, {f, f, 0}};
    stride = (long long)c.rows_layout * 2 * f;
    {
      Timed tm(m, DBT_STAGE_GATEUP, st);
      if ((size_t)S_gu * (size_t)stride > L.part) return fail(DBT_ERR_STATE, "internal: gate/up slabs");
      HIPCHK(launch_gemm(gu, 2 * f, d, cf.dtype, Xn + (size_t)xrow0 * d * es, d, M, P + (size_t)xrow0 * 2 * f,
                         2 * f, stride, g_gu, st));
    }
    HIPCHK(launch_swiglu_finish(P, stride, S_gu, 2 * f, f, c.mode, c.rows, W.b, ret_h, ret_h_keep, cf.dtype, Xh, f,
                                st));
  }

  // 5. down projection + c coupling + residual + next norm
  WSegs wd{{W.w_down, nullptr, nullptr}, {d, 0, 0}};
  stride = (long long)c.rows_layout * d;
  {
    Timed tm(m, DBT_STAGE_DOWN, st);
    HIPCHK(project(wd, d, f, Xh + (size_t)xrow0 * f * es, f, M, P + (size_t)xrow0 * d, d, stride, g_d, S_d));
  }
  const float *g_next = nullptr;
  if (l + 1 < cf.n_layers) g_next = m->layers[l + 1].attn_norm;
  else if (cf.vocab > 0 && c.last_norm) g_next = m->w.final_norm;
  HIPCHK(launch_down_finish(P, stride, S_d, d, d, c.mode, c.rows, W.c, ret_m,
                            Retain{c.retain ? ret_m : nullptr, map}, S, g_next, cf.rms_eps,
                            cf.dtype, Xn, d, st, l + 1 == cf.n_layers ? c.ho : HOut{}));
  return DBT_OK;
}

// Step inputs for the active rows: embeddings (Eq. (7)) or given residuals,
// then the first layer's attention norm.
dbt_status load_inputs(dbt_model *m, dbt_kv *kv, const dbt_step_in *in, const int *tokens, Rows rows,
                       hipStream_t st, const StepBegin *sb = nullptr) {
  const dbt_config &cf = m->cfg;
  const Layout &L = m->L;
  const float *g0 = m->layers[0].attn_norm;
  if (cf.has_embeddings) {
    HIPCHK(launch_embed(tokens, cf.vocab, m->w.emb1, m->w.emb2, m->w.emb_norm, g0, cf.rms_eps, cf.d_model, cf.dtype, rows,
                        m->at<float>(L.S), m->p(L.Xn), cf.d_model, st, sb, m->at<int>(L.pos), kv->page_table,
                        kv->mpps));
  } else {
    HIPCHK(launch_load_hidden(in->h1_in, in->h2_in, g0, cf.rms_eps, cf.d_model, cf.dtype, rows, m->at<float>(L.S),
                              m->p(L.Xn), cf.d_model, st, sb, m->at<int>(L.pos), kv->page_table, kv->mpps));
  }
  return DBT_OK;
}

// Where a call leaves its logits and states.  An output array takes them
// straight from the kernel that computes them when it is 16-byte aligned and
// shares no memory with another output; otherwise (or with no array) they go to
// the workspace, and the array is filled by a copy at the end of the call
// (arrays that overlap then hold what the last copy leaves: the readout's
// outputs, logits1, logits2, h1_out, h2_out in this order).
struct Sinks {
  const float *z[4];  // logits of path j, row b at z[j] + b*V
  bool copy_z1, copy_z2, copy_h1, copy_h2;
  HOut ho;
};

struct Span {
  const void *p;
  size_t bytes;
};

bool overlap(const Span &a, const Span &b) {
  return (uintptr_t)a.p < (uintptr_t)b.p + b.bytes && (uintptr_t)b.p < (uintptr_t)a.p + a.bytes;
}

// direct1 / direct2: whether the primary's / the branches' outputs may leave
// the call early (every later read of the call is of other memory).  late: an
// input that is still read when the first states leave.
Sinks make_sinks(const dbt_model *m, int B, int Bp, const dbt_step_out *out, bool direct1, bool direct2,
                 const Span &late = Span{}) {
  const dbt_config &cf = m->cfg;
  const int nb = n_branches(cf);
  const size_t V = cf.vocab, zrow = (size_t)B * V * 4, hrow = (size_t)B * cf.d_model * 4;
  Sinks k{};
  for (int j = 0; j <= nb; ++j) k.z[j] = m->at<float>(m->L.logits) + (size_t)j * Bp * V;
  if (!out) return k;
  const size_t rows = (size_t)cf.n_layers * B * 4, k1 = rows * cf.top_k1, k2 = rows * (cf.replay ? cf.top_k1 : cf.top_k2),
               re = rows * cf.n_experts;
  Span all[13];
  int n = 0;
  auto add = [&](const void *p, size_t bytes) {
    if (p) all[n++] = Span{p, bytes};
  };
  add(out->logits1, zrow);
  add(out->logits2, zrow * nb);
  add(out->h1_out, hrow);
  add(out->h2_out, hrow * nb);
  add(out->alpha, (size_t)B * 4);
  add(out->next_token, (size_t)B * 4);
  if (cf.n_experts > 0) {
    add(out->route_idx1, k1);
    add(out->route_idx2, k2);
    add(out->route_w1, k1);
    add(out->route_w2, k2);
    add(out->route_logits1, re);
    add(out->route_logits2, re);
  }
  add(late.p, late.bytes);
  auto fits = [&](const void *p) {  // one of the first four
    if (!p || (uintptr_t)p % 16) return false;
    for (int i = 0; i < n; ++i)
      if (all[i].p == p)
        for (int j = 0; j < n; ++j)
          if (i != j && overlap(all[i], all[j])) return false;
    return true;
  };
  k.copy_z1 = V > 0 && out->logits1;
  k.copy_z2 = V > 0 && out->logits2;
  k.copy_h1 = out->h1_out != nullptr;
  k.copy_h2 = out->h2_out != nullptr;
  k.ho.B = B;
  if (k.copy_z1 && direct1 && fits(out->logits1)) {
    k.z[0] = out->logits1;
    k.copy_z1 = false;
  }
  if (k.copy_z2 && direct2 && fits(out->logits2)) {
    for (int j = 0; j < nb; ++j) k.z[1 + j] = out->logits2 + (size_t)j * B * V;
    k.copy_z2 = false;
  }
  if (k.copy_h1 && direct1 && fits(out->h1_out)) {
    k.ho.h1 = out->h1_out;
    k.copy_h1 = false;
  }
  if (k.copy_h2 && direct2 && fits(out->h2_out)) {
    k.ho.h2 = out->h2_out;
    k.copy_h2 = false;
  }
  return k;
}

// Final norm is already in Xn (applied by the last layer); output matrix for the active rows.
dbt_status lm_head(dbt_model *m, Rows rows, const Sinks &k, hipStream_t st) {
  const dbt_config &cf = m->cfg;
  const Layout &L = m->L;
  const int xrow0 = rows.p0 * rows.Bp;
  WSegs lm{{m->w.lm_head, nullptr, nullptr}, {cf.vocab, 0, 0}};
  YRows yr{};
  for (int j = 0; j < rows.np; ++j) yr.p[j] = const_cast<float *>(k.z[rows.p0 + j]);
  yr.Bp = rows.Bp;
  yr.B = rows.B;
  Timed tm(m, DBT_STAGE_LMHEAD, st);
  const bool fused = gemm_stats_tiles(cf.vocab, L.g_lm, cf.dtype) > 0;
  HIPCHK(launch_gemm(lm, cf.vocab, cf.d_model, cf.dtype, m->p(L.Xn) + (size_t)xrow0 * cf.d_model * esize(cf),
                     cf.d_model, rows.np * rows.Bp, nullptr, cf.vocab, 0, L.g_lm, st,
                     fused ? m->at<float>(L.mstats) + (size_t)xrow0 * L.nstat * 3 : nullptr, &yr));
  return DBT_OK;
}

// Mixture readout from the logits at k, and the copies of those the
// projection did not write in place.
dbt_status readout(dbt_model *m, int B, int Bp, bool branch, dbt_step_out *out, const Sinks &k, hipStream_t st) {
  const dbt_config &cf = m->cfg;
  const Layout &L = m->L;
  if (cf.vocab <= 0) return DBT_OK;
  MixArgs mx{};
  for (int j = 0; j < 4; ++j) mx.z[j] = k.z[j];
  mx.V = cf.vocab;
  const int nb = n_branches(cf);
  mx.rows = Rows{B, Bp, 0, branch ? 1 + nb : 1};
  mx.chunk = kMixChunk;
  mx.stats = m->at<float>(L.mstats);
  mx.stats_ready = gemm_stats_tiles(cf.vocab, L.g_lm, cf.dtype) > 0;
  mx.tile_w = mx.stats_ready ? gemm_tile_rows(L.g_lm) : kMixChunk;
  mx.nstat = L.nstat;
  mx.alpha = out ? out->alpha : nullptr;
  mx.next = out ? out->next_token : nullptr;
  if (mx.alpha || mx.next) {
    Timed tm(m, DBT_STAGE_MIX, st);
    HIPCHK(launch_mixture(mx, st));
  }
  if (k.copy_z1)
    HIPCHK(hipMemcpyAsync(out->logits1, k.z[0], (size_t)B * cf.vocab * 4, hipMemcpyDeviceToDevice, st));
  if (k.copy_z2 && branch)
    for (int j = 0; j < nb; ++j)
      HIPCHK(hipMemcpyAsync(out->logits2 + (size_t)j * B * cf.vocab, k.z[1 + j], (size_t)B * cf.vocab * 4,
                            hipMemcpyDeviceToDevice, st));
  return DBT_OK;
}

// Final residual states of the branches: [n_branches][B][d].
dbt_status copy_branch_rows(dbt_model *m, float *dst, int B, int Bp, hipStream_t st) {
  const int d = m->cfg.d_model;
  for (int j = 0; j < n_branches(m->cfg); ++j)
    HIPCHK(hipMemcpyAsync(dst + (size_t)j * B * d, m->at<float>(m->L.S) + (size_t)(1 + j) * Bp * d, (size_t)B * d * 4,
                          hipMemcpyDeviceToDevice, st));
  return DBT_OK;
}

dbt_status check_model_kv(dbt_model *m, dbt_kv *kv) {
  if (!m || !kv) return fail(DBT_ERR_ARG, "model or cache is NULL");
  if (kv->m != m) return fail(DBT_ERR_ARG, "cache belongs to another model");
  return DBT_OK;
}

dbt_status check_step_in(dbt_model *m, dbt_kv *kv, const dbt_step_in *in, int need_branch_input) {
  const dbt_config &cf = m->cfg;
  if (!in) return fail(DBT_ERR_ARG, "step input is NULL");
  if (in->batch <= 0 || in->batch > cf.max_batch) return fail(DBT_ERR_ARG, "batch %d out of [1, %d]", in->batch, cf.max_batch);
  if (cf.has_embeddings) {
    if (!in->tokens) return fail(DBT_ERR_ARG, "tokens are NULL");
  } else {
    if (!in->h1_in || (need_branch_input && !in->h2_in)) return fail(DBT_ERR_ARG, "residual inputs are NULL");
  }
  int need = 0;
  for (int b = 0; b < in->batch; ++b) {
    if (kv->len[b] + 1 > cf.max_pos) return fail(DBT_ERR_SHAPE, "sequence %d would exceed max_pos", b);
    if (kv->needs_page(b)) {
      if (kv->len[b] / kPage >= kv->mpps) return fail(DBT_ERR_NO_PAGES, "sequence %d page table full", b);
      ++need;
    }
  }
  if (need > (int)kv->free_pages.size()) return fail(DBT_ERR_NO_PAGES, "need %d free pages, have %zu", need, kv->free_pages.size());
  return DBT_OK;
}

// Take pages for the new position of each sequence (batch order) and return
// the positions pos_b = len_b.
std::vector<int> begin_step(dbt_kv *kv, int B) {
  std::vector<int> pos(B);
  for (int b = 0; b < B; ++b) {
    pos[b] = kv->len[b];
    if (kv->needs_page(b)) {
      const int p = kv->take_page();
      kv->table[b].push_back(p);
      kv->pending.push_back({b, (int)kv->table[b].size() - 1, p});
    }
  }
  return pos;
}

// Everything of a step is enqueued: the sequences grow.
dbt_status step_done(dbt_kv *kv, int B) {
  kv->pending.clear();
  for (int b = 0; b < B; ++b) kv->len[b] += 1;
  return DBT_OK;
}

dbt_status copy_rows(float *dst, const float *src, int B, int d, hipStream_t st) {
  if (!dst) return DBT_OK;
  HIPCHK(hipMemcpyAsync(dst, src, (size_t)B * d * 4, hipMemcpyDeviceToDevice, st));
  return DBT_OK;
}

// Branch-only pass over all layers (ungrouped pass 2 and the boundary), then
// the output matrix over the branch rows, or over every path's rows where the
// primary's normed final rows wait in Xn (with_primary).
dbt_status branch_pass(dbt_model *m, dbt_kv *kv, int B, int Bp, const Sinks &k, hipStream_t st,
                       const dbt_step_out *out = nullptr, const HIn *hin = nullptr, bool with_primary = false) {
  LayerCall lc{};
  lc.out = out;
  lc.ho = k.ho;
  lc.hin = hin;
  const int nb = n_branches(m->cfg);
  lc.rows = Rows{B, Bp, 1, nb};
  lc.mode = MODE_BRANCH;
  lc.retain = false;
  lc.prefill = false;
  lc.rows_layout = (1 + nb) * Bp;
  lc.last_norm = true;
  for (int l = 0; l < m->cfg.n_layers; ++l) {
    dbt_status s = run_layer(m, kv, l, lc, st);
    if (s) return s;
  }
  if (m->cfg.vocab > 0) return lm_head(m, with_primary ? Rows{B, Bp, 0, 1 + nb} : lc.rows, k, st);
  return DBT_OK;
}

dbt_status decode_step_impl(dbt_model *m, dbt_kv *kv, const dbt_step_in *in, int32_t branch_on, dbt_step_out *out,
                            dbt_stream stream) {
  dbt_status s = check_model_kv(m, kv);
  if (s) return s;
  s = check_step_in(m, kv, in, branch_on);
  if (s) return s;
  hipStream_t st = (hipStream_t)stream;
  const dbt_config &cf = m->cfg;
  const int B = in->batch, Bp = round16(B);
  if ((s = ensure_device(m, st))) return s;  // before any state changes
  m->bnd_kv = nullptr;
  std::vector<int> pos = begin_step(kv, B);
  StepBegin sb;
  if ((s = flush(kv, pos.data(), B, st, &sb))) return s;
  const bool on = branch_on != 0;
  const int nb = n_branches(cf);
  const Rows rows{B, Bp, 0, on ? 1 + nb : 1};
  const bool fold = input_fold(m, B);
  const HIn hin{in->h1_in, in->h2_in, B};
  if (!fold && (s = load_inputs(m, kv, in, in->tokens, rows, st, &sb))) return s;
  LayerCall lc{};
  if (fold) {
    lc.hin = &hin;
    lc.sb = &sb;
  }
  lc.rows = rows;
  lc.mode = on ? MODE_GROUPED : MODE_PRIMARY;
  lc.retain = false;
  lc.prefill = false;
  lc.rows_layout = (1 + nb) * Bp;
  lc.last_norm = true;
  lc.out = out;
  // (the last layer is the first to write an output, after every read of the inputs)
  const Sinks k = make_sinks(m, B, Bp, out, true, on);
  lc.ho = k.ho;
  for (int l = 0; l < cf.n_layers; ++l)
    if ((s = run_layer(m, kv, l, lc, st))) return s;
  if (cf.vocab > 0 && (s = lm_head(m, rows, k, st))) return s;
  if (out) {
    if ((s = readout(m, B, Bp, on, out, k, st))) return s;
    if (k.copy_h1 && (s = copy_rows(out->h1_out, m->at<float>(m->L.S), B, cf.d_model, st))) return s;
    if (on && k.copy_h2 && (s = copy_branch_rows(m, out->h2_out, B, Bp, st))) return s;
  }
  return step_done(kv, B);
}

}  // namespace

// ===========================================================================

extern "C" {

const char *dbt_last_error(void) { return g_err.c_str(); }

size_t dbt_workspace_bytes(const dbt_config *cfg) {
  if (check_config(cfg) != DBT_OK) return 0;
  return make_prompt_layout(cfg, make_layout(cfg)).total;
}

size_t dbt_kv_pages_bytes(const dbt_config *cfg, int32_t num_pages) {
  if (check_config(cfg) != DBT_OK || num_pages <= 0) return 0;
  return (size_t)cfg->n_layers * num_pages * cfg->n_kv_heads * kPage * cfg->head_dim * (cfg->dtype == DBT_BF16 ? 2 : 4);
}

dbt_status dbt_create(const dbt_config *cfg, const dbt_weights *w, void *workspace, dbt_model **out) {
  if (!out) return fail(DBT_ERR_ARG, "out is NULL");
  *out = nullptr;
  if (dbt_status cs = check_config(cfg)) return cs;
  if (!w || !w->h_layers) return fail(DBT_ERR_ARG, "weights are NULL");
  if (!workspace || ((uintptr_t)workspace & 255)) return fail(DBT_ERR_ARG, "workspace NULL or not 256-byte aligned");
  if (cfg->has_embeddings && (!w->emb1 || !w->emb2 || !w->emb_norm)) return fail(DBT_ERR_ARG, "embeddings are NULL");
  if (cfg->vocab > 0 && (!w->lm_head || !w->final_norm)) return fail(DBT_ERR_ARG, "output matrix or final norm is NULL");
  for (int l = 0; l < cfg->n_layers; ++l) {
    const dbt_layer_weights &L = w->h_layers[l];
    if (!L.attn_norm || !L.wq || !L.wk || !L.wv || !L.wo || !L.mlp_norm || !L.a || !L.c)
      return fail(DBT_ERR_ARG, "layer %d has a NULL parameter", l);
    if (cfg->n_experts == 0 && (!L.w_gate || !L.w_up || !L.w_down || !L.b))
      return fail(DBT_ERR_ARG, "layer %d has a NULL MLP parameter", l);
    if (cfg->n_experts > 0 && (!L.router || !L.x_gate || !L.x_up || !L.x_down))
      return fail(DBT_ERR_ARG, "layer %d has a NULL expert parameter", l);
    if (cfg->n_experts > 0 && cfg->d_ff_shared > 0 && (!L.s_gate || !L.s_up || !L.s_down || !L.b))
      return fail(DBT_ERR_ARG, "layer %d has a NULL shared-expert parameter", l);
    if (cfg->compute_matched && (!L.g_attn_copy || !L.g_shared_copy))
      return fail(DBT_ERR_ARG, "layer %d has a NULL gate of the compute-matched variant", l);
  }
  dbt_model *m = new (std::nothrow) dbt_model();
  if (!m) return fail(DBT_ERR_ARG, "out of host memory");
  m->cfg = *cfg;
  m->w = *w;
  m->layers.assign(w->h_layers, w->h_layers + cfg->n_layers);
  m->w.h_layers = nullptr;
  m->ws = (char *)workspace;
  m->L = make_layout(cfg);
  m->Lp = make_prompt_layout(cfg, m->L);
  m->step = m->ws + m->L.state_total;
  // RoPE table (Eq. (8)): angle pos * theta^(-2i/d_h), evaluated in double.
  const int half = cfg->head_dim / 2;
  m->rope_host.resize((size_t)cfg->max_pos * half * 2);
  for (int p = 0; p < cfg->max_pos; ++p)
    for (int i = 0; i < half; ++i) {
      const double ang = (double)p * std::pow((double)cfg->rope_theta, -2.0 * i / cfg->head_dim);
      m->rope_host[((size_t)p * half + i) * 2 + 0] = (float)std::cos(ang);
      m->rope_host[((size_t)p * half + i) * 2 + 1] = (float)std::sin(ang);
    }
  *out = m;
  return DBT_OK;
}

dbt_status dbt_destroy(dbt_model *m) {
  delete m;
  return DBT_OK;
}

dbt_status dbt_kv_create(dbt_model *m, void *k_pages, void *v_pages, int32_t num_pages, int32_t *page_table,
                         int32_t max_pages_per_seq, dbt_kv **out) {
  if (!out) return fail(DBT_ERR_ARG, "out is NULL");
  *out = nullptr;
  if (!m || !k_pages || !v_pages || !page_table) return fail(DBT_ERR_ARG, "NULL argument");
  if (num_pages <= 0 || max_pages_per_seq <= 0) return fail(DBT_ERR_ARG, "num_pages and max_pages_per_seq must be positive");
  if ((long long)max_pages_per_seq * kPage < m->cfg.max_pos) return fail(DBT_ERR_SHAPE, "max_pages_per_seq * 16 < max_pos");
  dbt_kv *kv = new (std::nothrow) dbt_kv();
  if (!kv) return fail(DBT_ERR_ARG, "out of host memory");
  kv->m = m;
  kv->k = (char *)k_pages;
  kv->v = (char *)v_pages;
  kv->num_pages = num_pages;
  kv->page_table = page_table;
  kv->mpps = max_pages_per_seq;
  std::vector<int> all(num_pages);
  for (int i = 0; i < num_pages; ++i) all[i] = i;
  kv->free_pages = std::priority_queue<int, std::vector<int>, std::greater<int>>(std::greater<int>(), std::move(all));
  kv->table.assign(m->cfg.max_batch, {});
  kv->len.assign(m->cfg.max_batch, 0);
  *out = kv;
  return DBT_OK;
}

dbt_status dbt_kv_destroy(dbt_kv *kv) {
  delete kv;
  return DBT_OK;
}

dbt_status dbt_kv_reserve(dbt_kv *kv, int32_t b, int32_t len, int32_t *h_pages_out) {
  if (!kv) return fail(DBT_ERR_ARG, "cache is NULL");
  if (b < 0 || b >= kv->m->cfg.max_batch) return fail(DBT_ERR_ARG, "sequence %d out of range", b);
  if (len < kv->len[b]) return fail(DBT_ERR_ARG, "len %d below current length %d", len, kv->len[b]);
  if (len > kv->m->cfg.max_pos) return fail(DBT_ERR_SHAPE, "len %d exceeds max_pos", len);
  const int need_pages = (len + kPage - 1) / kPage;
  if (need_pages > kv->mpps) return fail(DBT_ERR_NO_PAGES, "page table row too short");
  const int extra = need_pages - (int)kv->table[b].size();
  if (extra > (int)kv->free_pages.size()) return fail(DBT_ERR_NO_PAGES, "need %d free pages, have %zu", extra, kv->free_pages.size());
  for (int i = 0; i < extra; ++i) {
    const int p = kv->take_page();
    kv->table[b].push_back(p);
    kv->pending.push_back({b, (int)kv->table[b].size() - 1, p});
  }
  kv->len[b] = len;
  if (h_pages_out)
    for (size_t i = 0; i < kv->table[b].size(); ++i) h_pages_out[i] = kv->table[b][i];
  if (kv->m->bnd_kv == kv) kv->m->bnd_kv = nullptr;
  return DBT_OK;
}

dbt_status dbt_kv_truncate(dbt_kv *kv, int32_t b, int32_t len) {
  if (!kv) return fail(DBT_ERR_ARG, "cache is NULL");
  if (b < 0 || b >= kv->m->cfg.max_batch) return fail(DBT_ERR_ARG, "sequence %d out of range", b);
  if (len < 0 || len > kv->len[b]) return fail(DBT_ERR_ARG, "len %d outside [0, %d]", len, kv->len[b]);
  const size_t keep = (len + kPage - 1) / kPage;
  for (size_t i = keep; i < kv->table[b].size(); ++i) kv->free_pages.push(kv->table[b][i]);
  kv->table[b].resize(keep);
  kv->len[b] = len;
  // entries of pages given back may still sit in the pending list; they are
  // harmless (a later take re-sends the slot) but drop those of this sequence
  kv->pending.erase(std::remove_if(kv->pending.begin(), kv->pending.end(),
                                   [&](const dbt_kv::Upd &u) { return u.b == b && (size_t)u.slot >= keep; }),
                    kv->pending.end());
  if (kv->m->bnd_kv == kv) kv->m->bnd_kv = nullptr;
  return DBT_OK;
}

int32_t dbt_kv_length(const dbt_kv *kv, int32_t b) {
  if (!kv || b < 0 || b >= kv->m->cfg.max_batch) return -1;
  return kv->len[b];
}

int32_t dbt_kv_pages(const dbt_kv *kv, int32_t b, int32_t *h_out, int32_t cap) {
  if (!kv || b < 0 || b >= kv->m->cfg.max_batch) return -1;
  const int n = (int)kv->table[b].size();
  for (int i = 0; i < n && i < cap && h_out; ++i) h_out[i] = kv->table[b][i];
  return n;
}

dbt_status dbt_kv_fill(dbt_kv *kv, int32_t layer, int32_t b, int32_t start, int32_t count, const void *k_src,
                       const void *v_src, dbt_stream stream) {
  if (!kv || !k_src || !v_src) return fail(DBT_ERR_ARG, "NULL argument");
  const dbt_config &cf = kv->m->cfg;
  if (layer < 0 || layer >= cf.n_layers) return fail(DBT_ERR_ARG, "layer %d out of range", layer);
  if (b < 0 || b >= cf.max_batch) return fail(DBT_ERR_ARG, "sequence %d out of range", b);
  if (start < 0 || count < 0 || start + count > kv->len[b]) return fail(DBT_ERR_ARG, "positions outside the reserved length");
  hipStream_t st = (hipStream_t)stream;
  dbt_status s = ensure_device(kv->m, st);
  if (s) return s;
  s = flush(kv, nullptr, 0, st);
  if (s) return s;
  HIPCHK(launch_kv_fill(kv_layer(kv, layer), b, start, count, k_src, v_src, cf.dtype, st));
  return DBT_OK;
}

dbt_status dbt_decode_step(dbt_model *m, dbt_kv *kv, const dbt_step_in *in, int32_t branch_on, dbt_step_out *out,
                           dbt_stream stream) {
  return decode_step_impl(m, kv, in, branch_on, out, stream);
}

dbt_status dbt_decode_step_ungrouped(dbt_model *m, dbt_kv *kv, const dbt_step_in *in, dbt_step_out *out,
                                     dbt_stream stream) {
  dbt_status s = check_model_kv(m, kv);
  if (s) return s;
  s = check_step_in(m, kv, in, 1);
  if (s) return s;
  hipStream_t st = (hipStream_t)stream;
  const dbt_config &cf = m->cfg;
  const int B = in->batch, Bp = round16(B);
  if ((s = ensure_device(m, st))) return s;  // before any state changes
  m->bnd_kv = nullptr;
  std::vector<int> pos = begin_step(kv, B);
  StepBegin sb;
  if ((s = flush(kv, pos.data(), B, st, &sb))) return s;
  // pass 1: every primary layer, keeping Q1, H1, M1
  const Rows prim{B, Bp, 0, 1};
  const bool fold = input_fold(m, B);
  const HIn hin{in->h1_in, in->h2_in, B};
  if (!fold && (s = load_inputs(m, kv, in, in->tokens, prim, st, &sb))) return s;
  LayerCall lc{};
  if (fold) {
    lc.hin = &hin;
    lc.sb = &sb;
  }
  lc.rows = prim;
  lc.mode = MODE_PRIMARY;
  lc.retain = true;
  lc.prefill = false;
  lc.rows_layout = (1 + n_branches(cf)) * Bp;
  lc.last_norm = true;
  lc.out = out;
  // (the second pass reads inputs: the primary's outputs are copied at the end)
  const Sinks k = make_sinks(m, B, Bp, out, false, true);
  for (int l = 0; l < cf.n_layers; ++l)
    if ((s = run_layer(m, kv, l, lc, st))) return s;
  if (cf.vocab > 0 && (s = lm_head(m, prim, k, st))) return s;
  // pass 2: every branch layer
  const Rows br{B, Bp, 1, n_branches(cf)};
  if (!fold && (s = load_inputs(m, kv, in, in->tokens, br, st))) return s;
  if ((s = branch_pass(m, kv, B, Bp, k, st, out, fold ? &hin : nullptr))) return s;
  if (out) {
    if ((s = readout(m, B, Bp, true, out, k, st))) return s;
    if (k.copy_h1 && (s = copy_rows(out->h1_out, m->at<float>(m->L.S), B, cf.d_model, st))) return s;
    if (k.copy_h2 && (s = copy_branch_rows(m, out->h2_out, B, Bp, st))) return s;
  }
  return step_done(kv, B);
}

// The boundary after a prefill whose primary logits are at k, or, as part of
// the prefill call (with_primary), still to be computed: the output matrix is
// then read once for every path.
static dbt_status boundary_impl(dbt_model *m, dbt_kv *kv, int B, dbt_step_out *out, const Sinks &k, bool with_primary,
                                hipStream_t st) {
  dbt_status s;
  const dbt_config &cf = m->cfg;
  const Layout &L = m->L;
  const int Bp = round16(B);
  std::vector<int> pos(B);
  for (int b = 0; b < B; ++b) pos[b] = kv->len[b] - 1;
  if ((s = flush(kv, pos.data(), B, st))) return s;
  const Rows br{B, Bp, 1, n_branches(cf)};
  HIPCHK(launch_embed(m->at<int>(L.btok), cf.vocab, m->w.emb1, m->w.emb2, m->w.emb_norm, m->layers[0].attn_norm, cf.rms_eps,
                      cf.d_model, cf.dtype, br, m->at<float>(L.S), m->p(L.Xn), cf.d_model, st));
  if ((s = branch_pass(m, kv, B, Bp, k, st, nullptr, nullptr, with_primary))) return s;
  m->bnd_kv = nullptr;
  if (out) {
    if ((s = readout(m, B, Bp, true, out, k, st))) return s;
    if (k.copy_h2 && (s = copy_branch_rows(m, out->h2_out, B, Bp, st))) return s;
  }
  return DBT_OK;
}

dbt_status dbt_prefill(dbt_model *m, dbt_kv *kv, const int32_t *tokens, const int32_t *h_prompt_lens, int32_t batch,
                       int32_t run_boundary, dbt_step_out *out, dbt_stream stream) {
  dbt_status s = check_model_kv(m, kv);
  if (s) return s;
  const dbt_config &cf = m->cfg;
  if (!tokens || !h_prompt_lens) return fail(DBT_ERR_ARG, "tokens or prompt lengths NULL");
  if (cf.max_prompt <= 0) return fail(DBT_ERR_STATE, "model created without prefill support (max_prompt = 0)");
  if (batch <= 0 || batch > cf.max_batch) return fail(DBT_ERR_ARG, "batch %d out of [1, %d]", batch, cf.max_batch);
  int need = 0;
  for (int b = 0; b < batch; ++b) {
    const int T = h_prompt_lens[b];
    if (T <= 0 || T > cf.max_prompt) return fail(DBT_ERR_SHAPE, "prompt %d length %d outside [1, %d]", b, T, cf.max_prompt);
    if (kv->len[b] != 0) return fail(DBT_ERR_STATE, "sequence %d is not empty", b);
    need += (T + kPage - 1) / kPage;
  }
  if (need > (int)kv->free_pages.size()) return fail(DBT_ERR_NO_PAGES, "need %d free pages, have %zu", need, kv->free_pages.size());
  hipStream_t st = (hipStream_t)stream;
  if ((s = ensure_device(m, st))) return s;  // before any state changes
  m->bnd_kv = nullptr;  // (a boundary needs a prefill that went through)
  for (int b = 0; b < batch; ++b) {  // pages for every sequence first, in batch order
    const int np = (h_prompt_lens[b] + kPage - 1) / kPage;
    for (int i = 0; i < np; ++i) {
      const int p = kv->take_page();
      kv->table[b].push_back(p);
      kv->pending.push_back({b, i, p});
    }
    kv->len[b] = h_prompt_lens[b];
  }
  if ((s = flush(kv, nullptr, 0, st))) return s;
  const Layout &L = m->L;
  const int d = cf.d_model;
  const int Bp = round16(batch);
  size_t off = 0, left = 0;
  for (int b = 0; b < batch; ++b) left += h_prompt_lens[b];
  const Sinks k = make_sinks(m, batch, Bp, out, run_boundary != 0, true, Span{tokens, left * sizeof(int)});
  // Packed passes over consecutive prompts: as few as the rows of the prompt
  // buffers allow, of about equal size.  A prompt's own length chooses its
  // attention kernel, so prompts of different kernels take passes of their own.
  const Layout &Lp = m->Lp;
  auto shares = [&](int len) { return prompt_shares_pages(cf.n_q_heads, cf.n_kv_heads, len, cf.dtype); };
  for (int b = 0; b < batch;) {
    const size_t passes = (left + Lp.pack_rows - 1) / Lp.pack_rows, share = (left + passes - 1) / passes;
    Pack pk;
    pk.n = 0;
    pk.seq0 = b;
    pk.off[0] = 0;
    LayerCall lc{};
    int T = 0;
    while (b < batch && pk.n < kPackSeqs &&
           (pk.n == 0 || ((size_t)T < share && T + h_prompt_lens[b] <= Lp.pack_rows && shares(h_prompt_lens[b]) == lc.tiles.shared))) {
      lc.tiles.shared = shares(h_prompt_lens[b]);
      T += h_prompt_lens[b];
      pk.off[++pk.n] = T;
      ++b;
    }
    left -= T;
    const Rows rows{T, T, 0, 1};
    lc.tiles.tp = prompt_tile_positions(cf.n_q_heads, cf.n_kv_heads, lc.tiles.shared);
    lc.tiles.tiles = m->at<PromptTile>(Lp.ptiles);
    HIPCHK(launch_prompt_plan(pk, lc.tiles.tp, m->at<PromptRow>(Lp.prow), m->at<PromptTile>(Lp.ptiles), &lc.tiles.ntiles, st));
    HIPCHK(launch_embed(tokens + off, cf.vocab, m->w.emb1, m->w.emb2, m->w.emb_norm, m->layers[0].attn_norm, cf.rms_eps, d,
                        cf.dtype, rows, m->at<float>(Lp.S), m->p(Lp.Xn), d, st));
    lc.rows = rows;
    lc.mode = MODE_PRIMARY;
    lc.retain = true;
    lc.prefill = true;
    lc.rows_layout = T;
    lc.last_norm = false;
    for (int l = 0; l < cf.n_layers; ++l)
      if ((s = run_layer(m, kv, l, lc, st))) return s;
    HIPCHK(launch_prompt_last(pk, m->at<float>(Lp.S), tokens + off, d, m->at<float>(L.slast), k.ho.h1,
                              m->at<int>(L.btok), st));
    off += T;
  }
  // primary logits at each prompt's final position (kept in the workspace
  // for a boundary call of its own)
  if (cf.vocab > 0) {
    HIPCHK(launch_rmsnorm_rows(m->at<float>(L.slast), m->w.final_norm, cf.rms_eps, d, cf.dtype, Rows{batch, 0, 0, 1},
                               m->p(L.Xn), d, st));
    if (!run_boundary && (s = lm_head(m, Rows{batch, Bp, 0, 1}, k, st))) return s;
  }
  if (k.copy_h1 && (s = copy_rows(out->h1_out, m->at<float>(L.slast), batch, d, st))) return s;
  if (run_boundary) return boundary_impl(m, kv, batch, out, k, true, st);
  if (out && (s = readout(m, batch, Bp, false, out, k, st))) return s;
  m->bnd_kv = kv;
  m->bnd_batch = batch;
  return DBT_OK;
}

dbt_status dbt_boundary(dbt_model *m, dbt_kv *kv, int32_t batch, dbt_step_out *out, dbt_stream stream) {
  dbt_status s = check_model_kv(m, kv);
  if (s) return s;
  if (m->bnd_kv != kv || batch != m->bnd_batch)
    return fail(DBT_ERR_STATE, "boundary must directly follow dbt_prefill on the same cache and batch");
  hipStream_t st = (hipStream_t)stream;
  if ((s = ensure_device(m, st))) return s;
  return boundary_impl(m, kv, batch, out, make_sinks(m, batch, round16(batch), out, false, true), false, st);
}

dbt_status dbt_stage_timing(dbt_model *m, int32_t stage, int32_t enable) {
  if (!m) return fail(DBT_ERR_ARG, "model is NULL");
  if (stage < 0 || stage >= DBT_STAGE_COUNT) return fail(DBT_ERR_ARG, "stage %d out of range", stage);
  m->timers[stage].on = enable != 0;
  m->timers[stage].used = 0;
  return DBT_OK;
}

double dbt_stage_time(dbt_model *m, int32_t stage, int32_t *h_launches) {
  if (!m || stage < 0 || stage >= DBT_STAGE_COUNT) return -1.0;
  StageTimer &t = m->timers[stage];
  double total = 0.0;
  for (size_t i = 0; i < t.used; ++i) {
    float ms = 0.f;
    if (hipEventSynchronize(t.ev[i].second) != hipSuccess) return -1.0;
    if (hipEventElapsedTime(&ms, t.ev[i].first, t.ev[i].second) != hipSuccess) return -1.0;
    total += ms;
  }
  if (h_launches) *h_launches = (int32_t)t.used;
  t.used = 0;
  return total;
}

}  // extern "C"

// ---------------------------------------------------------------------------
// Hooks for the allocation-free step (static_scratch.hip)
// ---------------------------------------------------------------------------
namespace dbt {

dbt_status set_error(dbt_status s, const char *msg) { return fail(s, "%s", msg); }

size_t step_bytes(const dbt_model *m) { return m->L.step_total - m->L.state_total; }

dbt_status decode_step_in(dbt_model *m, dbt_kv *kv, const dbt_step_in *in, int32_t branch_on, dbt_step_out *out,
                          dbt_stream stream, char *step_mem) {
  // the model's own step region again when the call returns, whatever it returns
  struct Restore {
    dbt_model *m;
    ~Restore() {
      m->step = m->ws + m->L.state_total;
      m->no_fork = false;
    }
  } restore{m};
  m->step = step_mem;
  m->no_fork = true;  // no stream of its own is created here: the shared expert stays on `stream`
  return decode_step_impl(m, kv, in, branch_on, out, stream);
}

}  // namespace dbt
