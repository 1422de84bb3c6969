// Launchers of the device kernels (internal to the library; the public
// interface is include/dbt.h).  Every launcher enqueues on `st` and returns
// hipGetLastError() of its launches.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dbt {

// Up to three stacked weight matrices that one projection reads as one
// [sum rows][K] operand (e.g. W_Q; W_K; W_V).  Unused entries have rows 0.
struct WSegs {
  const void *w[3];
  int rows[3];
};

// Which activation rows a kernel processes.  Activations of a call are laid
// out [2][Bp][width]: path p (0 primary, 1 branch) sequence b sits at
// physical row p*Bp + b, Bp = batch rounded up to 16.
struct Rows {
  int B;   // sequences
  int Bp;  // row stride between the two paths
  int p0;  // first active path
  int np;  // active paths (1 or 2)
};

// Compute units the launch rules fill.  A constant of the part (MI355X, not
// partitioned) rather than a query: the workspace is sized from the same rules
// by calls that need no GPU.
constexpr int kComputeUnits = 256;

enum Mode { MODE_GROUPED = 0, MODE_PRIMARY = 1, MODE_BRANCH = 2 };

// Prompts of several sequences are packed into one pass: row r of the pass is
// position pos of sequence seq; keep is the sequence at its prompt's last
// row (whose primary intermediates are kept for the boundary) and -1 elsewhere.
struct PromptRow {
  int pos, seq, keep, unused;
};
// One attention tile of a packed pass: query positions q0 .. of a prompt of T
// positions of sequence seq, whose position 0 is row row0 of the pass.
struct PromptTile {
  int row0, q0, T, seq;
};
// Sequences seq0 .. seq0 + n - 1 of a pass: rows off[i] .. off[i + 1] - 1.
constexpr int kPackSeqs = 128;
struct Pack {
  int n, seq0;
  int off[kPackSeqs + 1];
};
// Fills the row map of the pass and its attention tiles of tp positions,
// longest first; returns their number through *ntiles.
hipError_t launch_prompt_plan(const Pack &pk, int tp, PromptRow *rows, PromptTile *tiles, int *ntiles, hipStream_t st);
// After the last layer: each prompt's final residual row to slast[seq] (and
// hout[seq] unless NULL), its final token to btok[seq].
hipError_t launch_prompt_last(const Pack &pk, const float *S, const int *tokens, int d, float *slast, float *hout,
                              int *btok, hipStream_t st);

// Retention of primary intermediates for a later branch evaluation: row b of
// the call is kept at retained row b, or, in a pass over prompts, at
// map[b].keep when that is not negative.
struct Retain {
  float *ptr;  // NULL: nothing kept
  const PromptRow *map;
#ifdef __HIPCC__
  // the retained row of row b, -1 when it is not kept
  __device__ __forceinline__ int row(int b) const { return !ptr ? -1 : map ? map[b].keep : b; }
#endif
};

struct KVRef {
  void *k, *v;            // pages of this layer: k/v base + layer offset already applied
  const int *page_table;  // [max_batch][mpps]
  int mpps;               // entries per sequence
  int n_kv, d_h;
};

// ---- projections ----
struct GemmConfig {
  int RB;      // 16-row blocks per wave (a workgroup owns NW*16*RB weight rows)
  int PD;      // weight prefetch depth in 128-element chunks
  int S;       // reduction splits (one fp32 output slab per split)
  int NW = 4;  // waves per workgroup (4 or 8)
};
GemmConfig gemm_config(int n_full, int K, int dtype, int seg_gran, int max_rows);

// Gate/up projection with the SwiGLU + b-coupling epilogue fused (Eqs. (13)-(14)):
// writes the MLP intermediate H (bf16, rows p*Bp + b, leading dimension ldh)
// instead of fp32 gate/up outputs.  Branch rows take H1 from the primary rows of
// the same call (mode GROUPED) or from H1_in (mode BRANCH); primary rows are
// kept in ret when asked.  Usable when gemm_glu_ok() holds.
struct GluEpi {
  Rows rows;
  int mode;
  int f;
  const float *bvec;   // [f]
  const float *H1_in;  // [B][f] (mode BRANCH)
  Retain ret;
  uint16_t *Xh;
  int ldh;
};
bool gemm_glu_ok(int f, int M, int np, int dtype);
hipError_t launch_gemm_glu(const uint16_t *w_gate, const uint16_t *w_up, int f, int K, const void *X, int ldx, int M,
                           const GluEpi &ep, hipStream_t st);
// Where the rows of an unsplit projection go: row m of the call is row m % Bp
// of p[m / Bp] (Bp a multiple of 16), rows past B are not stored.  The output
// matrix writes its logits straight to the caller's arrays this way, one per
// path, instead of to padded rows that are copied afterwards.  Bp = 0: not used.
struct YRows {
  float *p[4];
  int Bp, B;
#ifdef __HIPCC__
  __device__ __forceinline__ float *row(int m, int ld, bool &live) const {
    float *q = p[0];
    if (m >= Bp) {
      q = p[1];
      m -= Bp;
      if (m >= Bp) {
        q = p[2];
        m -= Bp;
        if (m >= Bp) {
          q = p[3];
          m -= Bp;
        }
      }
    }
    live = m < B;
    return q + (size_t)m * ld;
  }
#endif
};
hipError_t launch_gemm(const WSegs &segs, int N, int K, int dtype, const void *X, int ldx, int M,
                       float *Y, int ldy, long long y_split_stride, const GemmConfig &g, hipStream_t st,
                       float *row_stats = nullptr, const YRows *yrows = nullptr);
// Tiles per row of the statistics the output projection writes when given
// row_stats (0: this shape does not produce them).
int gemm_stats_tiles(int N, const GemmConfig &g, int dtype);
int gemm_tile_rows(const GemmConfig &g);  // weight rows (output columns) per workgroup

// Projection of a pass over prompts (M >= 256 rows, K a multiple of 128, N a
// multiple of 16, bf16): tiles of 128 or 256 rows and columns on the matrix
// cores.  Plain: Y (fp32,
// [M][ldy]) = X W^T with W the stacked segments w[0..2] (rows[0..2] rows).
// GLU: w[0] = gate, w[1] = up (N = f rows each); writes H (bf16, [M][ldh]) =
// silu(X Wg^T) * (X Wu^T), and keeps rows of H in fp32 (ret).  QKV (rope !=
// NULL; bf16 cache, d_h 128, rows = prompt positions by the map `prompt`, w =
// W_Q, W_K, W_V): the rotary embedding on Q and K, Q (fp32, [M][rows[0]]) to
// Qout and its kept rows to ret, K and V into the cache slots of their
// positions; no Y.
struct TileGemm {
  const uint16_t *w[3];
  int rows[3];
  int N, K;
  const uint16_t *X;
  int ldx, M;
  float *Y;
  int ldy;
  int splits;          // plain: reduction splits, slab s at Y + s*y_stride (0 reads as 1)
  long long y_stride;
  uint16_t *H;
  int ldh;
  Retain ret;
  const float2 *rope;  // [max_pos][64] (cos, sin)
  float *Qout;
  KVRef kv;
  const PromptRow *prompt;
  // expert products (moe): X rows grouped by expert through arow (gate/up; NULL:
  // in expert order already), the experts' matrices behind each other in
  // w[0], w[1], outputs in expert order; M bounds the rows of all experts
  const int2 *tiles;
  const int *ntiles, *counts, *offsets, *arow;
  int max_tiles;
};
bool gemm_tile_ok(int N, int K, int M, int dtype);
// Prompt rows from which launch_gemm_tile is used.
constexpr int kTileRows = 256;
// Reduction splits launch_gemm_tile should run a plain projection with; the
// slabs of more than one have at most kTileSlabs elements together.
int gemm_tile_splits(int N, int K, int M);
constexpr int kTileSlabs = 256 * 256 * 256;
// Everything launch_gemm_tile requires of g (the shape test above, segment
// sizes multiples of 8 summing to N, row strides multiples of 8, element
// byte offsets within 32 bits); callers fall back to launch_gemm otherwise.
bool gemm_tile_args_ok(const TileGemm &g, bool glu);
hipError_t launch_gemm_tile(const TileGemm &g, bool glu, hipStream_t st);
// The expert products of a pass (see TileGemm::tiles).
bool gemm_tile_experts_ok(const TileGemm &g);
hipError_t launch_gemm_tile_experts(const TileGemm &g, bool glu, hipStream_t st);

// ---- row-wise and elementwise stages ----
struct StepBegin {
  int n_pos, b0;
  int pos[64];
  int n_pt;
  int pt_b[64], pt_slot[64], pt_page[64];
};
// Runs of consecutive page-table entries: slots slot .. slot + count - 1 of
// sequence b hold pages page, page + 1, ...
constexpr int kPageRuns = 128;
struct PageRuns {
  int n;
  int b[kPageRuns], slot[kPageRuns], page[kPageRuns], count[kPageRuns];
};
hipError_t launch_page_runs(const PageRuns &pr, int *page_table, int mpps, hipStream_t st);
hipError_t launch_step_begin(const StepBegin &sb, int *pos_arr, int *page_table, int mpps,
                             hipStream_t st);

// The step's first kernel also applies `sb` (positions and new page-table
// entries) when sb is not NULL.
hipError_t launch_embed(const int *tokens, int vocab, const void *e1, const void *e2, const float *g_emb,
                        const float *g_next, float eps, int d, int dtype, Rows rows, float *S,
                        void *Xn, int ldx, hipStream_t st, const StepBegin *sb = nullptr,
                        int *pos_arr = nullptr, int *page_table = nullptr, int mpps = 0);
hipError_t launch_load_hidden(const float *h1, const float *h2, const float *g_next, float eps,
                              int d, int dtype, Rows rows, float *S, void *Xn, int ldx,
                              hipStream_t st, const StepBegin *sb = nullptr, int *pos_arr = nullptr,
                              int *page_table = nullptr, int mpps = 0);
hipError_t launch_rmsnorm_rows(const float *S, const float *g, float eps, int d, int dtype,
                               Rows rows, void *Xn, int ldx, hipStream_t st);

// The first layer of a layer-only model read straight from the step's
// residual inputs, with no norm kernel before it: RMSNorm(h) W^T =
// (1/rms(h)) (h * g) W^T, so the QKV projection stages bf16(h * g) and
// writes, per reduction split, each row's sum of squares of h over the
// split's columns; the QKV finish scales each summed output by
// 1/sqrt(sum / d + eps) and the residual step reads h as the residual.
struct HIn {
  const float *h1;  // [B][d] primary rows (NULL: not in use)
  const float *h2;  // [n_b][B][d] branch rows
  int B;
};
struct XNorm {
  HIn h;
  Rows rows;     // the call's rows: row m is path p0 + m / Bp, sequence m % Bp
  const float *g;  // [d] attention-norm gain
  float *ss;     // [S][ss_ld] per split: ss[s * ss_ld + p*Bp + b]
  int ss_ld;
  StepBegin sb;  // applied by the first workgroup (positions, page-table entries)
  int *pos_arr, *page_table, mpps;
};
// Whether launch_gemm_xnorm runs this configuration.
bool gemm_xnorm_ok(const GemmConfig &g, int M);
hipError_t launch_gemm_xnorm(const WSegs &segs, int N, int K, const XNorm &xn, int M, float *Y, int ldy,
                             long long y_split_stride, const GemmConfig &g, hipStream_t st);

struct QKVFinish {
  const float *part;
  long long split_stride;
  int S, ldp;
  int n_q, n_kv, d_h;
  Rows rows;
  int mode;
  const float2 *rope;  // [max_pos][d_h/2] (cos, sin)
  const int *pos_arr;  // decode: position of sequence b (NULL: prefill)
  const PromptRow *prompt;  // prefill: position and sequence of row b
  const float *a;
  float *Q;            // [2Bp][n_q*d_h]
  const float *Q1_in;  // branch mode: retained primary queries [*, n_q*d_h]
  Retain ret;
  KVRef kv;
  int dtype;
  // rows from XNorm: each summed output of physical row R is scaled by
  // 1/sqrt(sum_{s < ss_S} ss[s * ss_ld + R] / d_model + eps) (ss NULL: 1)
  const float *ss;
  int ss_ld, ss_S, d_model;
  float eps;
};
hipError_t launch_qkv_finish(const QKVFinish &f, hipStream_t st);

// Compute-matched variant (App. B.3): a branch row takes g * (the primary
// row's value) instead of its own.  g == NULL: the standard model.
struct GatedCopy {
  const float *g;   // [d]
  const float *in;  // [B][d] primary values (branch-only calls)
  Retain ret;       // keep the primary values for a later branch-only call
};
// hin.h1 not NULL: the residual of row (path, b) is the step input h (see
// XNorm) instead of Sres; the sum is written to Sres either way.
hipError_t launch_resid_norm(const float *part, long long split_stride, int S, int ldp, float *Sres,
                             const float *g, float eps, int d, int dtype, Rows rows, void *Xn, int ldx,
                             hipStream_t st, const GatedCopy &gc = GatedCopy{}, const HIn &hin = HIn{});

hipError_t launch_swiglu_finish(const float *part, long long split_stride, int S, int ldp, int f,
                                int mode, Rows rows, const float *bvec, const float *H1_in,
                                Retain ret, int dtype, void *Xh, int ldh, hipStream_t st);

// The last layer's states go straight to the caller's arrays (an entry that is
// NULL: to Sres as in every other layer).
struct HOut {
  float *h1;  // [B][d]
  float *h2;  // [n_b][B][d]
  int B;
#ifdef __HIPCC__
  // row (path, b), or `s` where the path's array is not given
  __device__ __forceinline__ float4 *row(int path, int b, int d, float4 *s) const {
    if (path == 0) return h1 ? (float4 *)(h1 + (size_t)b * d) : s;
    return h2 ? (float4 *)(h2 + ((size_t)(path - 1) * B + b) * d) : s;
  }
#endif
};
hipError_t launch_down_finish(const float *part, long long split_stride, int S, int ldp, int d,
                              int mode, Rows rows, const float *cvec, const float *M1_in,
                              Retain ret, float *Sres, const float *g_next, float eps, int dtype,
                              void *Xn, int ldx, hipStream_t st, const HOut &ho = HOut{});

// ---- attention ----
struct AttnArgs {
  const float *Q;  // fp32: [2Bp][n_q*d_h]
  KVRef kv;
  const int *pos_arr;  // length of sequence b = pos_arr[b] + 1
  Rows rows;
  int n_q;
  int pages_per_split;  // target: a sequence of P pages is read in ceil(P / target) equal splits
  int max_splits;
  float *opart;  // [B][n_kv][max_splits][16][d_h]
  float *ostat;  // [B][n_kv][max_splits][16][2]
  int dtype;
  // one workgroup of eight waves per (sequence, KV head) writes the
  // normalised rows to O (row stride ldo; bf16: every sequence at most 1024
  // pages; fp32: at most one split); no partials and no combine launch
  int single;
  void *O;
  int ldo;
  // bf16: the queries and the cache append are computed by the attention
  // kernel itself from the QKV projection's split-K slabs, exactly as
  // k_qkv_finish would (one launch fewer); Q is then not read
  QKVFinish fin;
};
hipError_t launch_attn_decode(const AttnArgs &a, hipStream_t st);
hipError_t launch_attn_combine(const AttnArgs &a, void *O, int ldo, hipStream_t st);

// Causal attention of the prompts of a packed pass (rows by tiles[0..ntiles)).
struct PromptAttn {
  const float *Q;
  int ldq;
  KVRef kv;
  int n_q;
  int dtype;
  void *O;
  int ldo;
  const PromptTile *tiles;
  int ntiles;
  bool shared;      // prompt_shares_pages of every prompt of the pass
  int tp;           // positions per tile: prompt_tile_positions
};
// Whether a prompt of len positions (n_q / n_kv query heads per KV head) runs
// the kernel whose sixteen waves share each page through LDS.
bool prompt_shares_pages(int n_q, int n_kv, int len, int dtype);
// Query positions per workgroup of the prompt kernels.
int prompt_tile_positions(int n_q, int n_kv, bool shared);
hipError_t launch_attn_prefill(const PromptAttn &a, hipStream_t st);

// ---- cache fill ----
hipError_t launch_kv_fill(KVRef kv, int seq, int start, int count, const void *ksrc,
                          const void *vsrc, int dtype, hipStream_t st);

// ---- mixture readout (Sec. 4.2) ----
struct MixArgs {
  const float *z[4];    // logits of path j: row b at z[j] + b*V
  int V;
  Rows rows;            // np = 1 + n_b with the branches on (n_b <= 3), 1 (primary) otherwise
  int chunk;            // vocabulary entries per statistics chunk when the projection wrote none
  float *stats;         // [(1 + n_b) Bp][nstat][3] per tile (max, sum e^(z-max), sum e^(2(z-max)))
  int nstat;            // tiles per row in stats
  int tile_w;           // vocabulary entries per tile (the projection's rows per workgroup, or chunk)
  int stats_ready;      // 1: the output projection already wrote stats
  float *alpha;         // [B] or NULL
  int *next;            // [B] or NULL
};
hipError_t launch_mixture(const MixArgs &m, hipStream_t st);

// ---- MoE (Sec. 3.2, Sec. 4.3, Sec. 5) ----
// Per-row selections live in [2Bp][8] arrays (row = path*Bp + b, k <= 8).
constexpr int kRouteOne = 128;  // experts one workgroup of the router takes
struct MoeRoute {
  const float *Sbar;  // [2Bp][d] residual after attention (fp32)
  const float *g;     // MLP norm gain
  float eps;
  int d;
  const void *Wr;     // [E][d] bf16 router
  int E, k1, k2, replay;
  Rows rows;
  int mode;
  float *logits;      // [2Bp][256] router logits, for more than kRouteOne experts
  int *idx;           // [2Bp][8] selected experts (logit descending)
  float *wts;         // [2Bp][8] renormalised weights
  const int *idx1_in; // branch mode + replay: retained primary selections [*, 8]
  int *out_idx1, *out_idx2;
  float *out_w1, *out_w2;  // caller outputs [B][k] of this layer (may be NULL)
  float *out_lg1, *out_lg2;  // caller router logits [B][E] of this layer (may be NULL)
  int *ret_idx;       // retained primary selections (may be NULL), kept as Retain keeps rows
  const PromptRow *ret_map;
};
struct MoeDispatch {
  const int *idx;
  Rows rows;
  int k1, k2, E;
  int *counts;   // [E]
  int *offsets;  // [E+1]
  int *arow;     // [A] activation row of each expert-grouped assignment
  int *aslot;    // [2Bp][8] position of each (row, slot) in the expert-grouped order
  int2 *tiles;   // row tiles of kTileExpert rows: (expert, first row); NULL: not wanted
  int *ntiles;
};
constexpr int kTileExpert = 128;
struct MoeGemm {
  const void *X;  // gate/up: normalized MLP inputs (gathered by arow); down: expert intermediates
  int ldx;
  const void *W0, *W1;  // gate/up: x_gate, x_up; down: x_down
  int E, N, K;
  const int *counts, *offsets, *arow;
  void *Y;  // gate/up: [A][N] bf16 intermediates; down: [A][N] fp32 outputs
  int ldy;
};
struct MoeCombine {
  Rows rows;
  int mode, d, k1, k2;
  const int *idx;
  const float *wts;
  const int *aslot;
  const float *Yexp;  // [A][d]
  const float *part;  // shared-expert down projection slabs (S_sh of them)
  long long stride;
  int S_sh;
  const float *c;
  const float *M1_in;  // compute-matched: G1 (primary shared-expert output) instead
  Retain ret;          // compute-matched: keeps G1
  const float *gG;     // compute-matched variant (App. B.3): branch M2 = R2 + gG * G1; NULL otherwise
  float *S;
  HOut ho;
  const float *g_next;
  float eps;
  void *Xn;
  int ldx;
};
hipError_t launch_moe_route(const MoeRoute &a, hipStream_t st);
hipError_t launch_moe_dispatch(const MoeDispatch &a, hipStream_t st);
hipError_t launch_moe_gemm(const MoeGemm &a, bool gateup, int max_rows, hipStream_t st);
hipError_t launch_moe_combine(const MoeCombine &a, int dtype, hipStream_t st);

}  // namespace dbt
