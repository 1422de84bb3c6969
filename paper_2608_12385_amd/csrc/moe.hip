// MoE layer of the decode step (Sec. 3.2, Eqs. (5)-(6); router replay,
// Sec. 4.3 Eq. (19); independent primary/branch fan-outs k1, k2, Sec. 5
// Eq. (22)).
//
// 1. k_moe_route (above 128 experts followed by k_moe_select): the router
//    logits of each sequence's primary and branch rows from the fp32 MLP input
//    (RMSNorm of S_bar), top-k (logit descending, ties to the lower index) and
//    the renormalised softmax weights of the selected experts.
// 2. k_moe_dispatch: per expert, the list of (path, sequence, slot)
//    assignments in (path, sequence, slot) order; each assignment's
//    position in the expert-grouped order.
// 3. k_moe_gemm<GATEUP>: for each touched expert, its gate/up rows against
//    the gathered activation rows of all its assignments from both paths
//    (each expert weight tile is read once for the primary and branch rows
//    that selected it), SwiGLU in the epilogue.
// 4. k_moe_gemm<DOWN>: the expert down projections of the same rows.
//    (Prompt passes with enough rows per expert run 3 and 4 as tiles of the
//    prompt projections, prefill_gemm.hip.)
// 5. k_moe_combine: M_i = sum over selected experts (ascending id) of
//    w_e * Expert_e(U_i) + shared expert; M2 += c * M1; S += M; next norm.
//    Compute-matched variant (App. B.3): the shared expert runs on the
//    primary rows only and M2 = R2 + g_G * G1.
// Experts no row selected are never read.
#include "common.h"
#include "kernels.h"

namespace dbt {

namespace {

__device__ __forceinline__ int prow(const Rows &r, int path, int b) { return path * r.Bp + b; }

// Router: logits, top-k and weights of 16 rows per workgroup
// (eight sequences with both paths, so that a replayed branch finds its
// primary's experts, or sixteen of one path).  Bound by latency, not bytes:
// one kernel for the logits and the selection instead of two (64 sequences,
// two paths, 64 experts of width 2048: 12.9 + 11.4 us, now 20.0).
//
// Logits r = RMSNorm(S_bar) g W_r^T on the bf16 matrix instruction at fp32
// accuracy: the fp32 input v = S_bar * g is split exactly into three bf16
// parts (8 significant bits each; what is left is below 2^-27 of v), the
// router matrix is bf16, so every product is exact and the sums are fp32; the
// row's 1/rms multiplies the finished sum.  The waves take the 32-element pieces
// of the reduction in turn (lane (r, gq): elements 8 gq .. 8 gq + 7 of
// row / expert r), the waves are added in order through LDS.
// Waves per workgroup: sixteen where their partial logits fit LDS.  The kernel
// runs its code once, from a cold instruction cache, so loops stay rolled and
// more waves rather than unrolled pieces shorten the chain of loads (eight
// waves with four pieces each in flight: 20 us).
// Above 128 experts a workgroup would read a router of 0.5 to 1 MB by itself:
// blockIdx.y is then a group of 64 experts, the logits go to memory and
// k_moe_select follows (LOGITS).  Whole step with 256 experts and width 2048, one
// kernel against two: one sequence 115.2 and 94.4 us, eight 141.3 and 121.1,
// 64 sequences 229.4 and 206.2; at 128 experts one kernel (two before: 106.9
// against 95.9 us for one sequence).
constexpr int route_waves(int EB) { return EB <= 4 ? 16 : 8; }
constexpr int kRouteGroup = 64;

// Top-k of row (path p, sequence b) by one wave (logit descending, ties to the
// lower index) by repeated wave argmax, and the softmax over all experts
// gathered at the selection and renormalised = exp(r_e - max_sel) / sum over
// the selection.  Lane j holds selection j; sel0: the primary's, which a
// replaying branch of the same call (both) takes.
template <int VQ>
__device__ __forceinline__ void route_select(const MoeRoute &a, const float *lg, int p, int b, bool both, int &sel0) {
  const int E = a.E, lane = threadIdx.x & 63, k = p == 0 ? a.k1 : a.k2;
  int sel = 0;
  float val = -INFINITY;
  if (p == 1 && a.replay) {
    // the branch reuses the primary's experts
    sel = lane >= k ? 0 : both ? sel0 : a.idx1_in[(size_t)b * 8 + lane];
    val = lane >= k ? -INFINITY : lg[sel];
  } else {
    float v[VQ];
    bool open[VQ];  // not selected yet
#pragma unroll
    for (int q = 0; q < VQ; ++q) {
      open[q] = lane + 64 * q < E;
      v[q] = open[q] ? lg[lane + 64 * q] : -INFINITY;
    }
#pragma unroll 1
    for (int j = 0; j < k; ++j) {
      float best = -INFINITY;
#pragma unroll
      for (int q = 0; q < VQ; ++q) best = open[q] ? fmaxf(best, v[q]) : best;
      best = wave_max_dpp(best);
      int e = -1;
#pragma unroll
      for (int q = 0; q < VQ; ++q) {
        const unsigned long long m = __ballot(open[q] && v[q] == best);
        if (e < 0 && m) e = 64 * q + __ffsll(m) - 1;
      }
      if (e < 0)  // no number among what is left: the lowest of it
#pragma unroll
        for (int q = 0; q < VQ; ++q) {
          const unsigned long long m = __ballot(open[q]);
          if (e < 0 && m) e = 64 * q + __ffsll(m) - 1;
        }
#pragma unroll
      for (int q = 0; q < VQ; ++q) open[q] = open[q] && lane + 64 * q != e;
      if (lane == j) {
        sel = e;
        val = best;
      }
    }
  }
  sel0 = sel;
  const float mx = wave_max_dpp(lane < k ? val : -INFINITY), w = lane < k ? expf(val - mx) : 0.f;
  float den = 0.f;
#pragma unroll 1
  for (int j = 0; j < k; ++j) den += __shfl(w, j, 64);
  if (lane < k) {
    const size_t row = (size_t)prow(a.rows, p, b);
    int *oi = p == 0 ? a.out_idx1 : a.out_idx2;
    float *ow = p == 0 ? a.out_w1 : a.out_w2;
    const int kept = p != 0 || !a.ret_idx ? -1 : a.ret_map ? a.ret_map[b].keep : b;
    a.idx[row * 8 + lane] = sel;
    a.wts[row * 8 + lane] = w / den;
    if (oi) oi[(size_t)b * k + lane] = sel;
    if (ow) ow[(size_t)b * k + lane] = w / den;
    if (kept >= 0) a.ret_idx[(size_t)kept * 8 + lane] = sel;
  }
}

template <int EB, bool LOGITS = false>
__global__ __launch_bounds__(64 * route_waves(EB)) void k_moe_route(MoeRoute a) {
  constexpr int PITCH = 16 * EB + 4, kRouteWaves = route_waves(EB);
  __shared__ __attribute__((aligned(16))) float red[kRouteWaves][16][PITCH];
  __shared__ float ssr[kRouteWaves][16];
  const bool prim = a.mode != MODE_BRANCH, br = a.mode != MODE_PRIMARY;
  const bool both = prim && br;
  const int E = a.E, d = a.d, e0 = LOGITS ? (int)blockIdx.y * 16 * EB : 0;  // experts e0 ..
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, r = lane & 15, gq = lane >> 4;
  // row i of the workgroup: sequence and path
  const int per = both ? 8 : 16, b0 = blockIdx.x * per;
  auto path_of = [&](int i) { return both ? i / 8 : (prim ? 0 : 1); };
  auto seq_of = [&](int i) { return b0 + (both ? i % 8 : i); };
  const float *xr = a.Sbar + (size_t)prow(a.rows, path_of(r), min(seq_of(r), a.rows.B - 1)) * d + 8 * gq;
  const uint16_t *wr[EB];
#pragma unroll
  for (int q = 0; q < EB; ++q) wr[q] = (const uint16_t *)a.Wr + (size_t)min(e0 + 16 * q + r, E - 1) * d + 8 * gq;
  floatx4 acc[EB];
#pragma unroll
  for (int q = 0; q < EB; ++q) acc[q] = floatx4{0.f, 0.f, 0.f, 0.f};
  float ss = 0.f;
  struct Piece { floatx4 x[2], g[2]; u32x4 w[EB]; };
  auto load = [&](Piece &p, int k) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      p.x[h] = *(const floatx4 *)(xr + k + 4 * h);
      p.g[h] = *(const floatx4 *)(a.g + k + 8 * gq + 4 * h);
    }
#pragma unroll
    for (int q = 0; q < EB; ++q) p.w[q] = *(const u32x4 *)(wr[q] + k);
  };
  auto mul = [&](const Piece &p) {
    u32x4 part[3];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int e = 0; e < 4; e += 2) {
        float v0 = p.x[h][e], v1 = p.x[h][e + 1];
        ss = fmaf(v0, v0, fmaf(v1, v1, ss));
        v0 *= p.g[h][e];
        v1 *= p.g[h][e + 1];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const uint32_t u = pack2(v0, v1);
          part[c][2 * h + e / 2] = u;
          v0 -= __uint_as_float(u << 16);
          v1 -= __uint_as_float(u & 0xffff0000u);
        }
      }
#pragma unroll
    for (int c = 2; c >= 0; --c)  // smallest parts first
#pragma unroll
      for (int q = 0; q < EB; ++q)
        acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, p.w[q]),
                                                         __builtin_bit_cast(bf16x8, part[c]), acc[q], 0, 0, 0);
  };
  const int np = d / 32;  // a multiple of 16
  Piece cur, nxt;
  load(cur, wave * 32);
#pragma unroll 1
  for (int i = wave; i < np; i += kRouteWaves) {
    load(nxt, min(i + kRouteWaves, np - 1) * 32);
    mul(cur);
    cur = nxt;
  }
  // lane holds logits of experts 16 q + 4 gq .. + 3 for row r
#pragma unroll
  for (int q = 0; q < EB; ++q) *(floatx4 *)&red[wave][r][16 * q + 4 * gq] = acc[q];
  ss += __shfl_xor(ss, 16, 64);
  ss += __shfl_xor(ss, 32, 64);
  if (gq == 0) ssr[wave][r] = ss;
  __syncthreads();
  for (int e = t; e < 16 * 16 * EB; e += 64 * kRouteWaves) {
    const int i = e / (16 * EB), x = e % (16 * EB);
    float v = 0.f, q = 0.f;
#pragma unroll
    for (int w = 0; w < kRouteWaves; ++w) {
      v += red[w][i][x];
      q += ssr[w][i];
    }
    v *= 1.0f / sqrtf(q / (float)d + a.eps);
    red[0][i][x] = v;  // (read and written by this thread alone)
    const int b = seq_of(i);
    float *og = path_of(i) == 0 ? a.out_lg1 : a.out_lg2;
    if (e0 + x < E && b < a.rows.B) {
      if (og) og[(size_t)b * E + e0 + x] = v;
      if (LOGITS) a.logits[(size_t)prow(a.rows, path_of(i), b) * 256 + e0 + x] = v;
    }
  }
  if constexpr (LOGITS) return;
  __syncthreads();
  int sel0 = 0;
  // (a wave takes both rows of a sequence where the branch replays)
  const bool two = kRouteWaves == 8 || (both && a.replay);
  if (two && wave >= 8) return;
#pragma unroll 1
  for (int h = 0; h < (two ? 2 : 1); ++h) {
    const int i = !two ? wave : both ? wave + 8 * h : 2 * wave + h, p = path_of(i), b = seq_of(i);
    if (b >= a.rows.B) break;  // (uniform; later rows are past the end too)
    route_select<(EB + 3) / 4>(a, red[0][i], p, b, both, sel0);
  }
}

// The selection over logits in memory: a wave per sequence, its paths in turn.
template <int VQ>
__global__ __launch_bounds__(64) void k_moe_select(MoeRoute a) {
  const bool prim = a.mode != MODE_BRANCH, br = a.mode != MODE_PRIMARY;
  const int b = blockIdx.x;
  int sel0 = 0;
#pragma unroll 1
  for (int p = prim ? 0 : 1; p < (br ? 2 : 1); ++p)
    route_select<VQ>(a, a.logits + (size_t)prow(a.rows, p, b) * 256, p, b, prim && br, sel0);
}

// Expert-grouped order as a stable counting sort of the assignments
// (path, b, slot) by expert, in one workgroup of 16 waves: wave w takes the
// w-th of 16 equal ranges, 64 assignments at a time.  The lanes that chose the
// same expert find each other by ballots over the bits of its number, so a
// chunk costs the same whatever the choices; each wave counts its range, the
// counts are prefix-summed over the waves and the experts, and a second walk
// writes the positions.  Fixed order, no atomics.  (One thread per expert and
// range, each reading its whole range, took 13.6 us for 384 assignments and
// 42 us for 1400.)  Also lists the row tiles of kTileExpert rows of every
// expert for the tiled products.
__global__ __launch_bounds__(1024) void k_moe_dispatch(MoeDispatch a) {
  constexpr int W = 16;
  __shared__ int cnt[W][256];
  __shared__ int eoff[256];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int E = a.E, B = a.rows.B;
  const int n0 = a.rows.p0 == 0 ? B * a.k1 : 0, A = n0 + (a.rows.p0 + a.rows.np > 1 ? B * a.k2 : 0);
  const int chunks = (A + 63) / 64, c0 = wave * chunks / W, c1 = (wave + 1) * chunks / W;
  // assignment f: its row and slot
  auto where = [&](int f, int &slot) {
    const bool first = f < n0;
    const int k = first ? a.k1 : a.k2, q = first ? f : f - n0, b = q / k;
    slot = q - b * k;
    return prow(a.rows, first ? 0 : 1, b);
  };
  // lanes of the chunk that chose this lane's expert (e < 0: no assignment)
  auto same = [&](int e) {
    unsigned long long m = __ballot(e >= 0);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const unsigned long long b = __ballot((e >> i) & 1);
      m &= ((e >> i) & 1) ? b : ~b;
    }
    return m;
  };
  const unsigned long long below = (1ull << lane) - 1ull;
  for (int e = lane; e < 256; e += 64) cnt[wave][e] = 0;
  wave_lds_fence();
  constexpr int U = 4;  // chunks whose loads are in flight together
  auto walk = [&](auto &&take) {
    for (int c = c0; c < c1; c += U) {
      int e[U], row[U], slot[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int f = (c + u) * 64 + lane;
        const bool live = c + u < c1 && f < A;
        row[u] = where(live ? f : 0, slot[u]);
        const int x = a.idx[(size_t)row[u] * 8 + slot[u]];
        e[u] = live ? x : -1;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const unsigned long long m = same(e[u]);
        if (e[u] >= 0) take(e[u], row[u], slot[u], cnt[wave][e[u]] + __popcll(m & below));
        wave_lds_fence();
        if (e[u] >= 0 && (m & below) == 0) cnt[wave][e[u]] += __popcll(m);
        wave_lds_fence();
      }
    }
  };
  walk([](int, int, int, int) {});
  __syncthreads();
  if (t < 256) {
    int acc = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const int v = cnt[w][t];
      cnt[w][t] = acc;
      acc += v;
    }
    eoff[t] = acc;
    if (t < E) a.counts[t] = acc;
  }
  __syncthreads();
  if (t < 64) {
    // exclusive scans over experts (lane l: experts 4l..4l+3) of the
    // assignments and of the row tiles
    int v[4], n[4], s = 0, ts = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[i] = eoff[4 * lane + i];
      n[i] = (v[i] + kTileExpert - 1) / kTileExpert;
      s += v[i];
      ts += n[i];
    }
    int is = s, its = ts;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int u = __shfl_up(is, o, 64), ut = __shfl_up(its, o, 64);
      if (lane >= o) {
        is += u;
        its += ut;
      }
    }
    int off = is - s, toff = its - ts;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = 4 * lane + i;
      eoff[e] = off;
      if (e < E) a.offsets[e] = off;
      off += v[i];
      if (a.tiles)
        for (int j = 0; j < n[i]; ++j) a.tiles[toff + j] = make_int2(e, j * kTileExpert);
      toff += n[i];
    }
    if (lane == 63) {
      a.offsets[E] = is;
      if (a.ntiles) *a.ntiles = its;
    }
  }
  __syncthreads();
  for (int e = lane; e < 256; e += 64) cnt[wave][e] += eoff[e];
  wave_lds_fence();
  walk([&](int, int row, int slot, int pos) {
    a.arow[pos] = row;
    a.aslot[(size_t)row * 8 + slot] = pos;
  });
}

constexpr int kChunk = 128;
constexpr int kLdsRow = kChunk + 8;

// Expert projections over gathered rows.  GATEUP: workgroup = (expert,
// 64 hidden units); wave w owns hidden units h0+16w..+15 with row block 0 =
// gate rows and row block 1 = up rows, so SwiGLU is lane-local.  DOWN:
// workgroup = (expert, 64 output columns), wave w owns 16 of them.  The
// workgroup takes all rows of its expert in passes of 16*MB (one pass unless
// the expert is crowded; a further pass reads its weights again); an
// untouched expert's workgroups return before any weight read.
//
// Weight loads as in the dense projections: whole 128-byte row pieces with
// the non-temporal hint (eight rows per wave instruction), moved into the
// MFMA operand layout through the wave's LDS region half a chunk at a time.
template <int MB, bool GATEUP>
__global__ __launch_bounds__(256) void k_moe_gemm(MoeGemm a) {
  constexpr int RB = GATEUP ? 2 : 1;
  constexpr int PD = 2;
  constexpr int XR = 16 * MB;
  constexpr int PIECES = XR * (kChunk / 8);
  constexpr int PPT = (PIECES + 255) / 256;
  __shared__ uint16_t xs[PD][XR * kLdsRow];
  __shared__ int rows_s[XR];
  __shared__ u32x4 wt[4][RB * 16 * 8];
  const int tiles = a.N / 64;
  const int e = blockIdx.x / tiles, tile = blockIdx.x % tiles;
  const int Me = a.counts[e];
  if (Me <= 0) return;  // untouched expert: no weight read
  const int base = a.offsets[e];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, r = lane & 15, gq = lane >> 4;
  const int K = a.K, nch = K / kChunk;
  const int n0 = tile * 64 + wave * 16;
  // coalesced weight loads: row block rb, row group j (rows j*8 + lane/8 of
  // the block), 16-byte piece lane%8 of a 128-byte half chunk
  const int lr8 = lane >> 3, lp8 = lane & 7;
  const uint16_t *wrow[RB][2];
#pragma unroll
  for (int rb = 0; rb < RB; ++rb)
#pragma unroll
    for (int j = 0; j < 2; ++j)
      wrow[rb][j] = (const uint16_t *)(rb == 0 ? a.W0 : a.W1) + ((size_t)e * a.N + n0 + j * 8 + lr8) * K + lp8 * 8;
  u32x4 *wreg = wt[wave];
  u32x4 w[PD][RB][4];
  u32x4 stage[PPT];
  auto wload = [&](int slot, int c) {
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          w[slot][rb][2 * h + j] = __builtin_nontemporal_load((const u32x4 *)(wrow[rb][j] + c * kChunk + h * 64));
  };
  auto xload = [&](int c) {
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
      const int p = t + 256 * j;
      const int row = p >> 4, col = (p & 15) * 8;
      const int src = p < PIECES ? rows_s[row] : -1;
      stage[j] = src >= 0 ? *(const u32x4 *)((const uint16_t *)a.X + (size_t)src * a.ldx + c * kChunk + col)
                          : u32x4{0u, 0u, 0u, 0u};
    }
  };
  auto xstore = [&](int slot) {
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
      const int p = t + 256 * j;
      if (p < PIECES) *(u32x4 *)(&xs[slot][(p >> 4) * kLdsRow + (p & 15) * 8]) = stage[j];
    }
  };
  for (int m0 = 0; m0 < Me; m0 += XR) {
    if (m0 > 0) __syncthreads();  // the previous pass is done with rows_s and xs
    if (t < XR) rows_s[t] = (m0 + t < Me) ? (GATEUP ? a.arow[base + m0 + t] : base + m0 + t) : -1;
    const int nb = (min(Me - m0, XR) + 15) / 16;  // live activation blocks
    __syncthreads();
    floatx4 acc[RB][MB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
      for (int cb = 0; cb < MB; ++cb) acc[rb][cb] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < PD; ++u)
      if (u < nch) {
        xload(u);
        xstore(u);
        wload(u, u);
      }
    __syncthreads();
    for (int c0 = 0; c0 < nch; c0 += PD) {
#pragma unroll
      for (int u = 0; u < PD; ++u) {
        const int c = c0 + u;
        if (c < nch) {
          const bool more = c + PD < nch;
          if (more) xload(c + PD);
#pragma unroll
          for (int h = 0; h < 2; ++h) {
#pragma unroll
            for (int rb = 0; rb < RB; ++rb)
#pragma unroll
              for (int j = 0; j < 2; ++j) wreg[(rb * 16 + j * 8 + lr8) * 8 + (lp8 ^ lr8)] = w[u][rb][2 * h + j];
            wave_lds_fence();
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2) {
              const int s = 2 * h + s2;
              u32x4 wf[RB];
#pragma unroll
              for (int rb = 0; rb < RB; ++rb) wf[rb] = wreg[(rb * 16 + r) * 8 + ((4 * s2 + gq) ^ (r & 7))];
#pragma unroll
              for (int cb = 0; cb < MB; ++cb) {
                if (cb < nb) {
                  const u32x4 bx = *(const u32x4 *)(&xs[u][(cb * 16 + r) * kLdsRow + s * 32 + gq * 8]);
#pragma unroll
                  for (int rb = 0; rb < RB; ++rb)
                    acc[rb][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        __builtin_bit_cast(bf16x8, wf[rb]), __builtin_bit_cast(bf16x8, bx), acc[rb][cb], 0, 0, 0);
                }
              }
            }
            wave_lds_fence();
          }
          if (more) wload(u, c + PD);
          __syncthreads();
          if (more) xstore(u);
        }
      }
    }
    // lane holds D[n = n0 + 4gq + i][m = m0 + cb*16 + r]
#pragma unroll
    for (int cb = 0; cb < MB; ++cb) {
      const int m = m0 + cb * 16 + r;
      if (cb >= nb || m >= Me) continue;
      const size_t orow = (size_t)(base + m);
      if (GATEUP) {
        uint16_t h[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const float g = acc[0][cb][i], up = acc[RB - 1][cb][i];
          h[i] = f2bf(g / (1.0f + expf(-g)) * up);
        }
        uint2 v;
        v.x = (uint32_t)h[0] | ((uint32_t)h[1] << 16);
        v.y = (uint32_t)h[2] | ((uint32_t)h[3] << 16);
        *(uint2 *)((uint16_t *)a.Y + orow * a.ldy + n0 + gq * 4) = v;
      } else {
        *(floatx4 *)((float *)a.Y + orow * a.ldy + n0 + gq * 4) = acc[0][cb];
      }
    }
  }
}

// Routed sum (ascending expert id) + shared expert + c coupling + residual +
// next norm.  One workgroup per sequence (both paths), float4 columns.
template <typename T>
__global__ void k_moe_combine(MoeCombine a) {
  __shared__ float red[16];
  __shared__ int sl[2][8];
  __shared__ float sw[2][8];
  const int b = blockIdx.x;
  const bool prim = a.mode != MODE_BRANCH, br = a.mode != MODE_PRIMARY;
  const int d = a.d, d4 = d / 4;
  const int r1 = prow(a.rows, 0, b), r2 = prow(a.rows, 1, b);
  if (threadIdx.x < 2) {
    // selected experts of this path in ascending id order (insertion sort, k <= 8)
    const int p = threadIdx.x;
    const int k = p == 0 ? a.k1 : a.k2;
    const int r = p == 0 ? r1 : r2;
    if ((p == 0 && prim) || (p == 1 && br)) {
      // all eight slots of the row loaded at once (the arrays hold 8 per row),
      // then an odd-even transposition sort in registers; slots >= k sort last
      int id[8], sj[8];
      float wj[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int v = a.idx[(size_t)r * 8 + j];
        id[j] = j < k ? v : 0x7fffffff;
        sj[j] = a.aslot[(size_t)r * 8 + j];
        wj[j] = a.wts[(size_t)r * 8 + j];
      }
#pragma unroll
      for (int round = 0; round < 8; ++round)
#pragma unroll
        for (int j = round & 1; j + 1 < 8; j += 2)
          if (id[j + 1] < id[j]) {
            const int ti = id[j], ts = sj[j];
            const float tw = wj[j];
            id[j] = id[j + 1];
            sj[j] = sj[j + 1];
            wj[j] = wj[j + 1];
            id[j + 1] = ti;
            sj[j + 1] = ts;
            wj[j + 1] = tw;
          }
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        sl[p][j] = j < k ? sj[j] : sj[0];  // padding: a valid row with weight 0
        sw[p][j] = j < k ? wj[j] : 0.f;
      }
    }
  }
  __syncthreads();
  float4 *s1 = (float4 *)(a.S + (size_t)r1 * d);
  float4 *s2 = (float4 *)(a.S + (size_t)r2 * d);
  float4 *o1 = a.ho.row(0, b, d, s1), *o2 = a.ho.row(1, b, d, s2);
  const int kept_row = a.ret.row(b);
  const bool keep = kept_row >= 0;
  float4 *kept = keep ? (float4 *)(a.ret.ptr + (size_t)kept_row * d) : nullptr;
  // routed experts, ascending id; all eight slots (weight 0 past k: adding
  // zeros leaves the sum unchanged) so the loads are in flight together
  auto experts = [&](int p, int k, int i) {
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float4 y = ((const float4 *)(a.Yexp + (size_t)sl[p][j] * d))[i];
      const float w = sw[p][j];
      acc.x += w * y.x;
      acc.y += w * y.y;
      acc.z += w * y.z;
      acc.w += w * y.w;
    }
    return acc;
  };
  auto shared = [&](int row, int i) {  // shared-expert slabs in split order
    float4 sh = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
    for (int q = 0; q < a.S_sh; ++q) {
      const float4 v = ((const float4 *)(a.part + q * a.stride + (size_t)row * d))[i];
      sh.x += v.x;
      sh.y += v.y;
      sh.z += v.z;
      sh.w += v.w;
    }
    return sh;
  };
  const bool cm = a.gG != nullptr;  // compute-matched variant (App. B.3)
  for (int i = threadIdx.x; i < d4; i += blockDim.x) {
    float4 m1, g1;  // primary MoE output; primary shared-expert output
    if (prim) {
      const float4 r = experts(0, a.k1, i);
      g1 = shared(r1, i);
      m1 = make_float4(r.x + g1.x, r.y + g1.y, r.z + g1.z, r.w + g1.w);
      const float4 s = s1[i];
      o1[i] = make_float4(s.x + m1.x, s.y + m1.y, s.z + m1.z, s.w + m1.w);
      if (keep) kept[i] = cm ? g1 : m1;
    } else {
      m1 = g1 = ((const float4 *)(a.M1_in + (size_t)b * d))[i];
    }
    if (br) {
      const float4 r = experts(1, a.k2, i);
      const float4 s = s2[i];
      if (cm) {  // M2 = R2 + g_G * G1
        const float4 gg = ((const float4 *)a.gG)[i];
        o2[i] = make_float4(s.x + (r.x + gg.x * g1.x), s.y + (r.y + gg.y * g1.y), s.z + (r.z + gg.z * g1.z),
                            s.w + (r.w + gg.w * g1.w));
      } else {   // M2 = R2 + shared expert of the branch + c * M1
        const float4 g2 = shared(r2, i);
        const float4 c = ((const float4 *)a.c)[i];
        o2[i] = make_float4(s.x + ((r.x + g2.x) + c.x * m1.x), s.y + ((r.y + g2.y) + c.y * m1.y),
                            s.z + ((r.z + g2.z) + c.z * m1.z), s.w + ((r.w + g2.w) + c.w * m1.w));
      }
    }
  }
  if (!a.g_next) return;
  __syncthreads();
  for (int p = 0; p < 2; ++p) {
    if ((p == 0 && !prim) || (p == 1 && !br)) continue;
    const float *x = (const float *)(p == 0 ? o1 : o2);
    T *out = (T *)a.Xn + (size_t)(p == 0 ? r1 : r2) * a.ldx;
    float ss = 0.f;
    for (int i = threadIdx.x; i < d; i += blockDim.x) ss += x[i] * x[i];
    ss = block_sum(ss, red);
    const float inv = 1.0f / sqrtf(ss / (float)d + a.eps);
    for (int i = threadIdx.x; i < d; i += blockDim.x) st<T>(out, i, x[i] * inv * a.g_next[i]);
    __syncthreads();
  }
}

template <bool GATEUP>
hipError_t launch_moe_gemm_t(const MoeGemm &a, int MB, hipStream_t st) {
  dim3 grid(a.E * (a.N / 64), 1, 1);
  switch (MB) {
    case 1: hipLaunchKernelGGL((k_moe_gemm<1, GATEUP>), grid, dim3(256), 0, st, a); break;
    default: hipLaunchKernelGGL((k_moe_gemm<2, GATEUP>), grid, dim3(256), 0, st, a); break;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_moe_route(const MoeRoute &a, hipStream_t st) {
  if (a.E < 1 || a.E > 256 || a.d % 512 != 0 || a.d > 4096) return hipErrorInvalidValue;
  const int per = a.mode == MODE_GROUPED ? 8 : 16;
  const int eb = (a.E + 15) / 16;
  const dim3 grid((a.rows.B + per - 1) / per), block(64 * route_waves(eb));
  if (a.E > kRouteOne) {
    if (!a.logits) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_moe_route<kRouteGroup / 16, true>), dim3(grid.x, (a.E + kRouteGroup - 1) / kRouteGroup),
                       dim3(64 * route_waves(kRouteGroup / 16)), 0, st, a);
    hipLaunchKernelGGL(k_moe_select<4>, dim3(a.rows.B), dim3(64), 0, st, a);
  } else if (eb <= 1) hipLaunchKernelGGL(k_moe_route<1>, grid, block, 0, st, a);
  else if (eb <= 2) hipLaunchKernelGGL(k_moe_route<2>, grid, block, 0, st, a);
  else if (eb <= 4) hipLaunchKernelGGL(k_moe_route<4>, grid, block, 0, st, a);
  else hipLaunchKernelGGL(k_moe_route<8>, grid, block, 0, st, a);
  return hipGetLastError();
}

hipError_t launch_moe_dispatch(const MoeDispatch &a, hipStream_t st) {
  if (a.E < 1 || a.E > 256) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_moe_dispatch, dim3(1), dim3(1024), 0, st, a);
  return hipGetLastError();
}

// 32-row activation passes: an expert usually gets a handful of rows; the
// rare crowded expert takes more passes (its weights are then read again).
hipError_t launch_moe_gemm(const MoeGemm &a, bool gateup, int max_rows, hipStream_t st) {
  const int MB = max_rows > 16 ? 2 : 1;
  return gateup ? launch_moe_gemm_t<true>(a, MB, st) : launch_moe_gemm_t<false>(a, MB, st);
}

hipError_t launch_moe_combine(const MoeCombine &a, int dtype, hipStream_t st) {
  if (dtype == 1)
    hipLaunchKernelGGL(k_moe_combine<uint16_t>, dim3(a.rows.B), dim3(256), 0, st, a);
  else
    hipLaunchKernelGGL(k_moe_combine<float>, dim3(a.rows.B), dim3(256), 0, st, a);
  return hipGetLastError();
}

}  // namespace dbt
