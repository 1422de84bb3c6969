// Projections of a whole prompt (primary prefill, Sec. 4.4): Y = X W^T with
// thousands of activation rows, where every weight row is reused by many
// rows and the work is bound by the matrix cores, not by the weight read.
//
// Workgroup of eight waves per BM-row x BN-column output tile, reduction steps
// of BK.  Waves form a 2 (rows) x 4 (columns) grid; a wave owns BM/2 rows x
// BN/4 columns and multiplies with v_mfma_f32_16x16x32_bf16, W as the A
// operand and X as the B operand, so each lane ends with four consecutive
// output columns of one row (16-byte stores).
//
// Schedule: each SIMD holds two waves, and they alternate: while one issues
// half a step's multiplies, the other reads its next operands from LDS,
// starts loads of a later step and waits for what it needs; a barrier swaps
// the two roles (waves 4..7 run half a phase behind, set up by one extra
// barrier).  A step is two phases, the row halves of the wave's tile: the
// first reads W and X half 0, the second X half 1.  LDS holds two steps, each
// as four arrays (the halves of X and W).  Loads go straight from global
// memory into LDS (global_load_lds_dwordx4) as soon as both wave groups have
// read what they replace: W and X half 0 of step kt + 2 in the second phase of
// step kt, X half 1 of it in the first phase of step kt + 1, so each has a
// whole step to land; a phase waits until at most one step's loads are
// outstanding, which is when the next phase's operands are complete.
// Measured on 8192 rows of width 2048, against one barrier and one full wait
// per step with the two waves of a SIMD in lockstep: gate/up with 5632 units
// 325 -> 300 us (1.26 PFLOP/s; a library product of the same size 0.97; 319
// since its SwiGLU takes expf and a divide), W_O
// and down 64 + 165 -> 58 + 134 us.  Without its loads gate/up takes 227 us,
// without the half-phase offset 344 us.
//
// LDS rows are BK elements; the 16-byte chunk c of row r sits at chunk
// c ^ (r & (BK/8 - 1)): operand reads (16 consecutive rows at one chunk) and
// the loads' writes are then free of bank conflicts (measured).
//
// Epilogues (EPI): plain fp32 output; GLU, the gate/up projection of the
// SwiGLU MLP (Eq. (13), primary rows): a wave's column halves are the gate and
// the up rows of the same outputs, and the epilogue writes H = silu(gate) * up
// in bf16 (and keeps rows in fp32 when asked) instead of the fp32 gate/up
// outputs; QKV, the stacked Q/K/V projection of a prompt (Eq. (8)): a tile is
// BN/128 heads, a wave's column halves are dimensions i and i + 64 of one head
// (the rotary pairs), and the epilogue applies the rotary embedding to Q and
// K, writes Q in fp32 (and the kept rows) and K and V in the model dtype into
// the cache pages, instead of the fp32 Q/K/V outputs.
#include "common.h"
#include "kernels.h"

#include <algorithm>
#include <type_traits>

namespace dbt {

namespace {

typedef __attribute__((address_space(3))) void lds_void;

enum { EPI_PLAIN = 0, EPI_GLU = 1, EPI_QKV = 2 };

// Workgroup barrier without the waits of __syncthreads: loads into LDS stay in
// flight across it.
__device__ __forceinline__ void phase_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("" ::: "memory");
}

// s_waitcnt vmcnt(N), every LDS operation done (expcnt not waited).
template <int N>
__device__ __forceinline__ void wait_loads() {
  __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (0 << 8) | ((N >> 4) << 14));
}

template <int BM, int BN, int BK, int EPI, bool MOE = false>
__global__ __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_gemm_tile(TileGemm g) {
  constexpr bool GLU = EPI == EPI_GLU, QKV = EPI == EPI_QKV;
  constexpr int MH = BM / 64;   // 16-row blocks of a wave's row half
  constexpr int NH = BN / 128;  // 16-column blocks of a wave's column half
  constexpr int NS = BK / 32;   // 32-element pieces of a step
  constexpr int LPR = BK / 8, RPL = 64 / LPR;  // lanes (16-byte chunks) per row, rows per load instruction
  constexpr int XL = BM * BK / 8192, WL = BN * BK / 8192;  // loads of a wave per half operand
  constexpr int OUT = 2 * (XL + WL);           // loads of a step
  __shared__ __attribute__((aligned(16))) uint16_t xa0[BM / 2 * BK], xb0[BM / 2 * BK], xa1[BM / 2 * BK], xb1[BM / 2 * BK];
  __shared__ __attribute__((aligned(16))) uint16_t wa0[BN / 2 * BK], wb0[BN / 2 * BK], wa1[BN / 2 * BK], wb1[BN / 2 * BK];
  const int t = threadIdx.x, lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
  const int r = lane & 15, gq = lane >> 4;
  const int wm = (wave >> 1) & 1, wn = 2 * (wave >> 2) + (wave & 1);  // waves w and w + 4 share a SIMD and a row half
  // Output tile: the workgroups of one XCD (every eighth) take a contiguous
  // range of an order that walks down columns of eight row tiles, so the
  // tiles an XCD works on at a time share their rows and columns in its L2.
  const int gx = gridDim.x, gy = gridDim.y, total = gx * gy * gridDim.z;
  int tx, ty, split;
  {
    const int id = (blockIdx.z * gy + blockIdx.y) * gx + blockIdx.x, per = total / 8, rest = total % 8, xcd = id % 8;
    int p = xcd * per + min(xcd, rest) + id / 8;
    split = p / (gx * gy);
    p -= split * gx * gy;
    const int band = p / (8 * gx), rows = min(8, gy - 8 * band), q = p - band * 8 * gx;
    tx = q / rows;
    ty = 8 * band + q % rows;
  }
  // MOE: row tile ty of the list, an expert's rows m0 .. (XCD order aside: the
  // list is shorter than the grid, and an expert's tiles share no weights)
  int M = g.M, row0 = 0, m0 = ty * BM;
  size_t we = 0;
  if constexpr (MOE) {
    static_assert(BM == kTileExpert, "the list's tiles");
    if ((int)blockIdx.y >= *g.ntiles) return;
    const int2 tile = g.tiles[blockIdx.y];
    tx = blockIdx.x;
    m0 = tile.y;
    M = g.counts[tile.x];
    row0 = g.offsets[tile.x];
    we = (size_t)tile.x * g.N * g.K;
  }
  const int n0 = tx * (GLU ? BN / 2 : BN);
  // split z of the reduction: steps k_lo .. k_hi - 1, a whole number of
  // 128-element pieces (plain outputs, one slab per split)
  const int K = g.K, k_lo = split * (K / 128) / (int)gridDim.z * (128 / BK), k_hi = (split + 1) * (K / 128) / (int)gridDim.z * (128 / BK);
  const int nk = k_hi - k_lo;

  // A half operand is filled row group by row group: one instruction of a
  // wave fills RPL whole rows, lane l the 16-byte slot l % LPR of row l / LPR,
  // so each lane fetches the chunk that the swizzle places in its slot.  The base of a group's matrix stays in scalar registers, a lane
  // keeps a 32-bit byte offset; rows past the end re-read the last row.
  const int lrow = lane / LPR;
  auto lchunk = [&](int R) { return (lane % LPR) ^ ((R + lrow) & (LPR - 1)); };
  // X half h, its row R: tile row (R / (BM/4)) * BM/2 + h * BM/4 + R % (BM/4)
  uint32_t xo[2][XL];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < XL; ++i) {
      const int R = RPL * (XL * wave + i), row = m0 + R / (BM / 4) * (BM / 2) + h * (BM / 4) + R % (BM / 4) + lrow;
      int src = min(row, M - 1);
      if constexpr (MOE) src = g.arow ? g.arow[row0 + src] : row0 + src;
      xo[h][i] = ((uint32_t)src * (uint32_t)g.ldx + k_lo * BK + lchunk(R) * 8) * 2;
    }
  // W half h, its row R: wave column w = R / (BN/8), its row R % (BN/8)
  const uint16_t *wb[2][WL];
  uint32_t wo[2][WL];
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int i = 0; i < WL; ++i) {
      const int R = RPL * (WL * wave + i), w = R / (BN / 8), c = R % (BN / 8);
      if (GLU) {
        wb[h][i] = g.w[h] + we;
        wo[h][i] = ((uint32_t)min(n0 + w * (BN / 8) + c + lrow, g.N - 1) * (uint32_t)K + k_lo * BK + lchunk(R) * 8) * 2;
      } else {
        // first column of the group; QKV: head w / (512 / BN), dimension 64 h + ...
        const int col = QKV ? n0 + w / (512 / BN) * 128 + 64 * h + w % (512 / BN) * (BN / 8) + c
                            : n0 + w * (BN / 4) + h * (BN / 8) + c;
        int seg = min(col, g.N - 1), row = min(col + lrow, g.N - 1);
        const uint16_t *base = g.w[0];
        if (!MOE && seg >= g.rows[0]) {  // segment sizes are multiples of 8: one segment per group
          seg -= g.rows[0];
          row -= g.rows[0];
          base = g.w[1];
          if (seg >= g.rows[1]) {
            row -= g.rows[1];
            base = g.w[2];
          }
        }
        wb[h][i] = base + we;
        wo[h][i] = ((uint32_t)row * (uint32_t)K + k_lo * BK + lchunk(R) * 8) * 2;
      }
    }
  auto load_x = [&](int h, int kt, uint16_t *dst) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < XL; ++i)
      __builtin_amdgcn_global_load_lds((const void *)((const char *)(g.X + kt * BK) + xo[h][i]),
                                       (lds_void *)(dst + RPL * (XL * wave + i) * BK), 16, 0, 0);
  };
  auto load_w = [&](int h, int kt, uint16_t *dst) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < WL; ++i)
      __builtin_amdgcn_global_load_lds((const void *)((const char *)(wb[h][i] + kt * BK) + wo[h][i]),
                                       (lds_void *)(dst + RPL * (WL * wave + i) * BK), 16, 0, 0);
  };
  // operands: block b (16 rows) of the wave's half, piece s (32 elements)
  auto read_x = [&](const uint16_t *src, u32x4 (&f)[MH][NS]) __attribute__((always_inline)) {
#pragma unroll
    for (int b = 0; b < MH; ++b)
#pragma unroll
      for (int s = 0; s < NS; ++s)
        f[b][s] = *(const u32x4 *)&src[(wm * (BM / 4) + 16 * b + r) * BK + (((4 * s + gq) ^ (r & (LPR - 1))) * 8)];
  };
  auto read_w = [&](const uint16_t *src, u32x4 (&f)[NH][NS]) __attribute__((always_inline)) {
#pragma unroll
    for (int a = 0; a < NH; ++a)
#pragma unroll
      for (int s = 0; s < NS; ++s)
        f[a][s] = *(const u32x4 *)&src[(wn * (BN / 8) + 16 * a + r) * BK + (((4 * s + gq) ^ (r & (LPR - 1))) * 8)];
  };

  // acc[j][a][i][b]: column half j, block a; row half i, block b
  floatx4 acc[2][NH][2][MH];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int a = 0; a < NH; ++a)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int b = 0; b < MH; ++b) acc[j][a][i][b] = floatx4{0.f, 0.f, 0.f, 0.f};
  u32x4 xf[MH][NS], wf0[NH][NS], wf1[NH][NS];
  auto mma = [&](int i) __attribute__((always_inline)) {
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int a = 0; a < NH; ++a)
#pragma unroll
          for (int b = 0; b < MH; ++b)
            acc[j][a][i][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, j ? wf1[a][s] : wf0[a][s]),
                                                                      __builtin_bit_cast(bf16x8, xf[b][s]),
                                                                      acc[j][a][i][b], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
  };
  // Step kt on the arrays of its parity (xa, xb, wa, wb_); xbo: X half 1 of the
  // other parity.  LEFT: steps after this one, at most 2; the last two load
  // less and wait for what is left (compile-time, so that the compiler sees
  // which loads can be outstanding at each read and adds no waits of its own).
  auto step = [&](auto left, int kt, uint16_t *xa, uint16_t *xb, uint16_t *wa, uint16_t *wb_, uint16_t *xbo) __attribute__((always_inline)) {
    constexpr int LEFT = decltype(left)::value;
    auto turn = [&](auto n) __attribute__((always_inline)) {
      __builtin_amdgcn_sched_barrier(0);
      wait_loads<decltype(n)::value>();
      phase_barrier();
    };
    // row half 0
    read_w(wa, wf0);
    read_w(wb_, wf1);
    read_x(xa, xf);
    if constexpr (LEFT >= 1) load_x(1, kt + 1, xbo);
    turn(std::integral_constant<int, (LEFT >= 1 ? OUT : 0)>{});
    mma(0);
    phase_barrier();
    // row half 1
    read_x(xb, xf);
    if constexpr (LEFT >= 2) {
      load_w(0, kt + 2, wa);
      load_w(1, kt + 2, wb_);
      load_x(0, kt + 2, xa);
    }
    turn(std::integral_constant<int, (LEFT >= 2 ? OUT : LEFT == 1 ? XL : 0)>{});
    mma(1);
    phase_barrier();
  };

  using std::integral_constant;
  const int k1 = BK == 128 ? min(1, nk - 1) : 1;
  load_w(0, 0, wa0);
  load_w(1, 0, wb0);
  load_x(0, 0, xa0);
  load_x(1, 0, xb0);
  load_w(0, k1, wa1);
  load_w(1, k1, wb1);
  load_x(0, k1, xa1);
  wait_loads<OUT>();
  phase_barrier();
  if (wave >= 4) phase_barrier();  // half a phase behind from here on
  int kt = 0;
  if constexpr (BK == 128) {  // (nk may be odd: one step or three are left)
    for (; kt + 3 < nk; kt += 2) {
      step(integral_constant<int, 2>{}, kt, xa0, xb0, wa0, wb0, xb1);
      step(integral_constant<int, 2>{}, kt + 1, xa1, xb1, wa1, wb1, xb0);
    }
    if (nk - kt == 3) {
      step(integral_constant<int, 2>{}, kt, xa0, xb0, wa0, wb0, xb1);
      step(integral_constant<int, 1>{}, kt + 1, xa1, xb1, wa1, wb1, xb0);
      step(integral_constant<int, 0>{}, kt + 2, xa0, xb0, wa0, wb0, xb1);
    } else if (nk - kt == 2) {
      step(integral_constant<int, 1>{}, kt, xa0, xb0, wa0, wb0, xb1);
      step(integral_constant<int, 0>{}, kt + 1, xa1, xb1, wa1, wb1, xb0);
    } else {
      step(integral_constant<int, 0>{}, kt, xa0, xb0, wa0, wb0, xb1);
    }
  } else {
    for (; kt + 2 < nk; kt += 2) {
      step(integral_constant<int, 2>{}, kt, xa0, xb0, wa0, wb0, xb1);
      step(integral_constant<int, 2>{}, kt + 1, xa1, xb1, wa1, wb1, xb0);
    }
    step(integral_constant<int, 1>{}, kt, xa0, xb0, wa0, wb0, xb1);
    step(integral_constant<int, 0>{}, kt + 1, xa1, xb1, wa1, wb1, xb0);
  }
  if (wave < 4) phase_barrier();
  __syncthreads();  // no load into LDS outlives the workgroup

  // epilogue: lane holds output rows m0 + BM/2 wm + BM/4 i + 16 b + r, columns
  // 16 a + 4 gq .. + 3 of the wave's column half j
#pragma unroll
  for (int ib = 0; ib < 2 * MH; ++ib) {
    const int i = ib / MH, b = ib % MH;
    const int m = m0 + BM / 2 * wm + BM / 4 * i + 16 * b + r;
    if (m >= M) continue;
    const int kept_row = !MOE && (GLU || QKV) ? g.ret.row(m) : -1;
    if (QKV) {
      // heads of 128: Q, then K, then V
      const int hn0 = n0 + wn / (512 / BN) * 128;
      if (hn0 >= g.N) continue;
      const int dq = g.rows[0], dkv = g.rows[1];
      const int pos = g.prompt[m].pos;
      const size_t page = (size_t)g.kv.page_table[(size_t)g.prompt[m].seq * g.kv.mpps + pos / 16];
      const int slot = pos % 16;
#pragma unroll
      for (int a = 0; a < NH; ++a) {
        const int d0 = wn % (512 / BN) * (BN / 8) + 16 * a + 4 * gq;  // dimensions d0 .. d0+3 and d0+64 .. d0+67
        float x0[4], x1[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          x0[e] = acc[0][a][i][b][e];
          x1[e] = acc[1][a][i][b][e];
        }
        if (hn0 < dq + dkv) {  // uniform over the wave: rotary embedding on Q and K
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float2 y = rope_pair(x0[e], x1[e], g.rope[(size_t)pos * 64 + d0 + e]);
            x0[e] = y.x;
            x1[e] = y.y;
          }
        }
        if (hn0 < dq) {
          const int c0 = hn0 + d0;
          *(float4 *)(g.Qout + (size_t)m * dq + c0) = float4{x0[0], x0[1], x0[2], x0[3]};
          *(float4 *)(g.Qout + (size_t)m * dq + c0 + 64) = float4{x1[0], x1[1], x1[2], x1[3]};
          if (kept_row >= 0) {
            float *kept = g.ret.ptr + (size_t)kept_row * dq + c0;
            *(float4 *)kept = float4{x0[0], x0[1], x0[2], x0[3]};
            *(float4 *)(kept + 64) = float4{x1[0], x1[1], x1[2], x1[3]};
          }
        } else if (hn0 < dq + dkv) {
          const int hd = (hn0 - dq) / 128;
          uint16_t *kp = (uint16_t *)g.kv.k + ((page * g.kv.n_kv + hd) * 16 + slot) * 128;
          *(u32x2 *)(kp + d0) = u32x2{pack2(x0[0], x0[1]), pack2(x0[2], x0[3])};
          *(u32x2 *)(kp + d0 + 64) = u32x2{pack2(x1[0], x1[1]), pack2(x1[2], x1[3])};
        } else {
          const int hd = (hn0 - dq - dkv) / 128;
          uint16_t *vp = (uint16_t *)g.kv.v + (page * g.kv.n_kv + hd) * 128 * 16 + slot;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            vp[(d0 + e) * 16] = f2bf(x0[e]);
            vp[(d0 + 64 + e) * 16] = f2bf(x1[e]);
          }
        }
      }
    } else if (GLU) {
#pragma unroll
      for (int a = 0; a < NH; ++a) {
        const int j = n0 + wn * (BN / 8) + 16 * a + 4 * gq;
        if (j >= g.N) continue;
        float h[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          // silu as every other kernel of the framework computes it (the kept
          // rows are fp32, and a pass of fewer rows takes other kernels).
          // v_exp_f32 and v_rcp_f32 instead of expf and a divide: 951
          // instead of 974 us for 24 prompts of 17-300 positions, 2461
          // instead of 2500 us for one of 8192 (two layers of 5632 units)
          const float gt = acc[0][a][i][b][e], up = acc[1][a][i][b][e];
          h[e] = gt / (1.0f + expf(-gt)) * up;
        }
        *(u32x2 *)(g.H + (size_t)(row0 + m) * g.ldh + j) = u32x2{pack2(h[0], h[1]), pack2(h[2], h[3])};
        if (kept_row >= 0) *(float4 *)(g.ret.ptr + (size_t)kept_row * g.N + j) = float4{h[0], h[1], h[2], h[3]};
      }
    } else {
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int a = 0; a < NH; ++a) {
          const int n = n0 + wn * (BN / 4) + j * (BN / 8) + 16 * a + 4 * gq;
          if (n >= g.N) continue;
          *(floatx4 *)(g.Y + split * g.y_stride + (size_t)(row0 + m) * g.ldy + n) = acc[j][a][i][b];
        }
    }
  }
}

}  // namespace

namespace {

struct TileShape {
  int bm, bn;
};

// Tile of an M x N output (every tile takes a compute unit of its own: 96 to
// 128 KB of LDS).  Cost: rounds of one workgroup per unit, weighted by what a
// round of the shape was measured to take per 64 reduction elements (us: 1.41
// for 256 x 256, 0.86 for 128 x 256, 0.60 for 128 x 128, whose 128-element
// steps keep twice the bytes in flight); a last round of few workgroups takes
// about 0.7 of a full one, since they share the caches with nobody.
TileShape tile_shape(int M, int N) {
  auto cost = [&](int bm, int bn, double c) {
    const int tiles = ((M + bm - 1) / bm) * ((N + bn - 1) / bn), full = tiles / kComputeUnits, rest = tiles % kComputeUnits;
    return c * (full + (rest ? 0.7 + 0.3 * rest / kComputeUnits : 0.0));
  };
  const double a = cost(256, 256, 1.41), b = cost(128, 256, 0.86), c = cost(128, 128, 0.6);
  if (a <= b && a <= c) return {256, 256};
  return b <= c ? TileShape{128, 256} : TileShape{128, 128};
}

}  // namespace

// Reduction splits of a plain projection: where the tiles fill a fraction of
// the compute units, the reduction is divided over the rest (at most four
// slabs for the row kernels to sum, at least eight 128-element steps each).
int gemm_tile_splits(int N, int K, int M) {
  const TileShape t = tile_shape(M, N);
  const int tiles = ((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn);
  return std::max(1, std::min({kComputeUnits / tiles, 4, K / 1024}));
}

bool gemm_tile_ok(int N, int K, int M, int dtype) {
  return dtype == 1 && M >= kTileRows && K % 128 == 0 && N % 16 == 0;
}

bool gemm_tile_args_ok(const TileGemm &g, bool glu) {
  if (!gemm_tile_ok(g.N, g.K, g.M, 1) || g.ldx % 8 != 0) return false;
  if (!glu && (g.rows[0] % 8 != 0 || g.rows[1] % 8 != 0 || g.rows[0] + g.rows[1] + g.rows[2] != g.N)) return false;
  // the QKV epilogue: heads of 128 dimensions, Q then K then V (as many V as K heads)
  if (g.rope && (g.kv.d_h != 128 || g.rows[0] % 128 != 0 || g.rows[1] != g.kv.n_kv * 128 || g.rows[2] != g.rows[1] ||
                 !g.Qout || !g.prompt || !g.kv.k || !g.kv.v || !g.kv.page_table))
    return false;
  // splits: plain outputs, at least one 128-element step each
  if (g.splits > 1 && (glu || g.rope || g.splits > g.K / 128)) return false;
  // 32-bit byte offsets
  return (long long)g.M * g.ldx < (1LL << 31) && (long long)g.N * g.K < (1LL << 31);
}

hipError_t launch_gemm_tile(const TileGemm &g, bool glu, hipStream_t st) {
  if (!gemm_tile_args_ok(g, glu)) return hipErrorInvalidValue;
  const TileShape t = tile_shape(g.M, glu ? 2 * g.N : g.N);
  auto go = [&](auto bm, auto bn, auto bk) {
    constexpr int BM = decltype(bm)::value, BN = decltype(bn)::value, BK = decltype(bk)::value;
    const int mt = (g.M + BM - 1) / BM, block = 512;
    if (glu)
      hipLaunchKernelGGL((k_gemm_tile<BM, BN, BK, EPI_GLU>), dim3((g.N + BN / 2 - 1) / (BN / 2), mt), dim3(block), 0, st, g);
    else if (g.rope)
      hipLaunchKernelGGL((k_gemm_tile<BM, BN, BK, EPI_QKV>), dim3((g.N + BN - 1) / BN, mt), dim3(block), 0, st, g);
    else
      hipLaunchKernelGGL((k_gemm_tile<BM, BN, BK, EPI_PLAIN>), dim3((g.N + BN - 1) / BN, mt, g.splits > 1 ? g.splits : 1),
                         dim3(block), 0, st, g);
  };
  using std::integral_constant;
  if (t.bm == 256)
    go(integral_constant<int, 256>{}, integral_constant<int, 256>{}, integral_constant<int, 64>{});
  else if (t.bn == 256)
    go(integral_constant<int, 128>{}, integral_constant<int, 256>{}, integral_constant<int, 64>{});
  else
    go(integral_constant<int, 128>{}, integral_constant<int, 128>{}, integral_constant<int, 128>{});
  return hipGetLastError();
}


bool gemm_tile_experts_ok(const TileGemm &g) {
  return g.K % 128 == 0 && g.N % 16 == 0 && g.ldx % 8 == 0 && g.tiles && g.ntiles && g.counts && g.offsets &&
         g.max_tiles > 0 && g.max_tiles <= 65535 && (long long)g.M * g.ldx < (1LL << 31) &&
         (long long)g.N * g.K < (1LL << 31);
}

hipError_t launch_gemm_tile_experts(const TileGemm &g, bool glu, hipStream_t st) {
  if (!gemm_tile_experts_ok(g)) return hipErrorInvalidValue;
  if (glu)
    hipLaunchKernelGGL((k_gemm_tile<128, 256, 64, EPI_GLU, true>), dim3((g.N + 127) / 128, g.max_tiles), dim3(512), 0, st, g);
  else
    hipLaunchKernelGGL((k_gemm_tile<128, 256, 64, EPI_PLAIN, true>), dim3((g.N + 255) / 256, g.max_tiles), dim3(512), 0, st, g);
  return hipGetLastError();
}

}  // namespace dbt
