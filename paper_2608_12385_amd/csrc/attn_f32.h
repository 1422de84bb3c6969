// Attention over an fp32 paged cache on the fp32 matrix instruction
// (v_mfma_f32_16x16x4_f32), shared by the decode and the prompt kernel:
// sixteen query rows against a range of pages, the pages dealt to the
// workgroup's waves, one online softmax per wave, merged through LDS.
//
// One page (16 keys) per turn.  Scores S = K Q^T: lane (r, gq) reads dimensions
// 4 gq .. 4 gq + 3 of each 16-dimension piece of key r, and the j-th of a piece's
// four multiplies takes dimension 4 gq + j of both operands, so the lane ends
// with the scores of keys 4 gq .. 4 gq + 3 for query r.  Those are the operand
// of the value sum O^T = V^T P^T when its j-th multiply takes key 4 gq + j of
// every group: V pages are dimension-major, so lane (r, gq) reads the four keys
// of dimension 16 c + r as one float4.  No operand passes through LDS.
//
// Keys and values may be infinite or not a number: a key that a row does not
// see (after its position, stale, or of another row) leaves no trace in it,
// and one that it sees does, whichever wave reads its page.
#pragma once
#include "common.h"

namespace dbt {

constexpr int kWavesF32Attn = 8;

// The waves' partial results: O^T of 16 NC dimensions, maximum (base 2) and sum.
template <int NC>
struct F32Merge {
  float o[kWavesF32Attn][16 * NC][17];
  float m[kWavesF32Attn][16], l[kWavesF32Attn][16];
  // the sums of query row qr over all waves, relative to their maximum mx
  // (a wave without keys has sums of zero; one whose scores were all NaN has no
  // maximum either, but its sums are NaN and count)
  __device__ __forceinline__ void merged(int qr, int dh, float &os, float &ls, float &mx) const {
    mx = kNoScore;
#pragma unroll
    for (int w = 0; w < kWavesF32Attn; ++w) mx = fmaxf(mx, m[w][qr]);
    os = ls = 0.f;
#pragma unroll
    for (int w = 0; w < kWavesF32Attn; ++w) {
      const float f = exp2f(m[w][qr] - mx);
      os += o[w][dh][qr] * f;
      ls += l[w][qr] * f;
    }
  }
};

// qp: this lane's query row (row r = lane & 15; live = false: a stand-in whose
// results are not used); it sees keys 0 .. seen - 1.  Pages [pb, pe) of ptab;
// positions >= valid hold no key (stale slots).  CAUSAL: rows see different
// numbers of keys, but all of those before the last page.  Ends with a barrier.
template <int NC, bool CAUSAL>
__device__ __forceinline__ void attn_f32(F32Merge<NC> &mg, const float *qp, bool live, int seen, int valid,
                                         const float *kbase, const float *vbase, const int *ptab, int pb, int pe,
                                         int n_kv, int g, int DH) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, gq = lane >> 4;
  const float scale = kLog2e / sqrtf((float)DH);
  // dimensions past DH (DH is a multiple of 4) re-read dimension 0 of the
  // row: zero in the query, and not stored in the output
  int koff[NC], voff[NC];
  floatx4 q[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int d0 = 16 * c + 4 * gq, dv = 16 * c + r;
    koff[c] = r * DH + (d0 < DH ? d0 : 0);
    voff[c] = (dv < DH ? dv : 0) * 16 + 4 * gq;
    q[c] = *(const floatx4 *)(qp + (d0 < DH ? d0 : 0));
    if (d0 >= DH || !live) q[c] = floatx4{0.f, 0.f, 0.f, 0.f};
  }
  float m_run = kNoScore, l_run = 0.f;
  floatx4 acc[NC], k[NC], v[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) acc[c] = floatx4{0.f, 0.f, 0.f, 0.f};
  auto load = [&](int id) {
    const size_t blk = ((size_t)id * n_kv + g) * 16 * DH;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      k[c] = *(const floatx4 *)(kbase + blk + koff[c]);
      v[c] = *(const floatx4 *)(vbase + blk + voff[c]);
    }
  };
  int j = pb + wave;
  int next = j + kWavesF32Attn < pe ? ptab[j + kWavesF32Attn] : 0;  // page ids run one turn further ahead
  if (j < pe) load(ptab[j]);
  float p[4] = {0.f, 0.f, 0.f, 0.f};
  bool apart = false;  // the last page holds values that are not finite (CAUSAL)
  for (; j < pe; j += kWavesF32Attn) {
    floatx4 s = {0.f, 0.f, 0.f, 0.f};
    if (16 * NC > DH && 16 * (NC - 1) + 4 * gq >= DH) k[NC - 1] = floatx4{0.f, 0.f, 0.f, 0.f};  // (infinity * 0)
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int i = 0; i < 4; ++i) s = __builtin_amdgcn_mfma_f32_16x16x4f32(k[c][i], q[c][i], s, 0, 0, 0);
    floatx4 vc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) vc[c] = v[c];
    const int id = next;
    if (j + 2 * kWavesF32Attn < pe) next = ptab[j + 2 * kWavesF32Attn];
    if (j + kWavesF32Attn < pe) load(id);
    const int p0 = 16 * j + 4 * gq;  // position of this lane's first score
    float mt = -INFINITY;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      s[i] = p0 + i < seen ? s[i] * scale : -INFINITY;
      mt = fmaxf(mt, s[i]);
    }
    const float m_new = fmaxf(m_run, rows4_max(mt));
    const float corr = exp2f(m_run - m_new);
    l_run *= corr;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      p[i] = exp2f(s[i] - m_new);
      l_run += p[i];
    }
    m_run = m_new;
    if (16 * j + 16 > valid) {  // stale slots may hold anything: 0 * NaN
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (p0 + i >= valid) vc[c][i] = 0.f;
    }
    if (CAUSAL && j == pe - 1) {
      // the page of the tile's own positions: a probability of zero would not
      // hide a value that is not finite from the rows before it, so such
      // values are taken out here and added below
      bool odd = false;
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (!(fabsf(vc[c][i]) < INFINITY)) {
            vc[c][i] = 0.f;
            odd = true;
          }
      apart = __any(odd);
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      acc[c] = acc[c] * corr;
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(vc[c][i], p[i], acc[c], 0, 0, 0);
    }
  }
  if (CAUSAL && apart) {  // row by row, the keys it sees
    const int p0 = 16 * (pe - 1) + 4 * gq;
    const float *vp = vbase + ((size_t)ptab[pe - 1] * n_kv + g) * 16 * DH;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const floatx4 w = *(const floatx4 *)(vp + voff[c]);
#pragma unroll 1
      for (int row = 0; row < 16; ++row) {
        const int see = min(__shfl(seen, row, 64), valid);
        floatx4 o = acc[c];
#pragma unroll
        for (int i = 0; i < 4; ++i)
          o = __builtin_amdgcn_mfma_f32_16x16x4f32(p0 + i < see && !(fabsf(w[i]) < INFINITY) ? w[i] : 0.f, p[i], o, 0, 0, 0);
        if (r == row) acc[c] = o;
      }
    }
  }
  l_run += __shfl_xor(l_run, 16, 64);
  l_run += __shfl_xor(l_run, 32, 64);
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int i = 0; i < 4; ++i) mg.o[wave][16 * c + 4 * gq + i][r] = acc[c][i];
  if (gq == 0) {
    mg.m[wave][r] = m_run;
    mg.l[wave][r] = l_run;
  }
  __syncthreads();
}

}  // namespace dbt
