// One 32-key block of attention by a wave that takes the blocks w, w + splits, ... of a unit's keys for NQ tiles of 16 queries: S^T = K Q^T and
// O^T += V^T P^T in 16x16x32 matrix instructions, row sums one more tile of the latter, against ones.  K and V blocks lie in LDS in the layouts of
// swz_k and swz_v16.  Shared by the key-split kernel and by whole steps; HIP device code only.
#pragma once

#include <cfloat>

#include "device_util.h"

namespace hack {
namespace dev {

template <int D, int NQ>
struct SplitStage {
  static constexpr int KC = D / 32;    // MFMA steps over head_dim for S^T
  static constexpr int MT = D / 16;    // 16-row tiles of O^T
  static constexpr int CPR = D / 8;    // 16-byte chunks per row

  int col, g;            // of the lane: query column, row group
  float c2;              // log2 e times the scale
  int k_off[KC];         // K operand: row 16 kt + col, chunk 4 c + g
  int v_off[MT];         // V^T operand: rows 4 g + e and 16 + 4 g + e, head-dim 16 mt + 4 qd
  bf16x8 ones;
  floatx4 o[MT][NQ];     // O^T: head-dim 16 mt + 4 g + r, query 16 qt + col
  floatx4 ls[NQ];        // row sums of P: all four rows hold the same
  float mc[NQ];          // probabilities are 2^(c2 s - mc); finite from the start, so that keys whose score is -inf get 0

  __device__ __forceinline__ void init(float scale, int lane) {
    col = lane & 15;
    g = lane >> 4;
    c2 = scale * kLog2eF;
#pragma unroll
    for (int c = 0; c < KC; ++c) k_off[c] = col * D + (((4 * c + g) ^ swz_k<D>(col)) & (CPR - 1)) * 8;
    const int e = col >> 2, qd = col & 3;
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
      v_off[mt] = (4 * g + e) * D + (((2 * mt + (qd >> 1)) ^ swz_v16<D>(4 * g + e)) & (CPR - 1)) * 8 + 4 * (qd & 1);
#pragma unroll
    for (int j = 0; j < 8; ++j) ones[j] = (__bf16)1.0f;
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) o[mt][qt] = floatx4{0.f, 0.f, 0.f, 0.f};
      ls[qt] = floatx4{0.f, 0.f, 0.f, 0.f};
      mc[qt] = -FLT_MAX;
    }
  }

  // Scores of a block: sc[kt][qt], keys 16 kt + 4 g + r, query 16 qt + col.
  __device__ __forceinline__ void scores(const __bf16* Kt, const bf16x8 (&qf)[NQ][KC], floatx4 (&sc)[2][NQ]) const {
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int qt = 0; qt < NQ; ++qt) sc[kt][qt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < KC; ++c)
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        const bf16x8 kf = *reinterpret_cast<const bf16x8*>(&Kt[16 * kt * D + k_off[c]]);
#pragma unroll
        for (int qt = 0; qt < NQ; ++qt) sc[kt][qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[qt][c], sc[kt][qt], 0, 0, 0);
      }
  }
  // keys past the end, of total
  __device__ __forceinline__ void mask(floatx4 (&sc)[2][NQ], int b, int total) const {
    if ((b + 1) * 32 > total) {
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (b * 32 + 16 * kt + 4 * g + r >= total) {
#pragma unroll
            for (int qt = 0; qt < NQ; ++qt) sc[kt][qt][r] = -INFINITY;
          }
    }
  }
  // The reference is the largest score so far; what has been summed against the old one is brought to the new one.  A reference ahead of the
  // first block's scores, moved only when a probability outgrows it, spares most of this (200 random launches 0.987 of the time, 256^2 schedules the
  // same, odd sides 0.98), but the largest probabilities then lie anywhere between two powers of two instead of just below one, where bf16 rounds
  // them finest: 1.04 times the error against float64 over 128 to 300 keys, 1.1 (up to 1.2) over more.
  __device__ __forceinline__ void follow(const floatx4 (&sc)[2][NQ], bool nothing_yet) {
    float m_new[NQ];
    bool moved = false;
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) {
      float mx = sc[0][qt][0];
#pragma unroll
      for (int j = 1; j < 8; ++j) mx = maximum(mx, sc[j >> 2][qt][j & 3]);
      m_new[qt] = maximum(mc[qt], quad_maximum(mx) * c2);
      moved |= m_new[qt] != mc[qt];
    }
    if (!nothing_yet && __any(moved)) {
#pragma unroll
      for (int qt = 0; qt < NQ; ++qt) {
        const float a = __builtin_amdgcn_exp2f(mc[qt] - m_new[qt]);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          ls[qt][r] *= a;
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) o[mt][qt][r] *= a;
        }
      }
    }
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) mc[qt] = m_new[qt];
  }
  // Probabilities of a block in the order of the B operand of the PV product: element j of lane group g is key 4 g + j (j < 4) or
  // 16 + 4 g + j - 4, and the V^T operand is read in the same order.
  __device__ __forceinline__ void probs(const floatx4 (&sc)[2][NQ], bf16x8 (&pf)[NQ]) const {
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt)
#pragma unroll
      for (int j = 0; j < 8; ++j) pf[qt][j] = (__bf16)__builtin_amdgcn_exp2f(fmaf(sc[j >> 2][qt][j & 3], c2, -mc[qt]));
  }
  __device__ __forceinline__ void row_sums(const bf16x8 (&pf)[NQ]) {   // over the rounded probabilities, the numbers the PV product uses
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) ls[qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pf[qt], ls[qt], 0, 0, 0);
  }
  __device__ __forceinline__ void pv(const __bf16* Vt, const bf16x8 (&pf)[NQ], int mt) {
    const bf16x4 v0 = lds_read_tr(&Vt[v_off[mt]]), v1 = lds_read_tr(&Vt[16 * D + v_off[mt]]);
    const bf16x8 vf = {v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) o[mt][qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pf[qt], o[mt][qt], 0, 0, 0);
  }
  // Four values of a query's output row, `row`: head-dim 16 mt + 4 g + r.
  __device__ __forceinline__ void store(__bf16* row, int mt, const floatx4& x, float inv) const {
    *reinterpret_cast<bf16x4*>(row + 16 * mt + 4 * g) = bf16x4{(__bf16)(x[0] * inv), (__bf16)(x[1] * inv), (__bf16)(x[2] * inv), (__bf16)(x[3] * inv)};
  }
};

}  // namespace dev
}  // namespace hack
