// Scores of a bf16 unit by one work-group (Sec. 4.4, subset attention), and what they share with the scores of longer units: the parked
// format of the logits, row sums through LDS, the observation rows.  HIP device code only.
#pragma once

#include "device_util.h"
#include "hack_internal.h"

namespace hack {
namespace dev {

constexpr double kLog2e = 1.4426950408889634074;

// Logits are parked in registers between the two halves of the fused kernel as
// 32-bit fixed point, log2 units with 22 fractional bits: the quantisation moves
// 2^t by at most ln2 * 2^-23 = 8.3e-8 relative, and both the normaliser and the
// importance are formed from the same parked value.  |t| is clamped to 511
// (354 nats), far outside anything a float32 importance can resolve.
constexpr double kFixOne = 4194304.0;  // 2^22
constexpr int kFixLimit = 511 << 22;
__device__ __forceinline__ int fix_from(double t_scaled) {  // t_scaled = t * 2^22
  // the conversion saturates at the ends of the int range, far outside the clamp, so clamping the integer gives
  // what clamping the double first would (one three-operand median instead of two fp64 min / max)
  return min(max(__double2int_rn(t_scaled), -kFixLimit), kFixLimit);
}
// The same for a dot product well inside the clamp: adding 1.5 * 2^52 leaves the rounded integer in the low word.
__device__ __forceinline__ int fix_from_small(double dot, double c2) { return __double2loint(fma(dot, c2, 6755399441055744.0)); }
__device__ __forceinline__ double exp2_fix(int qv) {
  const float f = (float)(qv & 0x3FFFFF) * (float)(1.0 / kFixOne);  // [0, 1), exact
  const double m = (double)__builtin_amdgcn_exp2f(f);               // [1, 2]; the integer part goes to the exponent field
  return __hiloint2double(__double2hiint(m) + ((qv >> 22) << 20), __double2loint(m));
}
// Row sums of a wave, through 8 KiB of LDS: put_row leaves the value of register r (observation row c_row(r, half), column
// col) of every lane, take_rows returns the sum of row lane / 2 over the 32 columns.  256 bytes a row, the 16-byte chunk at
// position c holds columns 2 (c ^ row % 16) and the next: 16 writes and 8 reads without bank conflicts and
// 16 additions, where a shuffle tree for each of the 16 registers takes 240 vector instructions.  wave_lds_order() goes
// between the two, and before the buffer is written again.
__device__ __forceinline__ void put_row(char* buf, int r, int col, int half, double v) {
  const int row = c_row(r, half);
  *reinterpret_cast<double*>(buf + row * 256 + (((col >> 1) ^ (row & 15)) << 4) + (col & 1) * 8) = v;
}
__device__ __forceinline__ double take_rows(const char* buf, int lane) {
  const int row = lane >> 1;
  double s = 0.0;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const double2 x = *reinterpret_cast<const double2*>(buf + row * 256 + ((((lane & 1) * 8 + j) ^ (row & 15)) << 4));
    s += x.x;
    s += x.y;
  }
  return s + dpp_mov_f64<0xB1>(s);
}
// The observation rows of a unit on their way into LDS, in the layout of a tile of keys, shared out over the waves of a work-group.  Rows past
// n_obs repeat the first one; they get weight zero.  (Read straight from memory into the operand registers of every wave, 32 rows x
// 32 bytes an instruction, they kept the memory pipeline of a compute unit busy for 2000 cycles a work-group, against some 60 this way, and
// a row number loaded behind the first tile's copies was waited for with them.  Kernel trace, us a launch: 32 units of 2500 / 4000 / 6000 / 8000 keys, D = 128
// 11.0 / 16.0 / 19.8 / 20.6 -> 10.3 / 15.3 / 18.6 / 19.8; 480 units of 358 keys and 480 of 562, D = 64 18.6 + 38.5 -> 16.8 + 36.0.)
template <int D, int WAVES>
struct ObsRows {
  static constexpr int CPR = D / 8, RPI = 64 / CPR, COPIES = 32 / RPI, PER = (COPIES + WAVES - 1) / WAVES;
  int row[PER];
  // in front of every hand-issued copy: the compiler's wait for these loads counts none of them
  __device__ __forceinline__ void load(const int32_t* __restrict__ q_rows, int n_obs, int w, int lane) {
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      const int r = (w + p * WAVES) * RPI + lane / CPR;
      row[p] = q_rows[r < n_obs ? r : 0];
    }
#pragma unroll
    for (int p = 0; p < PER; ++p) asm volatile("" ::"v"(row[p]));
  }
  __device__ __forceinline__ void issue(const __bf16* q_unit, unsigned lds, int w, int lane) const {
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      const int i = w + p * WAVES, r = i * RPI + lane / CPR;
      if (COPIES % WAVES == 0 || i < COPIES)
        load_to_lds(q_unit + (int64_t)row[p] * D + (((lane % CPR) ^ swz_k<D>(r)) & (CPR - 1)) * 8, lds + (unsigned)(i * 1024));
    }
  }
};

// Importance of the keys of unit d by a work-group of NW waves, at most 32 TILES NW keys: keys[j] gets the float bits of key j's.  Wave w takes the
// tiles w, w + NW, ...; the row sums meet in LDS.  The numbers are those of score_fused up to the order in which the row sums are
// added in fp64.  bufs, red, inv_s, q_lds: LDS, q_lds 32 rows; keys is ready behind the caller's next barrier, bufs is free from there on.
template <int D, int NW, int TILES>
__device__ __forceinline__ void score_unit(const UnitDesc& d, const __bf16* __restrict__ q, const int32_t* __restrict__ q_rows, int n_obs, int N_k,
                                           float scale, const __bf16* __restrict__ k_cache, const __bf16* __restrict__ k_new, char (*bufs)[8192],
                                           double (*red)[kMaxObs], double (*inv_s)[kMaxObs], uint32_t* keys, __bf16* q_lds,
                                           int* __restrict__ fault) {
  constexpr int KK = D / 16, CPR = D / 8, RPI = 64 / CPR, IPT = 32 / RPI, TILE = 32 * D;   // as in score_fused
  constexpr int kBufs = 8192 / (TILE * 2);   // tile buffers per wave: the row sums need 8 KiB
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  ObsRows<D, NW> obs;
  obs.load(q_rows, n_obs, w, lane);
  const int col = lane & 31, half = lane >> 5;
  const int T_in = d.len_in + d.n_new;
  const int n_tiles = w * 32 >= T_in ? 0 : min(TILES, (T_in - w * 32 + 32 * NW - 1) / (32 * NW));   // of this wave
  const unsigned lds0 = lds_addr_of(&bufs[w][0]);

  int src_off[IPT];
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const int r = i * RPI + lane / CPR, c = lane % CPR;
    src_off[i] = (r * D + ((c ^ swz_k<D>(r)) & (CPR - 1)) * 8) * 2;
  }
  auto issue = [&](int t) {
    const int j0 = (w + t * NW) * 32;
    const unsigned dst = lds0 + (unsigned)((t % kBufs) * TILE * 2);
    const bool in_cache = j0 + 32 <= d.len_in;
    const bool in_new = j0 >= d.len_in && j0 + 32 <= T_in;
    if (in_cache || in_new) {
      const __bf16* base = in_cache ? k_cache + (d.in_off + j0) * D : k_new + ((int64_t)d.unit * N_k + (j0 - d.len_in)) * D;
#pragma unroll
      for (int i = 0; i < IPT; ++i) load_to_lds(base, (unsigned)src_off[i], dst + i * 1024);
    } else {   // rows past the end repeat the last key
#pragma unroll
      for (int i = 0; i < IPT; ++i) {
        const int r = i * RPI + lane / CPR, c = lane % CPR;
        const int j = min(j0 + r, T_in - 1);
        const __bf16* row = (j < d.len_in) ? k_cache + (d.in_off + j) * D : k_new + ((int64_t)d.unit * N_k + (j - d.len_in)) * D;
        load_to_lds(row + ((c ^ swz_k<D>(r)) & (CPR - 1)) * 8, dst + i * 1024);
      }
    }
  };
  obs.issue(q + (int64_t)d.unit * N_k * D, lds_addr_of(q_lds), w, lane);
  if (n_tiles > 0) issue(0);
  constexpr bool kBoth = TILES > 1 && kBufs > 1;   // both tiles of a wave are copied at once
  if (kBoth && n_tiles > 1) issue(1);

  const double c2 = (double)scale * kLog2e * kFixOne;
  const double dot_safe = (double)(kFixLimit - 1) / c2;
  int k_off[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) k_off[kk] = col * D + (((2 * kk + half) ^ swz_k<D>(col)) & (CPR - 1)) * 8;
  // Q~ has landed, the tiles may still be on their way
  if (kBoth && n_tiles > 1) dma_wait_but<2 * IPT>();
  else if (n_tiles > 0) dma_wait_but<IPT>();
  else dma_wait_but<0>();
  __syncthreads();
  bf16x8 qf[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) qf[kk] = *reinterpret_cast<const bf16x8*>(&q_lds[k_off[kk]]);

  // ---- logits (see score_fused) ----
  double pq[TILES][16];
  bool clamped = false;
#pragma unroll
  for (int t = 0; t < TILES; ++t) {
    if (t < n_tiles) {                 // wave-uniform
      if (kBufs > 1 && t + 1 < TILES && t + 1 < n_tiles) dma_wait_but<IPT>();
      else dma_wait_but<0>();
      const __bf16* Kt = reinterpret_cast<const __bf16*>(&bufs[w][(t % kBufs) * TILE * 2]);
      double sd[16];
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        const bf16x8 kf = *reinterpret_cast<const bf16x8*>(&Kt[k_off[kk]]);
        floatx16 c = {0};
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[kk], kf, c, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 16; ++r) sd[r] = (kk == 0) ? (double)c[r] : sd[r] + (double)c[r];
      }
      if (t + kBufs < TILES && t + kBufs < n_tiles) {
        // the sums above have consumed every operand read: the buffer may be refilled
#pragma unroll
        for (int r = 0; r < 16; ++r) asm volatile("" : "+v"(sd[r]) : : "memory");
        issue(t + kBufs);
      }
      double top = 0.0;
#pragma unroll
      for (int r = 0; r < 16; ++r) top = fmax(top, fabs(sd[r]));
      int qv[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) qv[r] = fix_from_small(sd[r], c2);
      if (__any(!(top < dot_safe))) {  // rare
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          qv[r] = fix_from(sd[r] * c2);
          clamped |= qv[r] >= kFixLimit || qv[r] <= -kFixLimit;
        }
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) pq[t][r] = exp2_fix(qv[r]);
    } else {
#pragma unroll
      for (int r = 0; r < 16; ++r) pq[t][r] = 0.0;
    }
  }
  if (__any(clamped)) {
    if (lane == 0) __hip_atomic_store(fault + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }

  // ---- normalisers ----
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    double lsum = 0.0;
#pragma unroll
    for (int t = 0; t < TILES; ++t)
      if (t < n_tiles && (w + t * NW) * 32 + col < T_in) lsum += pq[t][r];
    put_row(&bufs[w][0], r, col, half, lsum);
  }
  wave_lds_order();
  const double l = take_rows(&bufs[w][0], lane);
  if ((lane & 1) == 0) red[w][lane >> 1] = l;
  __syncthreads();                     // tile buffers are free from here on
  if (lane < kMaxObs) {
    double tot = 0.0;
#pragma unroll
    for (int k = 0; k < NW; ++k) tot += red[k][lane];
    inv_s[w][lane] = (lane < n_obs) ? 1.0 / tot : 0.0;
  }
  wave_lds_order();
  double inv_r[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) inv_r[r] = inv_s[w][c_row(r, half)];
#pragma unroll
  for (int t = 0; t < TILES; ++t) {
    if (t < n_tiles) {
      double imp = 0.0;
#pragma unroll
      for (int r = 0; r < 16; ++r) imp = fma(pq[t][r], inv_r[r], imp);
      imp += shfl_xor_f64(imp, 32);
      if (half == 0) keys[(w + t * NW) * 32 + col] = __float_as_uint((float)imp);
    }
  }
}

}  // namespace dev
}  // namespace hack
