// Budgeted selection (Sec. 4.4, f_C and f_S) on gfx950.
//
// One work-group per unit.  The host has already turned (head class, budget,
// N_init, N_k) into: rows [0, keep_a) and [keep_b, T) kept unconditionally and
// the sel_m most important rows of the ranked segment [sel_lo, sel_hi).
// The ranked segment is resolved by a radix select over order-preserving uint32
// keys; an index-ordered prefix scan then emits the kept rows in ascending order,
// taking rows equal to the threshold with the lowest indices first.
//
// What bounds a launch is the chain of barriers and LDS round trips of one
// work-group (32 to 1000 work-groups, 24 KB of keys each), so the chain is kept
// short:
//   * a thread holds PER consecutive keys in registers from the one load to the
//     emission; LDS carries histograms and wave totals only;
//   * the first digit covers sign, exponent and the leading mantissa bits (12 bits;
//     11 for short units): importance values of a unit spread over some fifty such
//     bins, so the histogram's atomics rarely meet on an address, and a few hundred
//     keys are left; the second digit leaves one key as a rule, and the passes end
//     as soon as the bin of the threshold is taken whole;
//   * all histograms are cleared together while the keys are on their way; a pass
//     has three barriers (counted, totals of the waves, bin found).
// Measured, us a launch with its gap in a graph, this form / the one it replaces (four
// 8-bit digits over keys in LDS): 32 units of 1500, 4000, 6039, 7981 keys 4.8 / 7.4,
// 5.9 / 10.4, 7.2 / 13.1, 7.9 / 16.0; 60 and 960 units of 356 keys 4.3 / 6.5, 6.1 / 7.5.
// More threads with fewer keys each won throughout (4000 keys: 256, 512, 1024 threads
// 8.1, 6.4, 5.9; 560 keys, 60 / 960 units: 128 threads 6.1 / 9.8, 256 4.5 / 7.0, 512 3.9 / 6.4,
// 1024 4.1 / 9.2, the last for want of resident work-groups).
#include <type_traits>

#include "hack_internal.h"

namespace hack {

namespace {

__device__ __forceinline__ uint32_t orderable(float f) {
  uint32_t u = __float_as_uint(f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Inclusive prefix over the wave: four shifts inside the 16-lane rows, then the row totals handed on.
__device__ __forceinline__ int wave_inclusive_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);   // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);   // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);   // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);   // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);   // lane 15 of rows 0, 2 -> rows 1, 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);   // lane 31 -> rows 2, 3
  return v;
}

// Exclusive prefix of v over the work-group in thread order.  wave_tot is used by this call only (one barrier).
template <int kWaves>
__device__ __forceinline__ int block_exclusive_scan(int v, int* wave_tot) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int incl = wave_inclusive_scan(v);
  if (lane == 63) wave_tot[w] = incl;
  __syncthreads();
  int base = 0;
#pragma unroll
  for (int i = 0; i < kWaves; ++i) {
    const int t = wave_tot[i];
    if (i < w) base += t;
  }
  return base + incl - v;
}

// NT threads, PER keys each (T <= NT * PER); digits of B0, B1 and 32 - B0 - B1 bits.
template <int NT, int PER, int B0, int B1>
__global__ __launch_bounds__(NT) void select_kernel(
    const UnitDesc* __restrict__ descs, const int32_t* __restrict__ list,
    const float* __restrict__ importance, int64_t imp_stride, int32_t* __restrict__ kept_idx,
    int64_t idx_stride, int32_t* __restrict__ seam) {
  constexpr int kWaves = NT / 64;
  constexpr int B2 = 32 - B0 - B1;
  constexpr int kHist = (1 << B0) + (1 << B1) + (1 << B2);
  __shared__ __attribute__((aligned(16))) uint32_t hist[kHist];
  __shared__ int wave_tot[5][kWaves];
  __shared__ int found[3][3];   // per pass: bin, rows still wanted from it, keys in it

  const UnitDesc d = descs[list[blockIdx.x]];
  const float* imp = importance + (int64_t)d.unit * imp_stride;
  int32_t* out = kept_idx + (int64_t)d.unit * idx_stride;
  const int T = d.len_in + d.n_new;
  const int tid = threadIdx.x;
  const int j0 = tid * PER;                   // first row of this thread

  const bool take_all = (d.sel_m >= d.sel_hi - d.sel_lo);
  const bool take_none = (d.sel_m <= 0);
  const bool ranked = !take_all && !take_none;

  uint32_t key[PER];
  unsigned in_seg = 0;                        // bit e: row j0 + e is in the ranked segment
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    key[e] = 0;
    if (j0 + e >= d.sel_lo && j0 + e < d.sel_hi) in_seg |= 1u << e;
  }
  if (ranked && in_seg) {
    // a whole piece of four stays inside the unit's row (j0 < T <= imp_stride, both multiples of four)
    const bool vec = PER % 4 == 0 && (imp_stride & 3) == 0 && ((uintptr_t)importance & 15) == 0;
    if (vec) {
#pragma unroll
      for (int e4 = 0; e4 < PER / 4; ++e4) {
        if ((in_seg >> (4 * e4)) & 15u) {
          const float4 x = *reinterpret_cast<const float4*>(imp + j0 + 4 * e4);
          key[4 * e4] = __float_as_uint(x.x);
          key[4 * e4 + 1] = __float_as_uint(x.y);
          key[4 * e4 + 2] = __float_as_uint(x.z);
          key[4 * e4 + 3] = __float_as_uint(x.w);
        }
      }
    } else {
#pragma unroll
      for (int e = 0; e < PER; ++e)
        if ((in_seg >> e) & 1u) key[e] = __float_as_uint(imp[j0 + e]);
    }
  }

  // ---- threshold of the ranked segment ----
  uint32_t pre = 0;     // keys with (key >> shift) > pre are kept, those equal to pre are candidates
  int shift = 0;
  int want = d.sel_m;   // candidates to keep
  bool all_candidates = true;
  if (ranked) {
    for (int i = tid * 4; i < kHist; i += NT * 4) *reinterpret_cast<uint4*>(&hist[i]) = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
    for (int e = 0; e < PER; ++e) key[e] = orderable(__uint_as_float(key[e]));
    __syncthreads();
    // One pass over a digit of BITS bits at bit SH; bins in descending order of the digit.
    auto pass = [&](auto idx_tag, auto bits_tag, auto sh_tag, uint32_t* h) {
      constexpr int P = decltype(idx_tag)::value, BITS = decltype(bits_tag)::value, SH = decltype(sh_tag)::value;
      constexpr uint32_t M = (1u << BITS) - 1u;
      constexpr int BPT = (1 << BITS) / NT > 0 ? (1 << BITS) / NT : 1;   // bins per thread
#pragma unroll
      for (int e = 0; e < PER; ++e)
        if (((in_seg >> e) & 1u) && (P == 0 || (key[e] >> ((SH + BITS) & 31)) == pre))
          atomicAdd(&h[(~(key[e] >> SH)) & M], 1u);
      __syncthreads();
      int c[BPT], tot = 0;
#pragma unroll
      for (int b = 0; b < BPT; ++b) {
        c[b] = tid * BPT + b < (1 << BITS) ? (int)h[tid * BPT + b] : 0;
        tot += c[b];
      }
      int run = block_exclusive_scan<kWaves>(tot, wave_tot[P]);
      if (run < want && want <= run + tot) {
#pragma unroll
        for (int b = 0; b < BPT; ++b) {
          if (run < want && want <= run + c[b]) {
            found[P][0] = tid * BPT + b;
            found[P][1] = want - run;
            found[P][2] = c[b];
          }
          run += c[b];
        }
      }
      __syncthreads();
      pre = (P == 0 ? 0u : pre << BITS) | (M - (uint32_t)found[P][0]);
      shift = SH;
      want = found[P][1];
      return want == found[P][2];   // the whole bin is kept
    };
    using std::integral_constant;
    all_candidates = pass(integral_constant<int, 0>{}, integral_constant<int, B0>{}, integral_constant<int, 32 - B0>{}, hist) ||
                     pass(integral_constant<int, 1>{}, integral_constant<int, B1>{}, integral_constant<int, B2>{}, hist + (1 << B0)) ||
                     pass(integral_constant<int, 2>{}, integral_constant<int, B2>{}, integral_constant<int, 0>{},
                          hist + (1 << B0) + (1 << B1));
  }

  // ---- ordered emission ----
  // forced rows, rows above the threshold and, as a rule, all candidates; if some equal rows are left out (only
  // whole keys are equal then), the lowest rows are taken
  unsigned keep = 0, cand = 0;
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const int j = j0 + e;
    const bool forced = j < d.keep_a || j >= d.keep_b;
    const bool seg = (in_seg >> e) & 1u;
    const uint32_t v = key[e] >> shift;
    const bool hit = forced || (seg && (take_all || (ranked && v > pre)));
    if (j < T && hit) keep |= 1u << e;
    if (seg && !forced && ranked && v == pre) cand |= 1u << e;
  }
  if (all_candidates) {
    keep |= cand;
  } else {
    int left = want - block_exclusive_scan<kWaves>(__popc(cand), wave_tot[3]);   // how many of this thread's candidates may stay
#pragma unroll
    for (int e = 0; e < PER; ++e)
      if (((cand >> e) & 1u) && left > 0) {
        keep |= 1u << e;
        --left;
      }
  }
  int pos = block_exclusive_scan<kWaves>(__popc(keep), wave_tot[4]);
  // how many kept rows precede row len_in, the first new one
  if (seam != nullptr && d.len_in >= j0 && d.len_in < j0 + PER) seam[d.unit] = pos + __popc(keep & ((1u << (d.len_in - j0)) - 1u));
#pragma unroll
  for (int e = 0; e < PER; ++e)
    if ((keep >> e) & 1u) out[pos++] = j0 + e;
}

}  // namespace

void launch_select(hipStream_t s, const UnitDesc* descs, const int32_t* list, int n_list,
                   int max_t_in, const float* importance, int64_t imp_stride, int32_t* kept_idx,
                   int64_t idx_stride, int32_t* seam) {
  if (n_list <= 0) return;
#define HACK_SELECT(NT_, PER_, B0_, B1_)                                                                                      \
  hipLaunchKernelGGL((select_kernel<NT_, PER_, B0_, B1_>), dim3(n_list), dim3(NT_), 0, s, descs, list, importance, imp_stride, \
                     kept_idx, idx_stride, seam)
  if (max_t_in <= 1024) HACK_SELECT(512, 2, 11, 11);
  else if (max_t_in <= 2048) HACK_SELECT(1024, 2, 12, 10);
  else if (max_t_in <= 4096) HACK_SELECT(1024, 4, 12, 10);
  else if (max_t_in <= 8192) HACK_SELECT(1024, 8, 12, 10);
  else if (max_t_in <= 16384) HACK_SELECT(1024, 16, 12, 10);
  else HACK_SELECT(1024, 32, 12, 10);
#undef HACK_SELECT
}

}  // namespace hack
