// The ranking half of the selection (Sec. 4.4, f_C and f_S), shared by the kernel that reads importance from memory and
// the one that has just formed it.  HIP device code only.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "hack_internal.h"

namespace hack {
namespace dev {

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

template <int NT, int B0, int B1>
struct SelectShared {
  static constexpr int kHist = (1 << B0) + (1 << B1) + (1 << (32 - B0 - B1));
  int wave_tot[5][NT / 64];
  int found[3][3];   // per pass: bin, rows still wanted from it, keys in it
};

template <int NT, int B0, int B1>
__device__ __forceinline__ void clear_hist(uint32_t* hist, int tid) {
  for (int i = tid * 4; i < SelectShared<NT, B0, B1>::kHist; i += NT * 4) *reinterpret_cast<uint4*>(&hist[i]) = make_uint4(0u, 0u, 0u, 0u);
}

// The work-group (NT threads) writes the kept rows of d to out (or NULL) in ascending order.  Thread tid holds the keys of the PER
// rows from tid * PER on: float bits where in_seg says that the row is ranked.  Digits of B0, B1 and 32 - B0 - B1 bits;
// hist: SelectShared::kHist words of LDS, 16-byte aligned, cleared in here unless the caller has done so in front of a barrier (CLEARED); kept_lds, if given, gets the list as well (words nobody reads any more once a barrier
// has been passed).
template <int NT, int PER, int B0, int B1, bool CLEARED = false>
__device__ __forceinline__ void select_rows(const UnitDesc& d, uint32_t (&key)[PER], unsigned in_seg, uint32_t* hist,
                                            SelectShared<NT, B0, B1>& sh, int32_t* __restrict__ out, int32_t* __restrict__ seam,
                                            uint32_t* kept_lds = nullptr) {
  constexpr int kWaves = NT / 64;
  constexpr int B2 = 32 - B0 - B1;
  auto& wave_tot = sh.wave_tot;
  auto& found = sh.found;
  const int T = d.len_in + d.n_new;
  const int tid = threadIdx.x;
  const int j0 = tid * PER;                   // first row of this thread
  const bool take_all = (d.sel_m >= d.sel_hi - d.sel_lo);
  const bool ranked = !take_all && d.sel_m > 0;

  // ---- threshold of the ranked segment ----
  uint32_t pre = 0;     // keys with (key >> shift) > pre are kept, those equal to pre are candidates
  int shift = 0;
  int want = d.sel_m;   // candidates to keep
  bool all_candidates = true;
  if (ranked) {
    if (!CLEARED) clear_hist<NT, B0, B1>(hist, tid);
#pragma unroll
    for (int e = 0; e < PER; ++e) key[e] = orderable(__uint_as_float(key[e]));
    if (!CLEARED) __syncthreads();
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
    if ((keep >> e) & 1u) {
      if (kept_lds != nullptr) kept_lds[pos] = (uint32_t)(j0 + e);
      if (out != nullptr) out[pos] = j0 + e;
      ++pos;
    }
}

}  // namespace dev
}  // namespace hack
