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
// Keys are dealt as evenly as their number allows: 6 a thread up to 6144 keys and 12 up to 12288 instead of 8 and 16 (4186, 5000, 6039 keys
// 6.9 / 6.3, 6.8 / 6.3, 7.0 / 6.6 us; 8831, 9500, 10521 11.0 / 9.3, 11.9 / 10.2, 10.5 / 8.9).
#include "hack_internal.h"
#include "select_device.h"

namespace hack {

namespace {

using namespace dev;

// NT threads, PER keys each (T <= NT * PER); digits of B0, B1 and 32 - B0 - B1 bits.
template <int NT, int PER, int B0, int B1>
__global__ __launch_bounds__(NT) void select_kernel(
    const UnitDesc* __restrict__ descs,
    const float* __restrict__ importance, int64_t imp_stride, int32_t* __restrict__ kept_idx,
    int64_t idx_stride, int32_t* __restrict__ seam) {
  using Shared = SelectShared<NT, B0, B1>;
  __shared__ __attribute__((aligned(16))) uint32_t hist[Shared::kHist];
  __shared__ Shared sh;

  const UnitDesc d = descs[blockIdx.x];
  const float* imp = importance + (int64_t)d.unit * imp_stride;
  int32_t* out = kept_idx + (int64_t)d.unit * idx_stride;
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
    // a whole piece of V stays inside the unit's row (j0 < T <= imp_stride, both multiples of it)
    constexpr int V = PER % 4 == 0 ? 4 : 2;
    typedef __attribute__((__vector_size__(V * sizeof(uint32_t)))) uint32_t piece;
    const bool vec = PER % V == 0 && (imp_stride & 3) == 0 && ((uintptr_t)importance & 15) == 0;
    if (vec) {
#pragma unroll
      for (int ev = 0; ev < PER / V; ++ev) {
        if ((in_seg >> (V * ev)) & ((1u << V) - 1u)) {
          const piece x = *reinterpret_cast<const piece*>(imp + j0 + V * ev);
#pragma unroll
          for (int e = 0; e < V; ++e) key[V * ev + e] = x[e];
        }
      }
    } else {
#pragma unroll
      for (int e = 0; e < PER; ++e)
        if ((in_seg >> e) & 1u) key[e] = __float_as_uint(imp[j0 + e]);
    }
  }

  select_rows<NT, PER, B0, B1>(d, key, in_seg, hist, sh, out, seam);
}

}  // namespace

void launch_select(hipStream_t s, const UnitDesc* descs, int n_units,
                   int max_t_in, const float* importance, int64_t imp_stride, int32_t* kept_idx,
                   int64_t idx_stride, int32_t* seam) {
  if (n_units <= 0) return;
#define HACK_SELECT(NT_, PER_, B0_, B1_)                                                                                      \
  hipLaunchKernelGGL((select_kernel<NT_, PER_, B0_, B1_>), dim3(n_units), dim3(NT_), 0, s, descs, importance, imp_stride, \
                     kept_idx, idx_stride, seam)
  if (max_t_in <= 1024) HACK_SELECT(512, 2, 11, 11);
  else if (max_t_in <= 2048) HACK_SELECT(1024, 2, 12, 10);
  else if (max_t_in <= 4096) HACK_SELECT(1024, 4, 12, 10);
  else if (max_t_in <= 6144) HACK_SELECT(1024, 6, 12, 10);
  else if (max_t_in <= 8192) HACK_SELECT(1024, 8, 12, 10);
  else if (max_t_in <= 12288) HACK_SELECT(1024, 12, 12, 10);
  else if (max_t_in <= 16384) HACK_SELECT(1024, 16, 12, 10);
  else HACK_SELECT(1024, 32, 12, 10);
#undef HACK_SELECT
}

}  // namespace hack
