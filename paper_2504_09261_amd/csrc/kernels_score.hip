// Subset-attention importance (Sec. 4.4, "Importance Estimation via Efficient
// Subset Attention") on gfx950:
//     A~ = Softmax(scale * Q~ K^T),   importance[j] = sum_i A~[i, j]
// over the uncompressed keys of the step (cache rows followed by the current
// scale's rows, read from their two homes without materialising the concat).
//
// The column sum needs each row's softmax normaliser l_i before any key's
// importance can be formed.
//
// bf16 (score_fused): one launch that reads K once.  One
// v_mfma_f32_32x32x16_bf16 column block holds all 32 observation rows; a wave
// takes 128 keys as four 32-key tiles copied HBM -> LDS asynchronously, parks
// the logits in registers, publishes its work-group's row sums in a per-unit
// exchange area, collects (bounded wait) those of the unit's other work-groups
// and then writes importance_j = sum_i 2^t_ij / l_i from the parked logits.
// fp32 (score_f32): two streaming passes over (unit, chunk of keys), fp64 dot
// products on the matrix cores:
//   pass 1  per chunk and observation row: max logit and sum of exp(logit - max)
//   pass 2  combine the chunk partials of the unit, recompute the logits and
//           write importance[j] = sum_i exp(s_ij - m_i) / l_i.
// n_obs <= 32 rows against every key is a skinny product (~31 flop per byte), so
// ALU is spent on accuracy: logits are accumulated in fp64 and the exponential
// is range-reduced exactly, which keeps float32 importance within a few ulp of
// the exact value; the ranking that follows is decided on those float32 numbers.
#include <mutex>

#include "device_util.h"
#include "hack_internal.h"
#include "score_device.h"
#include "select_device.h"

namespace hack {

namespace {

using namespace dev;

constexpr int kThreads = 256;

// 2^t for a double t with ~1 ulp float32 accuracy: the range reduction is done
// in fp64 so a large |t| does not cost relative accuracy; the result is a float
// (ldexp of the float mantissa part is exact).
__device__ __forceinline__ float exp2_split(double t) {
  const double n = rint(t);
  const float r = (float)(t - n);  // |r| <= 0.5
  return ldexpf(__builtin_amdgcn_exp2f(r), (int)n);
}
__device__ __forceinline__ double exp_neg(double x) { return (double)exp2_split(x * kLog2e); }

// Combine the per-chunk (maximum, sum) partials of one unit into sm[i] (maximum) and
// sinv[i] (1 / normaliser) for the rows i < n_obs.  The first 256 of the NT
// threads take part: thread (g, i) = (tid / 32, tid % 32) folds the chunks
// g, g + 8, ... of row i, then the eight groups are merged through LDS.
// m: maximum over this thread's chunks; sum(m): their sums relative to m.
// Ends with a barrier: sm / sinv are ready for every thread on return.
template <int NT, typename Sum>
__device__ __forceinline__ void combine_rows(double m, Sum sum, int n_obs, double* sm, double* sinv, double (*red)[kMaxObs]) {
  const int i = threadIdx.x & 31, g = threadIdx.x >> 5;
  if (NT == 256 || g < 8) red[g][i] = m;
  __syncthreads();
  m = red[0][i];
#pragma unroll
  for (int k = 1; k < 8; ++k) m = fmax(m, red[k][i]);
  __syncthreads();
  if (NT == 256 || g < 8) red[g][i] = sum(m);
  __syncthreads();
  if (g == 0) {
    double l = red[0][i];
#pragma unroll
    for (int k = 1; k < 8; ++k) l += red[k][i];
    sm[i] = m;                          // unused rows repeat row 0: exponents stay <= 0, weight zero
    sinv[i] = (i < n_obs) ? 1.0 / l : 0.0;
  }
  __syncthreads();
}
__device__ __forceinline__ void combine_stats(const double* __restrict__ st, int n_chunks, int n_obs,
                                              double* sm, double* sinv, double (*red)[kMaxObs]) {
  const int i = threadIdx.x & 31, g = threadIdx.x >> 5;
  double m = -INFINITY;
  for (int c = g; c < n_chunks; c += 8) m = fmax(m, st[(c * kMaxObs + i) * 2]);
  combine_rows<kThreads>(m, [&](double top) {
    double l = 0.0;
    for (int c = g; c < n_chunks; c += 8) {
      const double mc = st[(c * kMaxObs + i) * 2], lc = st[(c * kMaxObs + i) * 2 + 1];
      l += lc * exp_neg(mc - top);
    }
    return l;
  }, n_obs, sm, sinv, red);
}

// ---------------------------------------------------------------------------
// float32 inputs: float64 dot products on the matrix cores
// ---------------------------------------------------------------------------
// A wave forms the logits of 32 observation rows against tiles of 16 keys with
// v_mfma_f64_16x16x4_f64 (products and sums in float64, as exact as a chain of fp64
// fused multiply-adds).  Lane (i, g) = (l % 16, l / 16) feeds step 4 c + e with element
// 16 c + 4 g + e of its Q~ / K rows (any order of the contraction will do as long as
// both operands agree), so operands come from global memory in 16-byte loads without
// LDS; C register r of lane (i, g) is observation row 4 r + g, key i.  A work-group
// takes a chunk of 64 TPW keys, its four waves TPW tiles each.
// Latency bounds these launches (a 680-token schedule holds 44 Mflop of them), so the
// chunk is 64 keys (TPW = 1) while that gives at most 640 work-groups; beyond that 256 keys
// (TPW = 4), whose fewer partials are combined faster in pass 2.  Measured, us for both
// passes, TPW 1 / 4: head_dim 64, 16 units x 680 keys 11.3 / 19.2, 32 x 680 (352
// work-groups of 64 keys) 16.0 / 19.6, 64 x 1000 (1024) 27.0 / 22.2, 128 x 2000 79 / 59;
// head_dim 128: 15.4 / 29.6, 24.1 / 29.8, 40.1 / 33.7, 132 / 98.  One key per lane with a
// work-group reduction per observation row, the form this replaces, took 69 us at 16 x 680.
typedef __attribute__((__vector_size__(4 * sizeof(double)))) double doublex4;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;

// all-reduce over the 16 lanes of a row
template <typename Op>
__device__ __forceinline__ double row16_reduce(double v, Op op) {
  v = op(v, dpp_mov_f64<0xB1>(v));
  v = op(v, dpp_mov_f64<0x4E>(v));
  v = op(v, dpp_mov_f64<0x141>(v));
  return op(v, dpp_mov_f64<0x140>(v));
}

// The float32 kernels form every number with the same operations in the same order: a step that scores and selects in one launch
// keeps what hack_score and hack_select keep, and a weight depends on its logit alone, so equal keys have equal importance.
// Logits of a tile: s[h][r] of lane (i, g) is observation row 16 h + 4 r + g, key i.
template <int C>
__device__ __forceinline__ void tile_logits(const floatx4 (&qf)[2][C], const floatx4 (&kf)[C], doublex4 (&acc)[2]) {
#pragma unroll
  for (int h = 0; h < 2; ++h) acc[h] = doublex4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int c = 0; c < C; ++c)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const double kd = (double)kf[c][e];
#pragma unroll
      for (int h = 0; h < 2; ++h) acc[h] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)qf[h][c][e], kd, acc[h], 0, 0, 0);
    }
}

// Maximum and sum of exp(logit - maximum) per observation row: of this wave's TPW tiles from key0 on into red_m[w], red[w], and,
// behind a barrier, of the chunk of four such waves.
template <int TPW>
__device__ __forceinline__ void wave_stats(const double (&s)[TPW][2][4], int key0, int T_in, double (*red_m)[kMaxObs], double (*red)[kMaxObs]) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int i = lane & 15, g = lane >> 4;
  double m[8], l[8];
#pragma unroll
  for (int x = 0; x < 8; ++x) {
    m[x] = -INFINITY;
#pragma unroll
    for (int t = 0; t < TPW; ++t) m[x] = fmax(m[x], key0 + 16 * t + i < T_in ? s[t][x / 4][x % 4] : -INFINITY);
    m[x] = row16_reduce(m[x], [](double a, double b) { return fmax(a, b); });
  }
#pragma unroll
  for (int x = 0; x < 8; ++x) {
    l[x] = 0.0;
#pragma unroll
    for (int t = 0; t < TPW; ++t) l[x] += key0 + 16 * t + i < T_in ? exp_neg(s[t][x / 4][x % 4] - m[x]) : 0.0;
    l[x] = row16_reduce(l[x], [](double a, double b) { return a + b; });
  }
  if (i == 0) {   // one branch behind all eight chains, which then overlap
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      red_m[w][16 * (x / 4) + 4 * (x % 4) + g] = m[x];
      red[w][16 * (x / 4) + 4 * (x % 4) + g] = l[x];
    }
  }
}
__device__ __forceinline__ void chunk_stats(int row, const double (*red_m)[kMaxObs], const double (*red)[kMaxObs], double* m_out, double* l_out) {
  double m = red_m[0][row];     // finite: the chunk's first key exists, and wave 0 holds it
#pragma unroll
  for (int k = 1; k < 4; ++k) m = fmax(m, red_m[k][row]);
  double l = 0.0;
#pragma unroll
  for (int k = 0; k < 4; ++k)
    if (red_m[k][row] > -INFINITY) l += red[k][row] * exp_neg(red_m[k][row] - m);
  *m_out = m;
  *l_out = l;
}

// Importance of key i of a tile, in all four lanes that share it.
__device__ __forceinline__ double tile_importance(const double (&s)[2][4], int g, const double* sm, const double* sinv) {
  double imp = 0.0;
#pragma unroll
  for (int h = 0; h < 2; ++h)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 16 * h + 4 * r + g;
      imp += exp_neg(s[h][r] - sm[row]) * sinv[row];
    }
  imp += shfl_xor_f64(imp, 16);
  imp += shfl_xor_f64(imp, 32);
  return imp;
}

template <int D, int TPW, int PASS>
__global__ __launch_bounds__(kThreads) void score_f32(
    const UnitDesc* __restrict__ descs, int max_chunks,
    const float* __restrict__ q, const int32_t* __restrict__ q_rows, int n_obs, int N_k, float scale,
    const float* __restrict__ k_cache, const float* __restrict__ k_new, double* __restrict__ stats,
    float* __restrict__ importance, int64_t imp_stride) {
  constexpr int C = D / 16;             // 16-byte pieces of a row per lane
  constexpr int kChunk = 64 * TPW;      // keys per work-group
  const UnitDesc d = descs[blockIdx.y];
  const int T_in = d.len_in + d.n_new;
  if ((int)blockIdx.x * kChunk >= T_in) return;
  const int n_chunks = (T_in + kChunk - 1) / kChunk;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int i = lane & 15, g = lane >> 4;
  const int key0 = blockIdx.x * kChunk + w * 16 * TPW;

  __shared__ double red[8][kMaxObs];
  __shared__ double red_m[4][kMaxObs];
  __shared__ double sm[kMaxObs], sinv[kMaxObs];

  // Q~ rows i and 16 + i (a row past n_obs repeats row 0; it gets weight zero)
  floatx4 qf[2][C], kf[C];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    const int row = 16 * h + i;
    const float* p = q + ((int64_t)d.unit * N_k + q_rows[row < n_obs ? row : 0]) * D + 4 * g;
#pragma unroll
    for (int c = 0; c < C; ++c) qf[h][c] = *reinterpret_cast<const floatx4*>(p + 16 * c);
  }
  auto load_k = [&](int t) {
    const int j = min(key0 + 16 * t + i, T_in - 1);
    const float* p = (j < d.len_in ? k_cache + (d.in_off + j) * D : k_new + ((int64_t)d.unit * N_k + (j - d.len_in)) * D) + 4 * g;
#pragma unroll
    for (int c = 0; c < C; ++c) kf[c] = *reinterpret_cast<const floatx4*>(p + 16 * c);
  };
  load_k(0);
  double* st_unit = stats + (int64_t)blockIdx.y * max_chunks * kMaxObs * 2;
  if (PASS == 2) combine_stats(st_unit, n_chunks, n_obs, sm, sinv, red);

  double s[TPW][2][4];   // logits of tile t
#pragma unroll
  for (int t = 0; t < TPW; ++t) {
    doublex4 acc[2];
    tile_logits(qf, kf, acc);
    if (t + 1 < TPW) load_k(t + 1);
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int r = 0; r < 4; ++r) s[t][h][r] = acc[h][r] * (double)scale;
  }

  if (PASS == 1) {
    wave_stats<TPW>(s, key0, T_in, red_m, red);
    __syncthreads();
    if (threadIdx.x < kMaxObs) {
      double m, l;
      chunk_stats(threadIdx.x, red_m, red, &m, &l);
      double* o2 = st_unit + ((int64_t)blockIdx.x * kMaxObs + threadIdx.x) * 2;
      o2[0] = m;
      o2[1] = l;
    }
  } else {
#pragma unroll
    for (int t = 0; t < TPW; ++t) {
      const double imp = tile_importance(s[t], g, sm, sinv);
      const int j = key0 + 16 * t + i;
      if (g == 0 && j < T_in) importance[(int64_t)d.unit * imp_stride + j] = (float)imp;
    }
  }
}

// ---------------------------------------------------------------------------
// float32, short units: score and selection in one launch
// ---------------------------------------------------------------------------
// Pass 1 of chunks of 64 keys, whose waves also store their logits; the work-group that draws its unit's last ticket does pass 2 over
// the stored logits and ranks what it has just formed.  The chunks come from
// different XCDs: logits, partials and tickets travel as device-scope relaxed atomics, a ticket drawn only after the
// work-group's stores have been acknowledged; nobody waits for anybody.  Pass 2's operands and products, its launch and the selection's
// are saved: these launches are chains of latencies (a 256^2 schedule 118.0 -> 105.8 us; use_score_select_f32 has the steps).
// Keeping the weights instead, rounded against their tile's own maximum, would spare the last work-group the exponentials, but equal keys
// of two tiles would round differently and no longer rank by index.
template <typename T>
__device__ __forceinline__ void store_agent(T* p, T v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
template <typename T>
__device__ __forceinline__ T load_agent(const T* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

// Four waves score, eight do pass 2, whose float64 chains one wave a SIMD does not hide (16 units of 384 keys, us a step, four / eight:
// 24.1 / 22.3), and rank, PER rows a thread (T_in <= 512 PER).  logits: 2048 doubles per work-group; stats as score_f32.
template <int D, int PER>
__global__ __launch_bounds__(512) void score_select_f32(
    const UnitDesc* __restrict__ descs, const float* __restrict__ q, const int32_t* __restrict__ q_rows, int n_obs, int N_k, float scale,
    const float* __restrict__ k_cache, const float* __restrict__ k_new, double* __restrict__ logits, double* __restrict__ stats,
    unsigned* __restrict__ counters, int32_t* __restrict__ kept_idx, int64_t idx_stride, int32_t* __restrict__ seam) {
  constexpr int C = D / 16;
  constexpr int kTile = 8 * 64;                    // logits of a tile, as its wave holds them
  constexpr int NT = 512, NW = NT / 64;
  constexpr int kPerWave = NT * PER / 16 / NW;     // tiles per wave at most, all of them in flight
  using Shared = SelectShared<NT, 11, 11>;
  __shared__ __attribute__((aligned(16))) uint32_t hist[Shared::kHist];
  __shared__ Shared sh;
  __shared__ double red[8][kMaxObs], red_m[4][kMaxObs];
  __shared__ double sm[kMaxObs], sinv[kMaxObs];
  __shared__ float imp_sh[NT * PER];
  __shared__ int last_ticket;
  const UnitDesc d = descs[blockIdx.y];
  const int T_in = d.len_in + d.n_new;
  const int n_chunks = (T_in + 63) / 64, n_tiles = (T_in + 15) / 16;
  if ((int)blockIdx.x >= n_chunks) return;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15, g = lane >> 4;
  const int key0 = (blockIdx.x * 4 + w) * 16;
  double* const unit_logits = logits + (int64_t)blockIdx.y * gridDim.x * 4 * kTile + lane;
  double* const unit_stats = stats + (int64_t)blockIdx.y * gridDim.x * kMaxObs * 2;

  if (w < 4) {
    floatx4 qf[2][C], kf[C];
    // (the row numbers come in front: behind the keys they would be waited for with them)
    const int row0 = q_rows[i < n_obs ? i : 0], row1 = q_rows[16 + i < n_obs ? 16 + i : 0];
    asm volatile("" ::"v"(row0), "v"(row1));
    const int j = min(key0 + i, T_in - 1);
    const float* p = (j < d.len_in ? k_cache + (d.in_off + j) * D : k_new + ((int64_t)d.unit * N_k + (j - d.len_in)) * D) + 4 * g;
#pragma unroll
    for (int c = 0; c < C; ++c) kf[c] = *reinterpret_cast<const floatx4*>(p + 16 * c);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const float* p = q + ((int64_t)d.unit * N_k + (h == 0 ? row0 : row1)) * D + 4 * g;
#pragma unroll
      for (int c = 0; c < C; ++c) qf[h][c] = *reinterpret_cast<const floatx4*>(p + 16 * c);
    }
    doublex4 acc[2];
    tile_logits(qf, kf, acc);
    double s[1][2][4];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int r = 0; r < 4; ++r) s[0][h][r] = acc[h][r] * (double)scale;
    if (key0 < T_in) {
      double* out = unit_logits + (key0 / 16) * kTile;
#pragma unroll
      for (int x = 0; x < 8; ++x) store_agent(out + x * 64, s[0][x / 4][x % 4]);
    }
    wave_stats<1>(s, key0, T_in, red_m, red);
  }
  __syncthreads();
  if (tid < kMaxObs) {
    double m, l;
    chunk_stats(tid, red_m, red, &m, &l);
    double* o2 = unit_stats + ((int64_t)blockIdx.x * kMaxObs + tid) * 2;
    store_agent(o2, m);
    store_agent(o2 + 1, l);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's stores have been acknowledged
  __syncthreads();                                    // ... and so have the work-group's
  if (tid == 0)
    last_ticket = __hip_atomic_fetch_add(&counters[2 * blockIdx.y], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)(n_chunks - 1);
  __syncthreads();
  if (!last_ticket) return;
  if (tid == 0) store_agent(&counters[2 * blockIdx.y], 0u);   // as the next launch expects it
  clear_hist<NT, 11, 11>(hist, tid);

  // ---- pass 2: wave w takes the tiles w, w + NW, ..., whose logits arrive while the rows' partials are combined ----
  double s[kPerWave][2][4];
  auto load = [&](int slot, int t) {
    if (t < n_tiles) {
      const double* in = unit_logits + t * kTile;
#pragma unroll
      for (int x = 0; x < 8; ++x) s[slot][x / 4][x % 4] = load_agent(in + x * 64);
    }
  };
  constexpr int kChunks = (NT * PER / 64 + 7) / 8;   // of a thread in combine_rows
  double mc[kChunks], lc[kChunks];
#pragma unroll
  for (int k = 0; k < kChunks; ++k) {
    const int c = (tid >> 5) + 8 * k;
    mc[k] = -INFINITY;
    lc[k] = 0.0;
    if (tid < 256 && c < n_chunks) {
      mc[k] = load_agent(unit_stats + (c * kMaxObs + (tid & 31)) * 2);
      lc[k] = load_agent(unit_stats + (c * kMaxObs + (tid & 31)) * 2 + 1);
    }
  }
#pragma unroll
  for (int k = 0; k < kPerWave; ++k) load(k, w + NW * k);
  double top = mc[0];
#pragma unroll
  for (int k = 1; k < kChunks; ++k) top = fmax(top, mc[k]);
  combine_rows<NT>(top, [&](double m) {
    double l = 0.0;
#pragma unroll
    for (int k = 0; k < kChunks; ++k)
      if ((tid >> 5) + 8 * k < n_chunks) l += lc[k] * exp_neg(mc[k] - m);
    return l;
  }, n_obs, sm, sinv, red);
#pragma unroll
  for (int k = 0; k < kPerWave; ++k) {
    const int t = w + NW * k;
    if (t < n_tiles) {
      const double imp = tile_importance(s[k], g, sm, sinv);
      if (g == 0) imp_sh[16 * t + i] = (float)imp;
    }
  }
  __syncthreads();

  // ---- rank of rows tid PER .. of the unit ----
  const int j0 = tid * PER;
  uint32_t key[PER];
  unsigned in_seg = 0;
#pragma unroll
  for (int e = 0; e < PER; ++e) {
    const bool ranked = j0 + e >= d.sel_lo && j0 + e < d.sel_hi;
    if (ranked) in_seg |= 1u << e;
    key[e] = ranked ? __float_as_uint(imp_sh[j0 + e]) : 0u;
  }
  select_rows<NT, PER, 11, 11, true>(d, key, in_seg, hist, sh, kept_idx + (int64_t)d.unit * idx_stride, seam);
}

// ---------------------------------------------------------------------------
// bf16 MFMA path
// ---------------------------------------------------------------------------
// C = Q~ K^T per 32-key tile: A operand = Q~ (row = observation query lane%32),
// B operand = K^T (column = key lane%32); see c_row() for where the results sit.

// ---- wave-private tile pipeline -------------------------------------------
// A work item is (unit, chunk of 32 TILES keys, TILES = 1, 2, 3, 4, 6 or 8) and belongs to ONE wave: the
// wave copies its 32-key tiles HBM -> LDS with global_load_lds (16 B per lane,
// whole rows, fully coalesced), double-buffered in a private LDS region, and
// reads MFMA operands back with ds_read_b128 (XOR-swizzled chunks, conflict
// free on the 64-bank LDS).  No work-group barrier while tiles stream: waves only
// wait on their own copies (hand-placed s_waitcnt vmcnt), so they drift freely and
// keep HBM busy.  Reading K fragments straight from HBM in operand layout would touch
// 32 rows x 32 bytes per instruction and re-fetch every cache line several times.

constexpr int kMaxGroups = 64;                 // work-groups per unit the exchange supports (4 * 128 keys each)
constexpr unsigned long long kEmpty = ~0ull;   // exchange slot not published yet (a NaN pattern no row sum can have)
// One launch, K read once.  Every wave
//   A. forms the logits t_ij (log2 units) of its item, 32 observation rows x up
//      to 32 TILES keys, and parks them in registers as fixed point;
//   B. forms the row sums of p_ij = 2^t_ij (doubles: the fp64 exponent range makes
//      a running maximum unnecessary); the four waves of a work-group (always items
//      of one unit) add theirs and publish the 32 sums in the work-group's own slot
//      of the unit's exchange area with device-coherent stores;
//   C. collects the slots of all work-groups of the unit (device-coherent loads,
//      repeated until a slot no longer holds the "empty" bit pattern), adds them in
//      a fixed order, so every work-group gets the same normalisers l_i bit for bit,
//      and writes importance_j = sum_i p_ij / l_i for its keys.
// A slot value carries its own validity (a sum of powers of two is never the
// all-ones NaN pattern), so no ordering between different addresses is needed:
// one store and, normally, one or two rounds of loads replace atomic round trips.
// The wait in C needs every work-group of a unit to be resident at the same time:
// the host never launches more waves than the device holds at once (occupancy x
// compute units), so all of them run concurrently and each publishes without
// depending on anyone else.  The wait is bounded all the same: a thread that runs
// out of polls raises fault[0] (host-visible), the work-group leaves without
// writing, and the host refuses further work on the context.  fault[1] reports
// clamped logits.  Each work-group draws a ticket after it has read; the one that
// draws the unit's last ticket marks the unit's slots empty again for the next launch.
// A work-group that gives up also raises *abort_flag in device memory; every later
// launch that finds it set leaves at once, before it reads any slot, so the sums a
// failed launch left behind are never taken for valid ones.  The host clears the
// flag when it re-arms the workspace.
//
// MODE selects what a launch does:
//   kScoreFused   everything above, one launch;
//   kScoreSums    A and B only: every work-group stores its row sums (pass 1 of 2);
//   kScoreWrite   A again, then C with the sums pass 1 left (no waiting: pass 1 has
//                 completed), pass 2 of 2.  The two-pass form reads K twice but does
//                 not depend on the launch being resident as a whole.
// What bounds a launch is the latency of its stages (first tile, exchange) and then the vector unit, 30 to 47 %
// busy with some 500 instructions per 32 keys of a wave.  Rounding by one fused multiply-add instead of
// multiply, round, convert and clamp (fix_from_small), the integer part added to the exponent field and the row
// sums through LDS took 200 to 300 of 800 (one tile per wave) or 570 (four) away: 12.8 / 17.2 / 21.2 / 22.2 -> 11.6 /
// 16.1 / 19.7 / 21.0 us at 32 units of 2500 / 4000 / 6000 / 8000 keys, D = 128 (kernel trace).  Tried and slower: copies two tiles
// ahead (23 registers more; eight-tile items spill), single-tile items with one buffer and five work-groups a compute unit
// (18.2 against 16.1 us at 4000 keys: four times the slots to exchange).
// skip_publish: test hook, index of a work-group of the launch that does not publish its
// sums (-1: none); with a small spin_limit this makes the give-up path run
// deterministically while every work-group still exits normally.
enum : int { kScoreFused = 0, kScoreSums = 1, kScoreWrite = 2 };

template <int D, int TILES, int MODE>
__global__ __launch_bounds__(kThreads, 2) void score_fused(
    const ScoreItem* __restrict__ items, int n_items, const __bf16* __restrict__ q,
    const int32_t* __restrict__ q_rows, int n_obs, int N_k, float scale,
    const __bf16* __restrict__ k_cache, const __bf16* __restrict__ k_new,
    unsigned long long* __restrict__ slots, int slot_groups, unsigned* __restrict__ counters,
    float* __restrict__ importance, int64_t imp_stride, int* __restrict__ fault, int spin_limit,
    const unsigned* __restrict__ abort_flag_in, int skip_publish) {
  unsigned* abort_flag = const_cast<unsigned*>(abort_flag_in);
  // read now, acted upon once the loads of the Q~ fragments have been waited for anyway
  const unsigned aborted = (MODE == kScoreFused) ? __hip_atomic_load(abort_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
  constexpr int KK = D / 16;            // MFMA steps over the head dimension
  constexpr int CPR = D / 8;            // 16-byte chunks per row
  constexpr int RPI = 64 / CPR;         // rows per wave-wide copy instruction
  constexpr int IPT = 32 / RPI;         // copy instructions per 32-key tile (8 or 4)
  constexpr int TILE = 32 * D;          // elements per tile

  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int item = blockIdx.x * 4 + w;  // the host pads every unit to whole work-groups
  const ScoreItem it = items[item];
  ObsRows<D, 4> obs;
  obs.load(q_rows, n_obs, w, lane);
  const int T_in = it.t_in;
  constexpr int kItemTiles = TILES;
  const int key0 = it.chunk * (32 * TILES);
  const int n_tiles = max(0, min(kItemTiles, (T_in - key0 + 31) / 32));  // 0: padding item
  const int col = lane & 31, half = lane >> 5;

  __shared__ __attribute__((aligned(1024))) __bf16 tiles[4][2][TILE];
  const unsigned lds0 = (unsigned)(uintptr_t)(const __attribute__((address_space(3))) void*)&tiles[w][0][0];
  // exchange area of the unit: [work-group of the unit][observation row], kEmpty = not published yet
  unsigned long long* unit_slots = slots + (int64_t)it.pos * slot_groups * kMaxObs;
  const int group = it.chunk >> 2;         // this work-group's index inside the unit (4 items per work-group)
  unsigned* cnt = counters + 2 * it.pos;   // [1] work-groups that have read the unit's slots

  // copy of tile t (keys key0 + 32t ..) into buffer t & 1.  A tile that lies
  // wholly inside the cached rows or wholly inside the new rows (the common
  // case) is addressed as wave-uniform base + loop-invariant lane offset; a tile
  // that straddles the seam or the end picks every row's source on its own and
  // repeats the last key past the end.
  int src_off[IPT];
#pragma unroll
  for (int i = 0; i < IPT; ++i) {
    const int r = i * RPI + lane / CPR, c = lane % CPR;
    src_off[i] = (r * D + ((c ^ swz_k<D>(r)) & (CPR - 1)) * 8) * 2;
  }
  auto issue = [&](int t) {
    const int j0 = key0 + t * 32;
    const unsigned dst = lds0 + (unsigned)((t & 1) * TILE * 2);
    const bool in_cache = j0 + 32 <= it.len_in;
    const bool in_new = j0 >= it.len_in && j0 + 32 <= T_in;
    if (in_cache || in_new) {
      const __bf16* base = in_cache ? k_cache + (it.in_off + j0) * D
                                    : k_new + ((int64_t)it.unit * N_k + (j0 - it.len_in)) * D;
#pragma unroll
      for (int i = 0; i < IPT; ++i) load_to_lds(base, (unsigned)src_off[i], dst + i * 1024);
    } else {
#pragma unroll
      for (int i = 0; i < IPT; ++i) {
        const int r = i * RPI + lane / CPR, c = lane % CPR;
        const int j = min(j0 + r, T_in - 1);
        const __bf16* row = (j < it.len_in) ? k_cache + (it.in_off + j) * D
                                            : k_new + ((int64_t)it.unit * N_k + (j - it.len_in)) * D;
        load_to_lds(row + ((c ^ swz_k<D>(r)) & (CPR - 1)) * 8, dst + i * 1024);
      }
    }
  };
  // Q~ goes into the second buffer of wave 0, which no tile uses before every wave has read it.
  const __bf16* const q_lds = &tiles[0][1][0];
  obs.issue(q + (int64_t)it.unit * N_k * D, lds_addr_of(q_lds), w, lane);
  if (n_tiles > 0) issue(0);

  int k_off[KK];   // operand reads: row col, chunk 2 kk + half
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) k_off[kk] = col * D + (((2 * kk + half) ^ swz_k<D>(col)) & (CPR - 1)) * 8;
  const double c2 = (double)scale * kLog2e * kFixOne;  // logits in log2 units, fixed point: t * 2^22 = dot * c2
  // Q~ has landed, the first tile may still be on its way
  if (n_tiles > 0) dma_wait_but<IPT>();
  else dma_wait_but<0>();
  __syncthreads();
  bf16x8 qf[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) qf[kk] = *reinterpret_cast<const bf16x8*>(&q_lds[k_off[kk]]);
  __syncthreads();   // (a wave's row sums need both of its buffers at head_dim 64, whatever TILES is)
  if (MODE == kScoreFused && __builtin_amdgcn_readfirstlane(aborted) != 0) {
    // an earlier launch gave up: its sums may still sit in the slots, so nothing here may be trusted
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the first tile's copy must not outlive the wave
    return;
  }

  // ---- A: logits of the item's tiles ---------------------------------------
  // Between A and C a logit waits in registers either as its fixed-point value (one register; 2^t is
  // formed again in C) or, for all but the largest items (TILES <= 4, where the registers are there), as the
  // double 2^t of that same fixed-point value (two registers; nothing is recomputed).  Both forms give
  // the same numbers bit for bit.
  constexpr bool kParkP = TILES <= 4;
  int tq[kParkP ? 1 : kItemTiles][16];
  double pq[kParkP ? kItemTiles : 1][16];
  auto p_of = [&](int t, int r) -> double { return kParkP ? pq[t][r] : exp2_fix(tq[t][r]); };
  bool clamped = false;                // a logit hit the clamp of the parked format
  const double dot_safe = (double)(kFixLimit - 1) / c2;   // a dot product below this stays clear of it
#pragma unroll
  for (int t = 0; t < kItemTiles; ++t) {
    if (t < n_tiles) {                 // wave-uniform
      if (t + 1 < n_tiles) {
        issue(t + 1);
        dma_wait_but<IPT>();          // tile t has landed, tile t+1 stays in flight
      } else {
        dma_wait_but<0>();
      }
      const __bf16* Kt = &tiles[w][t & 1][0];
      // Raw dot products: every MFMA covers 16 head-dim elements and starts from a
      // zero accumulator; the slice results are summed in fp64, so float32 rounding
      // only ever acts on partial sums that are small next to the full dot product.
      double sd[16];
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) {
        const bf16x8 kf = *reinterpret_cast<const bf16x8*>(&Kt[k_off[kk]]);
        floatx16 c = {0};
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[kk], kf, c, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 16; ++r) sd[r] = (kk == 0) ? (double)c[r] : sd[r] + (double)c[r];   // 0.0 + x == x: same bits
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
      for (int r = 0; r < 16; ++r) {
        if (kParkP) pq[t][r] = exp2_fix(qv[r]);
        else tq[t][r] = qv[r];
      }
    } else {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        if (kParkP) pq[t][r] = 0.0;
        else tq[t][r] = 0;
      }
    }
  }

  // A logit that hit the clamp of the parked format makes the result differ from
  // the definition: tell the host (second flag word; the launch still completes).
  if (__any(clamped)) {
    if (lane == 0) __hip_atomic_store(fault + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }

  // ---- B: row sums of the work-group -> its slot ------------------------------
  // Each wave's tile buffers are free by now, so they carry the reduction inside the wave and the
  // exchange inside the work-group: every wave leaves its 32 row sums there, wave 0 adds the four
  // and publishes one value per row.
  double* red = reinterpret_cast<double*>(&tiles[w][0][0]);
  if (MODE != kScoreWrite) {
    char* buf = reinterpret_cast<char*>(red);
    if (kParkP) {
      double lsum[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) lsum[r] = 0.0;
#pragma unroll
      for (int t = 0; t < kItemTiles; ++t)
        if (t < n_tiles && key0 + t * 32 + col < T_in) {
#pragma unroll
          for (int r = 0; r < 16; ++r) lsum[r] += p_of(t, r);
        }
#pragma unroll
      for (int r = 0; r < 16; ++r) put_row(buf, r, col, half, lsum[r]);
    } else {
      // row by row: there are no registers for 16 sums beside the parked logits
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        double lsum = 0.0;
#pragma unroll
        for (int t = 0; t < kItemTiles; ++t)
          if (t < n_tiles && key0 + t * 32 + col < T_in) lsum += p_of(t, r);
        put_row(buf, r, col, half, lsum);
      }
    }
    wave_lds_order();
    const double l = take_rows(buf, lane);
    wave_lds_order();
    if ((lane & 1) == 0) red[lane >> 1] = l;
  }
  __syncthreads();
  if (MODE != kScoreWrite && w == 0 && lane < kMaxObs && (MODE != kScoreFused || (int)blockIdx.x != skip_publish)) {
    double tot = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) tot += reinterpret_cast<const double*>(&tiles[k][0][0])[lane];
    __hip_atomic_store(&unit_slots[group * kMaxObs + lane], (unsigned long long)__double_as_longlong(tot),
                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (MODE == kScoreSums) return;
  // ---- C: collect the unit's slots ---------------------------------------------
  // thread (sub, row) = (tid / 32, tid % 32) takes work-groups sub, sub + 8, ... of row `row`
  double* part8 = reinterpret_cast<double*>(&tiles[1][0][0]) + 64;   // [8][32] partial sums, behind wave 1's row sums
  double* inv_s = reinterpret_cast<double*>(&tiles[0][0][0]) + 64;   // [32], behind wave 0's row sums
  int* ok_s = reinterpret_cast<int*>(inv_s + kMaxObs);
  if (tid == 0) *ok_s = 1;
  __syncthreads();
  {
    const int row = tid & 31, sub = tid >> 5;
    // up to kMaxGroups / 8 slots per thread: all loads are issued first, then each is
    // repeated until it is valid (work-groups past the end count as +0.0)
    unsigned long long bits[kMaxGroups / 8];
#pragma unroll
    for (int k = 0; k < kMaxGroups / 8; ++k) {
      const int g2 = sub + 8 * k;
      bits[k] = (g2 < it.n_groups) ? __hip_atomic_load(&unit_slots[g2 * kMaxObs + row], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                   : 0ull;
    }
    double acc = 0.0;
    bool ok = true;
#pragma unroll
    for (int k = 0; k < kMaxGroups / 8; ++k) {
      int polls = 0;
      while (MODE == kScoreFused && bits[k] == kEmpty) {
        if (++polls > spin_limit) { ok = false; break; }
        __builtin_amdgcn_s_sleep(1);
        bits[k] = __hip_atomic_load(&unit_slots[(sub + 8 * k) * kMaxObs + row], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      acc += __longlong_as_double((long long)bits[k]);
    }
    part8[sub * kMaxObs + row] = acc;
    if (!ok) *ok_s = 0;
  }
  __syncthreads();
  if (*ok_s == 0) {
    if (tid == 0) {
      __hip_atomic_store(abort_flag, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(fault, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    return;
  }
  unsigned ticket = 0;
  if (MODE == kScoreFused && w == 0) {
    if (lane < kMaxObs) {
      double l = 0.0;
#pragma unroll
      for (int k = 0; k < 8; ++k) l += part8[k * kMaxObs + lane];   // fixed order: the same bits in every work-group
      inv_s[lane] = (lane < n_obs) ? 1.0 / l : 0.0;
    }
    // every slot this work-group needed has been read (the values were used above):
    // whoever draws the last ticket may mark the slots empty without racing a reader
    if (lane == 0) ticket = atomicAdd(&cnt[1], 1u);
  }
  if (MODE == kScoreWrite && w == 0 && lane < kMaxObs) {
    double l = 0.0;
#pragma unroll
    for (int k = 0; k < 8; ++k) l += part8[k * kMaxObs + lane];
    inv_s[lane] = (lane < n_obs) ? 1.0 / l : 0.0;
  }
  __syncthreads();
  double inv_r[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) inv_r[r] = inv_s[c_row(r, half)];

#pragma unroll
  for (int t = 0; t < kItemTiles; ++t) {
    if (t < n_tiles) {
      double imp = 0.0;
#pragma unroll
      for (int r = 0; r < 16; ++r) imp = fma(p_of(t, r), inv_r[r], imp);
      imp += shfl_xor_f64(imp, 32);
      const int j = key0 + t * 32 + col;
      if (j < T_in && half == 0) importance[(int64_t)it.unit * imp_stride + j] = (float)imp;
    }
  }
  if (MODE == kScoreFused && w == 0) {
    // the work-group that drew a unit's last ticket leaves slots and counter as the next launch expects them
    ticket = __builtin_amdgcn_readfirstlane(ticket);
    if ((int)ticket == it.n_groups - 1) {
      for (int e = lane; e < it.n_groups * kMaxObs; e += 64)
        __hip_atomic_store(&unit_slots[e], kEmpty, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (lane == 0) cnt[1] = 0;
    }
  }
}

// ---------------------------------------------------------------------------
// bf16, short units: score and selection in one launch
// ---------------------------------------------------------------------------
// A work-group of NW waves owns a unit of at most 32 TILES NW keys (NW = 4, 8, 16): wave w takes the tiles w and (TILES = 2) w + NW, the row
// sums meet in LDS instead of the exchange area, importance goes to LDS only and thread j ranks key j.  The numbers
// are those of score_fused up to the order in which the row sums are added in fp64.  Latency bounds these launches: a
// score launch, whose work-groups wait for each other through L2, and a selection launch behind it take 8 + 4.4 us (kernel trace) at
// 60 units of 46 to 475 keys (one 256^2 image: 108.6 -> 100.6 us, 960 units 349 -> 318).
// MOVE: the work-group also moves the rows that it keeps, and further work-groups append the new rows of the n_append units
// that keep everything (append_descs), in place of a launch of move_kernel behind this one: its copies run beside other
// work-groups' arithmetic, and nobody reads the list back.  Schedules whose last step compresses, us, two launches / one: 128 units of 500
// keys 40.8 / 38.2 (half of them compressing 42.9 / 39.5), 256 of 240 33.5 / 29.7, 512 of 1000 181 / 179; head_dim 128, 128 of 250 38.9 / 35.8, 256 of
// 500 84 / 80; 60 units of 1000 45.6 / 45.7; a batch of 32 256^2 images (960 units, three such steps) 307.6 / 295.
struct StepMove {
  const UnitDesc* append_descs;
  CachePtrs cache;
  const __bf16* v_new;
  int pos_new;
};

// Rows of K, V and position ids of one unit to where the next step expects them, by a work-group of THREADS: rows list[i] (LDS) of
// [cached | new] behind out_off, or, list NULL, all new rows behind the cached ones.
template <int D, int THREADS>
__device__ __forceinline__ void move_unit(const UnitDesc& d, const uint32_t* list, const __bf16* k_new, const StepMove& mv, int N_k) {
  constexpr int LPR = D / 8, RPP = THREADS / LPR, BATCH = 4;   // lanes per row, rows per pass, passes in flight
  const int lane = threadIdx.x % LPR;
  const int n_rows = list ? d.n_out : d.n_new;
  const int64_t dst0 = list ? d.out_off : d.in_off + d.len_in, new0 = (int64_t)d.unit * N_k;
  for (int i0 = threadIdx.x / LPR; i0 < n_rows; i0 += BATCH * RPP) {
    uintx4 kr[BATCH], vr[BATCH];
    int pos[BATCH];
#pragma unroll
    for (int b = 0; b < BATCH; ++b) {
      const int i = min(i0 + b * RPP, n_rows - 1);
      const int s = list ? (int)list[i] : d.len_in + i;
      const bool cached = s < d.len_in;
      const int64_t row = cached ? d.in_off + s : new0 + (s - d.len_in);
      kr[b] = (cached ? static_cast<const uintx4*>(mv.cache.k) : reinterpret_cast<const uintx4*>(k_new))[row * LPR + lane];
      vr[b] = (cached ? static_cast<const uintx4*>(mv.cache.v) : reinterpret_cast<const uintx4*>(mv.v_new))[row * LPR + lane];
      pos[b] = mv.pos_new + (s - d.len_in);
      if (cached && mv.cache.pos != nullptr) pos[b] = mv.cache.pos[row];
    }
#pragma unroll
    for (int b = 0; b < BATCH; ++b) {
      const int i = i0 + b * RPP;
      if (i < n_rows) {
        static_cast<uintx4*>(mv.cache.k)[(dst0 + i) * LPR + lane] = kr[b];
        static_cast<uintx4*>(mv.cache.v)[(dst0 + i) * LPR + lane] = vr[b];
        if (mv.cache.pos != nullptr && lane == 0) mv.cache.pos[dst0 + i] = pos[b];
      }
    }
  }
}

template <int D, int NW, int TILES, bool MOVE>
__global__ __launch_bounds__(64 * NW) void score_select(
    const UnitDesc* __restrict__ descs, const __bf16* __restrict__ q,
    const int32_t* __restrict__ q_rows, int n_obs, int N_k, float scale, const __bf16* __restrict__ k_cache,
    const __bf16* __restrict__ k_new, int32_t* __restrict__ kept_idx, int64_t idx_stride, int32_t* __restrict__ seam,
    int* __restrict__ fault, int n_units, StepMove mv) {
  if (MOVE && (int)blockIdx.x >= n_units) {
    move_unit<D, 64 * NW>(mv.append_descs[blockIdx.x - n_units], nullptr, k_new, mv, N_k);
    return;
  }
  using Shared = SelectShared<64 * NW, 11, 11>;
  static_assert(Shared::kHist * 4 <= NW * 8192, "histograms fit the tile buffers");
  __shared__ __attribute__((aligned(1024))) char bufs[NW][8192];
  __shared__ double red[NW][kMaxObs], inv_s[NW][kMaxObs];
  __shared__ uint32_t keys[64 * NW];
  __shared__ Shared sh;
  __shared__ __attribute__((aligned(1024))) __bf16 q_lds[32 * D];

  const UnitDesc d = descs[blockIdx.x];
  const int tid = threadIdx.x;
  score_unit<D, NW, TILES>(d, q, q_rows, n_obs, N_k, scale, k_cache, k_new, bufs, red, inv_s, keys, q_lds, fault);
  uint32_t* const hist = reinterpret_cast<uint32_t*>(&bufs[0][0]);
  clear_hist<64 * NW, 11, 11>(hist, tid);
  __syncthreads();

  // ---- selection ----
  uint32_t key[1] = {0};
  const unsigned in_seg = tid >= d.sel_lo && tid < d.sel_hi ? 1u : 0u;
  if (in_seg) key[0] = keys[tid];
  select_rows<64 * NW, 1, 11, 11, true>(d, key, in_seg, hist, sh, kept_idx + (int64_t)d.unit * idx_stride, seam, MOVE ? keys : nullptr);
  if constexpr (MOVE) {
    __syncthreads();
    move_unit<D, 64 * NW>(d, keys, k_new, mv, N_k);
  }
}

template <int D, int TPW>
void launch_f32(hipStream_t s, const UnitDesc* descs, int n_units, int max_t_in, const float* q,
                const int32_t* q_rows, int n_obs, int N_k, float scale, const float* k_cache, const float* k_new, double* stats,
                float* importance, int64_t imp_stride) {
  const int max_chunks = (max_t_in + 64 * TPW - 1) / (64 * TPW);
  const dim3 grid(max_chunks, n_units);
  hipLaunchKernelGGL((score_f32<D, TPW, 1>), grid, dim3(kThreads), 0, s, descs, max_chunks, q, q_rows, n_obs, N_k, scale,
                     k_cache, k_new, stats, importance, imp_stride);
  hipLaunchKernelGGL((score_f32<D, TPW, 2>), grid, dim3(kThreads), 0, s, descs, max_chunks, q, q_rows, n_obs, N_k, scale,
                     k_cache, k_new, stats, importance, imp_stride);
}

}  // namespace

int score_max_groups() { return kMaxGroups; }

// Items (= waves) of one fused launch the device keeps resident at once, for items of item_keys keys.
int score_fused_capacity(int head_dim, int item_keys) {
  int dev = 0, cus = 0, blocks = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  hipError_t e = hipErrorInvalidValue;
#define HACK_OCC(D_, TILES_) hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, score_fused<D_, TILES_, kScoreFused>, kThreads, 0)
  switch (item_keys) {
    case 32: e = head_dim == 64 ? HACK_OCC(64, 1) : HACK_OCC(128, 1); break;
    case 64: e = head_dim == 64 ? HACK_OCC(64, 2) : HACK_OCC(128, 2); break;
    case 96: e = head_dim == 64 ? HACK_OCC(64, 3) : HACK_OCC(128, 3); break;
    case 128: e = head_dim == 64 ? HACK_OCC(64, 4) : HACK_OCC(128, 4); break;
    case 192: e = head_dim == 64 ? HACK_OCC(64, 6) : HACK_OCC(128, 6); break;
    case 256: e = head_dim == 64 ? HACK_OCC(64, 8) : HACK_OCC(128, 8); break;
    default: break;
  }
#undef HACK_OCC
  if (e != hipSuccess) return 0;
  return blocks * cus * (kThreads / 64);
}

template <int D, int TILES>
static void launch_score_t(hipStream_t s, dim3 grid, bool two_pass, const ScoreItem* items, int n_items, const __bf16* q,
                           const int32_t* q_rows, int n_obs, int N_k, float scale, const __bf16* k_cache,
                           const __bf16* k_new, unsigned long long* slots, int slot_groups, unsigned* counters,
                           float* importance, int64_t imp_stride, int* fault, int spin_limit,
                           const unsigned* abort_flag, int skip_publish) {
#define HACK_SCORE_ARGS grid, dim3(kThreads), 0, s, items, n_items, q, q_rows, n_obs, N_k, scale, k_cache, k_new, slots, \
                        slot_groups, counters, importance, imp_stride, fault, spin_limit, abort_flag, skip_publish
  if (two_pass) {
    hipLaunchKernelGGL((score_fused<D, TILES, kScoreSums>), HACK_SCORE_ARGS);
    hipLaunchKernelGGL((score_fused<D, TILES, kScoreWrite>), HACK_SCORE_ARGS);
  } else {
    hipLaunchKernelGGL((score_fused<D, TILES, kScoreFused>), HACK_SCORE_ARGS);
  }
#undef HACK_SCORE_ARGS
}

void launch_score_fused(hipStream_t s, int head_dim, int item_keys, bool two_pass, const ScoreItem* items, int n_items,
                        const void* q, const int32_t* q_rows, int n_obs, int N_k, float scale, const void* k_cache,
                        const void* k_new, unsigned long long* slots, int slot_groups, unsigned* counters,
                        float* importance, int64_t imp_stride, int* fault, int spin_limit, const unsigned* abort_flag,
                        int skip_publish) {
  if (n_items <= 0) return;
  typedef __bf16 T;
  dim3 grid((n_items + 3) / 4);
#define HACK_SCORE_CALL(D_, TILES_)                                                                                   \
  launch_score_t<D_, TILES_>(s, grid, two_pass, items, n_items, (const T*)q, q_rows, n_obs, N_k, scale, (const T*)k_cache, \
                             (const T*)k_new, slots, slot_groups, counters, importance, imp_stride, fault, spin_limit,  \
                             abort_flag, skip_publish)
  if (head_dim == 64) {
    switch (item_keys) {
      case 32: HACK_SCORE_CALL(64, 1); break;
      case 64: HACK_SCORE_CALL(64, 2); break;
      case 96: HACK_SCORE_CALL(64, 3); break;
      case 192: HACK_SCORE_CALL(64, 6); break;
      case 256: HACK_SCORE_CALL(64, 8); break;
      default: HACK_SCORE_CALL(64, 4); break;
    }
  } else {
    switch (item_keys) {
      case 32: HACK_SCORE_CALL(128, 1); break;
      case 64: HACK_SCORE_CALL(128, 2); break;
      case 96: HACK_SCORE_CALL(128, 3); break;
      case 192: HACK_SCORE_CALL(128, 6); break;
      case 256: HACK_SCORE_CALL(128, 8); break;
      default: HACK_SCORE_CALL(128, 4); break;
    }
  }
#undef HACK_SCORE_CALL
}

// ---------------------------------------------------------------------------
// hack_score_static: the same importance with every scratch buffer in a fixed
// device array of this library, for callers that must not allocate
// ---------------------------------------------------------------------------
// The score kernels' scratch (work items, q-row table, row-sum exchange slots) lives in
// a file-scope device array instead of context memory; the work items are written by a
// small planning kernel from by-value arguments, so nothing is copied from the host.
// The array is one per GPU and shared by every call on that GPU.
namespace {

constexpr int kStaticItemsMax = kStaticUnitsMax * 4 * kMaxGroups;   // 4 items per work-group, kMaxGroups work-groups per unit
struct StaticScratch {
  ScoreItem items[kStaticItemsMax];                                        // 512 KiB
  unsigned long long slots[(size_t)kStaticUnitsMax * kMaxGroups * kMaxObs]; // 1 MiB
  int32_t q_rows[kMaxObs];
  unsigned counters[2 * kStaticUnitsMax + 64];                             // unused by the two-pass form; abort word last
};
static __device__ __align__(256) unsigned char scratch[sizeof(StaticScratch)];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
StaticScratch* g_scratch_ptr[kMaxDevices] = {};   // device address of `scratch` on each GPU (its name is not one in host code)

// Writes the work items of the planned units (4 * wgs items per unit, in caller order) and the
// q-row table.  One work-group.
__global__ __launch_bounds__(256) void score_static_plan(StaticScorePlan plan, ScoreItem* __restrict__ items,
                                                          int32_t* __restrict__ q_rows) {
  __shared__ int first[kStaticUnitsMax + 1];
  if (threadIdx.x == 0) {
    int n = 0;
    for (int i = 0; i < plan.n_units; ++i) {
      first[i] = n;
      const int t_in = plan.len_in[i] + plan.n_new;
      n += 4 * (((t_in + plan.item_keys - 1) / plan.item_keys + 3) / 4);
    }
    first[plan.n_units] = n;
  }
  if (threadIdx.x < kMaxObs) q_rows[threadIdx.x] = plan.q_rows[threadIdx.x];
  __syncthreads();
  for (int i = 0; i < plan.n_units; ++i) {
    const int n = first[i + 1] - first[i];
    const int t_in = plan.len_in[i] + plan.n_new;
    for (int c = threadIdx.x; c < n; c += blockDim.x)
      items[first[i] + c] = ScoreItem{plan.in_off[i], plan.unit[i], plan.len_in[i], t_in, c, i, n / 4};
  }
}

}  // namespace

int score_static_units_max() { return kStaticUnitsMax; }
size_t score_static_scratch_bytes() { return sizeof(StaticScratch); }

int score_static_item_count(const StaticScorePlan& plan) {
  int n = 0;
  for (int i = 0; i < plan.n_units; ++i)
    n += 4 * (((plan.len_in[i] + plan.n_new + plan.item_keys - 1) / plan.item_keys + 3) / 4);
  return n;
}

// Looks up (once per device, with that device current) where this GPU keeps its copy of `scratch`.
hipError_t score_static_setup(int device) {
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[device]) return hipSuccess;
  int cur = -1;
  hipError_t e = hipGetDevice(&cur);
  if (e != hipSuccess) return e;
  if (cur != device && (e = hipSetDevice(device)) != hipSuccess) return e;
  void* p = nullptr;
  e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (cur != device) (void)hipSetDevice(cur);
  if (e != hipSuccess) return e;
  g_scratch_ptr[device] = static_cast<StaticScratch*>(p);
  return hipSuccess;
}

hipError_t launch_score_static(hipStream_t s, int device, int head_dim, const StaticScorePlan& plan, const void* q, int n_obs,
                               int N_k, float scale, const void* k_cache, const void* k_new, float* importance,
                               int64_t imp_stride, int* fault) {
  StaticScratch* sc = (device >= 0 && device < kMaxDevices) ? g_scratch_ptr[device] : nullptr;
  if (!sc) return hipErrorNotInitialized;
  const int n_items = score_static_item_count(plan);
  if (n_items <= 0) return hipSuccess;
  if (n_items > kStaticItemsMax) return hipErrorInvalidValue;
  hipLaunchKernelGGL(score_static_plan, dim3(1), dim3(256), 0, s, plan, sc->items, sc->q_rows);
  // the two-pass form: every slot that pass 2 reads is written by pass 1 of the same call, so the
  // array needs no clearing between calls
  launch_score_fused(s, head_dim, plan.item_keys, true, sc->items, n_items, q, sc->q_rows, n_obs, N_k, scale, k_cache, k_new,
                     sc->slots, kMaxGroups, sc->counters, importance, imp_stride, fault, 0,
                     sc->counters + 2 * kStaticUnitsMax, -1);
  return hipGetLastError();
}

// Where one work-group per unit beats two launches.  Measured, us a schedule of four steps whose last compresses, two
// launches / one, at 8, 32, 128, 512 units: head_dim 64, 210 keys 33.0 / 30.3, 33.7 / 31.0, 37.4 / 34.6, 62.5 / 57.0; 498 keys
// 33.9 / 32.6, 35.8 / 34.5, 54.0 / 50.8, 91 / 88; 690 keys 35.0 / 36.3, 38.8 / 39.8, 61.9 / 59.9, 131 / 129.5; 975 keys 37.5 / 39.6,
// 44 / 46.4, 74.7 / 71.9, 178 / 179; head_dim 128, 210 keys 38.0 / 35.8, 39.9 / 37.3, 51.3 / 48.5, 80.3 / 77.0; 303 keys 38.4 / 37.4, 41 / 39.9,
// 60.5 / 57.4, 103 / 104.6; 498 keys 40.2 / 40.4, 47.1 / 46.6, 67 / 64.2, 145 / 147.4; 690 keys 41.8 / 46.6, 55.5 / 58.7, 84.4 / 84.8,
// 214 / 211 (16 waves of 128 registers, dropped).
bool use_score_select(int head_dim, int n_units, int max_t_in) {
  if (head_dim == 64) return max_t_in <= 512 || (max_t_in <= 1024 && n_units >= 128);
  return max_t_in <= 256 || (max_t_in <= 512 && n_units <= 256);
}

template <bool MOVE>
static void launch_small(hipStream_t s, int head_dim, const UnitDesc* descs, int n_units, int max_t_in,
                         const void* q, const int32_t* q_rows, int n_obs, int N_k, float scale, const void* k_cache,
                         const void* k_new, int32_t* kept_idx, int64_t idx_stride, int32_t* seam, int* fault, int n_append,
                         const StepMove& mv) {
  if (n_units <= 0) return;
#define HACK_SMALL(D_, NW_, TILES_)                                                                                          \
  hipLaunchKernelGGL((score_select<D_, NW_, TILES_, MOVE>), dim3(n_units + n_append), dim3(64 * NW_), 0, s, descs, \
                     (const __bf16*)q, q_rows, n_obs, N_k, scale, (const __bf16*)k_cache, (const __bf16*)k_new, kept_idx, idx_stride, seam, \
                     fault, n_units, mv)
  // one tile a wave while every unit has a compute unit to itself: 30 units of 155 keys 7.6 -> 7.1 us (kernel trace); sixteen waves of
  // one tile lose (60 units of 420 keys 9.2 -> 10.2)
  const bool few = n_units <= 256;
  if (head_dim == 64) {
    if (max_t_in <= 256 && few) HACK_SMALL(64, 8, 1);
    else if (max_t_in <= 256) HACK_SMALL(64, 4, 2);
    else if (max_t_in <= 512) HACK_SMALL(64, 8, 2);
    else HACK_SMALL(64, 16, 2);
  } else {
    if (max_t_in <= 256 && few) HACK_SMALL(128, 8, 1);
    else if (max_t_in <= 256) HACK_SMALL(128, 4, 2);
    else HACK_SMALL(128, 8, 2);
  }
#undef HACK_SMALL
}

void launch_score_select(hipStream_t s, int head_dim, const UnitDesc* descs, int n_units, int max_t_in,
                         const void* q, const int32_t* q_rows, int n_obs, int N_k, float scale, const void* k_cache,
                         const void* k_new, int32_t* kept_idx, int64_t idx_stride, int32_t* seam, int* fault) {
  launch_small<false>(s, head_dim, descs, n_units, max_t_in, q, q_rows, n_obs, N_k, scale, k_cache, k_new, kept_idx, idx_stride,
                      seam, fault, 0, StepMove{});
}

void launch_score_select_move(hipStream_t s, int head_dim, const UnitDesc* descs, int n_units, const UnitDesc* append_descs, int n_append,
                              int max_t_in, const void* q, const int32_t* q_rows, int n_obs, int N_k, float scale, CachePtrs cache,
                              const void* k_new, const void* v_new, int pos_new, int32_t* kept_idx, int64_t idx_stride, int* fault) {
  launch_small<true>(s, head_dim, descs, n_units, max_t_in, q, q_rows, n_obs, N_k, scale, cache.k, k_new, kept_idx, idx_stride,
                     nullptr, fault, n_append, StepMove{append_descs, cache, (const __bf16*)v_new, pos_new});
}

void launch_score_select_f32(hipStream_t s, int head_dim, const UnitDesc* descs, int n_units, int max_t_in, const void* q,
                             const int32_t* q_rows, int n_obs, int N_k, float scale, const void* k_cache, const void* k_new,
                             double* logits, double* stats, unsigned* counters, int32_t* kept_idx, int64_t idx_stride, int32_t* seam) {
  if (n_units <= 0 || max_t_in <= 0) return;
  const dim3 grid((max_t_in + 63) / 64, n_units);
#define HACK_SMALL(D_, PER_)                                                                                                     \
  hipLaunchKernelGGL((score_select_f32<D_, PER_>), grid, dim3(512), 0, s, descs, (const float*)q, q_rows, n_obs, N_k, scale, \
                     (const float*)k_cache, (const float*)k_new, logits, stats, counters, kept_idx, idx_stride, seam)
  if (head_dim == 64) {
    if (max_t_in <= 512) HACK_SMALL(64, 1);
    else HACK_SMALL(64, 2);
  } else {
    if (max_t_in <= 512) HACK_SMALL(128, 1);
    else HACK_SMALL(128, 2);
  }
#undef HACK_SMALL
}

void launch_score_f32(hipStream_t s, int head_dim, const UnitDesc* descs, int n_units,
                      int max_t_in, const void* q, const int32_t* q_rows, int n_obs, int N_k, float scale,
                      const void* k_cache, const void* k_new, double* stats, float* importance,
                      int64_t imp_stride) {
  if (n_units <= 0 || max_t_in <= 0) return;
  const bool small = score_f32_chunk(n_units, max_t_in) == 64;
  typedef float T;
#define HACK_ARGS s, descs, n_units, max_t_in, (const T*)q, q_rows, n_obs, N_k, scale, (const T*)k_cache, (const T*)k_new, \
                  stats, importance, imp_stride
  if (head_dim == 64) {
    if (small) launch_f32<64, 1>(HACK_ARGS);
    else launch_f32<64, 4>(HACK_ARGS);
  } else {
    if (small) launch_f32<128, 1>(HACK_ARGS);
    else launch_f32<128, 4>(HACK_ARGS);
  }
#undef HACK_ARGS
}

}  // namespace hack
