// Final-step merge of contextual heads (Sec. 4.4, paragraph after the f_C
// equation; supplementary "Compression Setting": only f_C, only the last
// generation step) on gfx950.
//
// The rows a unit discards at its last compression are folded into the rows it
// keeps: every evicted row e goes to its nearest retained counterpart
//     n(e) = argmax_r cos(k_e, k_r)      (r over the kept rows, ties to the lower index)
// with weight w_e = max(cos(k_e, k_n(e)), 0), and every kept row becomes the weighted
// average of itself (weight 1) and the rows that went to it, keys and values alike:
//     K^_r = (k_r + sum_{e: n(e)=r} w_e k_e) / (1 + sum w_e),   V^_r likewise.
// (The paper names the operation and refers to another work for its definition; the
// formulas above are this library's reading of "similarity-weighted averaging into the
// nearest retained counterpart".)
//
// Three launches, after the gather has written K[I], V[I] into the unit's output rows:
//   merge_norms    1/|k_r| of the kept keys;
//   merge_nearest  MFMA pass: a wave holds 32 cache rows (candidates) as the B operand,
//                  the kept keys stream through LDS as the A operand together with
//                  their inverse norms; per lane a running (best, arg-best) over 16 kept
//                  rows per block, the lane pair (l, l^32) combined at the end.  Which of its
//                  rows are kept a work-group finds from the kept indices (marks in LDS), so that no
//                  launch has to mark them in memory: one launch and 2 us a merge less than with a
//                  fill and a scatter of marks;
//   merge_apply    a work-group takes 8 or 32 kept rows: its waves scan the assignment once,
//                  each a contiguous quarter, and leave the rows that go to one of them
//                  in LDS lists (ascending); every wave then folds the listed rows, eight
//                  loads in flight, into its 2 or 8 kept rows in ascending row order (so the float32 sums are formed
//                  in a fixed order: the result is reproducible bit for bit) and rewrites
//                  them in place.
// bf16 only.  The products of bf16 values are exact in float32; dots accumulate in
// float32 on the matrix core, the averages in float32 on the vector ALU.
#include <algorithm>

#include "device_util.h"
#include "hack_internal.h"

namespace hack {

namespace {

using namespace dev;

constexpr int kThreads = 256;
constexpr int kWaves = 4;
constexpr int kRing = 4;          // LDS ring slots (32-row blocks of kept keys): two stages of two blocks

constexpr int kNearRows = kWaves * 32;              // cache rows per work-group of merge_nearest in one part
constexpr int kPartsRing = 12;                      // LDS ring slots in four parts: three stages of four blocks
// Work-groups (32 cache rows each) of merge_nearest up to which it runs in four parts: as many as are resident at once, one on
// a compute unit at head_dim 128 (103 KB LDS) and at least two at 64; a second wave of them costs what the shorter walk gains.
// Measured, us a merge of all its launches, one part / four; head_dim 128, units of cache rows and kept rows (groups): 1 of 5024
// and 2000 (157) 49.8 / 29.3, 7 of 656 and 40 (147) 19.2 / 18.9, 2 of 5024 and 1200 (314) 37.0 / 36.4, 8 of 1256 and 150 (320)
// 18.7 / 21.9, 3 of 5024 and 600 (471) 28.1 / 29.5, 12 of 2704 and 400 (1020) 28.1 / 40.9; head_dim 64: 2 of 5024 and 1200 (314)
// 33.3 / 25.1, 16 of 896 and 150 (448) 17.2 / 17.2, 12 of 1256 and 350 (480) 19.0 / 17.4, 40 of 656 and 150 (840) 17.7 / 20.8.
template <int D>
constexpr int64_t kPartsGroups = D == 128 ? 256 : 512;
constexpr int kNormRows = kThreads / 8;             // kept rows per work-group in merge_norms (8 lanes per row)
// Cache rows that the work-groups of merge_apply may scan together while each takes 8 kept rows; beyond that it takes 32.  Measured, us
// a schedule that ends with the merge, 32 / 16 / 8 rows (rows scanned at 8): 12 units of 5500 and 648 kept rows (5.3M) 512 / 506 / 503;
// 60 of 358 and 102 (0.1M) 128 / 118 / 114; 480 such units (2.2M) 352 / 348 / 346; 32 of 1200 and 190 (0.9M) 126 / 109 / 100; 12 of 6039 and 1943
// (17.6M) 821 / 820 / 825; 48 of 5500 and 648 (21M) 1305 / 1296 / 1301; 12 of 8700 and 3900 (35M) 1190 / 1194 / 1208.
constexpr int64_t kApplyScan = 16 << 20;
constexpr int kScanSteps = 8;                        // 64-row steps of that scan in flight
constexpr int kFold = 8;                             // evicted rows a wave of merge_apply folds in at a time
constexpr int kScanPerWave = 2048;                  // cache rows a wave of merge_apply scans per round = capacity of its list

// Work item = (merging unit, 32 kept rows): 8 lanes per row.
template <int D>
__global__ __launch_bounds__(kThreads) void merge_norms(
    const UnitDesc* __restrict__ descs, const int32_t* __restrict__ list, const __bf16* __restrict__ k_out,
    float* __restrict__ inv_norm, int64_t ws_stride) {
  const UnitDesc d = descs[list[blockIdx.y]];
  const int b = d.n_out;
  const int r = blockIdx.x * kNormRows + (threadIdx.x >> 3), sub = threadIdx.x & 7;
  if (blockIdx.x * kNormRows >= b) return;
  // inverse norms of the kept keys (already gathered into the unit's output rows)
  constexpr int CPR = D / 8;
  float ss = 0.f;
  if (r < b) {
    const __bf16* row = k_out + (d.out_off + r) * D;
#pragma unroll
    for (int c = 0; c < CPR / 8; ++c) {
      const bf16x8 x = *reinterpret_cast<const bf16x8*>(row + (sub + 8 * c) * 8);
#pragma unroll
      for (int i = 0; i < 8; ++i) ss = fmaf((float)x[i], (float)x[i], ss);
    }
  }
  ss += __shfl_xor(ss, 1, 64);
  ss += __shfl_xor(ss, 2, 64);
  ss += __shfl_xor(ss, 4, 64);
  if (r < b && sub == 0) inv_norm[(int64_t)d.unit * ws_stride + r] = ss > 0.f ? 1.f / sqrtf(ss) : 0.f;
}

// Work item = (merging unit, 128 / PARTS rows of its uncompressed cache).  PARTS = 1: wave w takes rows [e0, e0 + 32) of
// them and meets every kept key; PARTS = 4: all waves take the same 32 rows and wave w meets every fourth block of the kept
// keys, the four results are combined through LDS.  The kept keys K^ (rows [out_off, out_off + b)) stream through LDS.
//
// A stage is copied, waited for and met at a barrier, so the walk is a chain of stages whose length a copy's latency sets
// while work-groups are few; four times as many work-groups of a quarter of the stages shorten it as long as the chip has room.
template <int D, int PARTS>
__global__ __launch_bounds__(kThreads, PARTS == 1 ? 4 : 1) void merge_nearest(
    const UnitDesc* __restrict__ descs, const int32_t* __restrict__ list, const __bf16* __restrict__ k_in,
    const __bf16* __restrict__ k_new, const __bf16* __restrict__ k_out, int N_k, const int32_t* __restrict__ kept_idx,
    int64_t idx_stride, const float* __restrict__ inv_norm, int32_t* __restrict__ nearest, float* __restrict__ weight,
    int64_t ws_stride) {
  using St = BlockStream<D, kWaves>;
  constexpr int KK = D / 16;
  constexpr int TILE = kNearRows / PARTS;
  constexpr int RING = PARTS == 1 ? kRing : kPartsRing;
  __shared__ __attribute__((aligned(1024))) __bf16 ring[RING][St::BLK];
  __shared__ __attribute__((aligned(256))) float inv_ring[RING][PARTS == 1 ? kWaves : 1][64];
  __shared__ int kept[TILE];
  const UnitDesc d = descs[list[blockIdx.y]];
  const int T = d.len_in + d.n_new, b = d.n_out;
  if ((int)blockIdx.x * TILE >= T) return;             // whole work-group past the end of this unit
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 31, half = lane >> 5;
  const int n_blocks = (b + 31) / 32;
  St st;
  st.init(k_out + d.out_off * D, b, &ring[0][0], lane, w);
  const float* inv_base = inv_norm + (int64_t)d.unit * ws_stride;
  const unsigned inv_lds = lds_addr_of(&inv_ring[0][0][0]);
  // the 32 inverse norms of block blk (a row past the end repeats the last one)
  auto issue_norms = [&](int blk, int at) {
    const int r = min(blk * 32 + (lane & 31), b - 1);
    load_to_lds_dword(inv_base, (unsigned)r * 4u, inv_lds + (unsigned)(at * 256));
  };
  // PARTS = 1: block blk and its norms (every wave copies the norms itself, so all waves issue the same number of copies)
  auto issue = [&](int blk) {
    st.issue(blk, blk % RING);
    issue_norms(blk, (blk % RING) * kWaves + w);
  };
  // PARTS = 4: the four blocks of stage s, of them as many as there are, and the norms of the one that this wave meets
  auto issue_stage = [&](int s) {
    const int slot = (s * 4) % RING;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (4 * s + i < n_blocks) st.issue(4 * s + i, slot + i);
    if (4 * s + w < n_blocks) issue_norms(4 * s + w, slot + w);
  };
  if constexpr (PARTS == 1) {
    issue(0);
    if (n_blocks > 1) issue(1);
  } else {
    issue_stage(0);
    if (n_blocks > 4) issue_stage(1);
  }
  // which rows of the tile are kept
  const int tile0 = blockIdx.x * TILE;
  if (threadIdx.x < TILE) kept[threadIdx.x] = 0;
  // this wave's candidate rows of the virtual concatenation [cached rows | new rows] (B operands);
  // a wave whose rows all lie past the end still takes part in the copies and barriers
  const int e0 = tile0 + (PARTS == 1 ? w * 32 : 0);
  bf16x8 ef[KK];
  const int e = min(e0 + col, T - 1);
  const __bf16* erow = (e < d.len_in) ? k_in + (d.in_off + e) * D : k_new + ((int64_t)d.unit * N_k + (e - d.len_in)) * D;
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) ef[kk] = *reinterpret_cast<const bf16x8*>(erow + 16 * kk + 8 * half);
  __syncthreads();                                        // the marks are clear
  const int32_t* idx = kept_idx + (int64_t)d.unit * idx_stride;
  for (int r0 = 0; r0 < b; r0 += kScanSteps * kThreads) {
    int at[kScanSteps];                                   // these steps' loads in flight together
#pragma unroll
    for (int u = 0; u < kScanSteps; ++u) at[u] = idx[min(r0 + u * kThreads + (int)threadIdx.x, b - 1)] - tile0;
#pragma unroll
    for (int u = 0; u < kScanSteps; ++u)
      if ((unsigned)at[u] < (unsigned)TILE) kept[at[u]] = 1;   // read behind the barriers of the loop below
  }
  float ss = 0.f;
#pragma unroll
  for (int kk = 0; kk < KK; ++kk)
#pragma unroll
    for (int i = 0; i < 8; ++i) ss = fmaf((float)ef[kk][i], (float)ef[kk][i], ss);
  ss = pair_sum(ss);
  const float inv_e = ss > 0.f ? 1.f / sqrtf(ss) : 0.f;
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) asm volatile("" ::"v"(ef[kk]));   // waited for here, not inside the loop

  float best = -INFINITY;   // largest dot(k_e, k_r) / |k_r| so far among this lane's kept rows
  int arg = 0;
  // One block against this lane's 16 kept rows: the block's largest value displaces the running best only if it
  // is strictly larger (an equal later row does not displace an earlier one), and among equal values of the block
  // the lowest row wins.  A short tree of maxima, then the lowest row that attains the maximum.
  auto update = [&](const floatx16& sc, const float* invs, int blk, int nv, bool ragged) {
    float v[16];
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      const float4 iv = *reinterpret_cast<const float4*>(invs + 8 * r4 + 4 * half);
      const float ivs[4] = {iv.x, iv.y, iv.z, iv.w};
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = 8 * r4 + 4 * half + i;            // = c_row(4 r4 + i, half): ascending in (r4, i)
        v[4 * r4 + i] = (ragged && row >= nv) ? -INFINITY : sc[4 * r4 + i] * ivs[i];
      }
    }
    float m4[4];
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) m4[g4] = fmaxf(fmaxf(v[4 * g4], v[4 * g4 + 1]), fmaxf(v[4 * g4 + 2], v[4 * g4 + 3]));
    const float vmax = fmaxf(fmaxf(m4[0], m4[1]), fmaxf(m4[2], m4[3]));
    const bool moved = vmax > best;
    if (__any(moved)) {                                   // the row is only looked for when some lane's best moved
      int first = 0;
#pragma unroll
      for (int q = 15; q >= 0; --q)                       // descending, so the lowest matching row is written last
        first = (v[q] == vmax) ? 8 * (q >> 2) + 4 * half + (q & 3) : first;
      best = moved ? vmax : best;
      arg = moved ? blk * 32 + first : arg;
    }
  };
  auto scores = [&](const __bf16* slot, floatx16& sc) {
#pragma unroll
    for (int r = 0; r < 16; ++r) sc[r] = 0.f;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
      sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lds_frag<D>(slot, col, half, kk), ef[kk], sc, 0, 0, 0);
  };
  // the ragged form (rows past the end masked) is a separate instance, taken by the last block only
  auto meet = [&](const floatx16& sc, const float* invs, int blk) {
    const int nv = min(32, b - blk * 32);
    if (nv == 32) update(sc, invs, blk, 32, false);
    else update(sc, invs, blk, nv, true);
  };
  if constexpr (PARTS == 1) {
    // A stage is two blocks of kept keys (one barrier per stage); while a stage is worked on, the copies of the
    // next one are in flight into the other two ring slots.
    for (int blk = 0; blk < n_blocks; blk += 2) {
      dma_wait_but<0>();                                    // this wave's copies of blocks blk, blk+1 have landed
      __syncthreads();                                      // ... and everybody's; the slots of blocks blk-2, blk-1 are free
      if (blk + 2 < n_blocks) issue(blk + 2);
      if (blk + 3 < n_blocks) issue(blk + 3);
      floatx16 s0, s1;
      const bool two = blk + 1 < n_blocks;                  // wave-uniform
      scores(&ring[blk % RING][0], s0);
      if (two) scores(&ring[(blk + 1) % RING][0], s1);
      meet(s0, &inv_ring[blk % RING][w][0], blk);
      if (two) meet(s1, &inv_ring[(blk + 1) % RING][w][0], blk + 1);
    }
  } else {
    // A stage is four blocks, one per wave; two stages are in flight behind the one that is worked on.
    for (int s = 0; 4 * s < n_blocks; ++s) {
      if (4 * (s + 2) <= n_blocks) dma_wait_but<4 * St::IPW + 1>();   // stage s + 1, whole, may be in flight
      else dma_wait_but<0>();
      __syncthreads();                                      // all of stage s is visible; the slots of stage s - 1 are free
      if (4 * (s + 2) < n_blocks) issue_stage(s + 2);
      const int blk = 4 * s + w, slot = (4 * s) % RING + w;
      if (blk < n_blocks) {                                 // wave-uniform
        floatx16 sc;
        scores(&ring[slot][0], sc);
        meet(sc, &inv_ring[slot][0][0], blk);
      }
    }
  }
  // Larger value wins, equal values go to the lower index, whatever the order: the partner lane holds the other 16 rows
  // of every block, the other waves (PARTS = 4) the other blocks.
  auto combine = [&](float best_o, int arg_o) {
    if (best_o > best || (best_o == best && arg_o < arg)) {
      best = best_o;
      arg = arg_o;
    }
  };
  combine(__builtin_bit_cast(float, pair_other(__builtin_bit_cast(unsigned, best))), (int)pair_other((unsigned)arg));
  if constexpr (PARTS > 1) {
    __shared__ float best_sh[kWaves][32];
    __shared__ int arg_sh[kWaves][32];
    if (half == 0) {
      best_sh[w][col] = best;
      arg_sh[w][col] = arg;
    }
    __syncthreads();
    if (w > 0) return;
#pragma unroll
    for (int o = 1; o < kWaves; ++o) combine(best_sh[o][col], arg_sh[o][col]);
  }
  const int ej = e0 + col;
  if (half == 0 && ej < T) {
    const bool keep = kept[ej - tile0] != 0;
    nearest[(int64_t)d.unit * ws_stride + ej] = keep ? -1 : arg;
    if (!keep) weight[(int64_t)d.unit * ws_stride + ej] = fmaxf(best * inv_e, 0.f);
  }
}

// Work item = (merging unit, ROWS kept rows from r0 on); wave w owns the ROWS / 4 from r0 + w ROWS / 4 on.
// Folding is a chain of loads per wave, as long as the rows that go to its kept rows are many: few kept rows per wave keep it
// short.  Every work-group scans the whole assignment, so their number is bounded by what all of them scan (kApplyScan).
template <int D, int ROWS>
__global__ __launch_bounds__(kThreads) void merge_apply(
    const UnitDesc* __restrict__ descs, const int32_t* __restrict__ list, const __bf16* __restrict__ k_in,
    const __bf16* __restrict__ v_in, const __bf16* __restrict__ k_new, const __bf16* __restrict__ v_new, int N_k,
    const int32_t* __restrict__ nearest, const float* __restrict__ weight, int64_t ws_stride,
    __bf16* __restrict__ k_out, __bf16* __restrict__ v_out, int cap) {
  constexpr int EPL = D / 64;                   // elements per lane
  constexpr int RPW = ROWS / kWaves;            // kept rows per wave
  static_assert(ROWS <= 32, "a list entry keeps the row's offset in 5 bits");
  // entry: (cache row - first row of the round) << 5 | (kept row - r0); each wave's list is ascending
  extern __shared__ uint32_t lst[];   // [kWaves][cap]
  __shared__ int cnt[kWaves];
  const UnitDesc d = descs[list[blockIdx.y]];
  const int T = d.len_in + d.n_new, b = d.n_out;
  const int r0 = blockIdx.x * ROWS;
  if (r0 >= b) return;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int32_t* nn = nearest + (int64_t)d.unit * ws_stride;
  const float* wt = weight + (int64_t)d.unit * ws_stride;
  float ak[RPW][EPL], av[RPW][EPL], wsum[RPW];
#pragma unroll
  for (int i = 0; i < RPW; ++i) {
    wsum[i] = 0.f;
#pragma unroll
    for (int x = 0; x < EPL; ++x) ak[i][x] = av[i][x] = 0.f;
  }
  // rows a wave scans per round: a quarter of the cache (in whole 64-row steps), at most its list's capacity
  const int per = min(cap, (T + 64 * kWaves - 1) / (64 * kWaves) * 64);
  for (int seg0 = 0; seg0 < T; seg0 += kWaves * per) {
    // wave w scans cache rows [seg0 + per w, + per): the rows assigned to one of this work-group's kept rows
    int n = 0;
    const int base = seg0 + w * per;
    for (int t0 = 0; t0 < per && base + t0 < T; t0 += kScanSteps * 64) {
      int v[kScanSteps];                                      // these steps' loads in flight together
#pragma unroll
      for (int u = 0; u < kScanSteps; ++u) {
        const int j = base + t0 + 64 * u + lane;
        v[u] = (t0 + 64 * u < per && j < T) ? nn[j] : -1;
      }
#pragma unroll
      for (int u = 0; u < kScanSteps; ++u) {
        const int j = base + t0 + 64 * u + lane;
        const unsigned rl = (unsigned)(v[u] - r0);            // kept (-1) and unassigned rows wrap to large values
        const bool hit = rl < (unsigned)ROWS;
        const unsigned long long m = __ballot(hit);
        if (hit) lst[w * cap + n + __builtin_popcountll(m & ((1ull << lane) - 1ull))] = ((unsigned)(j - seg0) << 5) | rl;
        n += __builtin_popcountll(m);
      }
    }
    if (lane == 0) cnt[w] = n;
    __syncthreads();
    // The lists of waves 0..3 one after the other are in ascending row order: a fixed summation order per kept
    // row.  A wave takes the entries of its RPW kept rows (2 or 8) kFold at a time, whatever rows they go to: the loads of all of
    // them are issued together, then each is added to its row.
    for (int q = 0; q < kWaves; ++q) {
      const int nq = cnt[q];
      for (int t0 = 0; t0 < nq; t0 += 64) {
        const bool in = t0 + lane < nq;
        const unsigned ent = in ? lst[q * cap + t0 + lane] : 0u;
        unsigned long long left = __ballot(in && (int)((ent & 31u) / RPW) == w);
        while (left) {
          static_assert(EPL == 1 || EPL == 2, "one or two elements per lane");
          float we[kFold];
          bf16x2 kx[kFold], vx[kFold];
          int to[kFold];                                      // kept row of the wave, -1: no entry left
#pragma unroll
          for (int i = 0; i < kFold; ++i) {
            to[i] = -1;
            if (left) {                                       // wave-uniform
              const unsigned x = __builtin_amdgcn_readlane(ent, __builtin_ctzll(left));
              left &= left - 1;
              to[i] = (int)(x & 31u) % RPW;
              const int e = seg0 + (int)(x >> 5);
              we[i] = wt[e];
              const bool cached = e < d.len_in;
              const int64_t row = cached ? d.in_off + e : (int64_t)d.unit * N_k + (e - d.len_in);
              const __bf16* kr = (cached ? k_in : k_new) + row * D + lane * EPL;
              const __bf16* vr = (cached ? v_in : v_new) + row * D + lane * EPL;
              if (EPL == 2) {
                kx[i] = *reinterpret_cast<const bf16x2*>(kr);
                vx[i] = *reinterpret_cast<const bf16x2*>(vr);
              } else {
                kx[i][0] = kr[0];
                vx[i][0] = vr[0];
              }
            }
          }
#pragma unroll
          for (int i = 0; i < kFold; ++i)
            if (to[i] >= 0 && we[i] >= 0.f)                   // wave-uniform; weights are >= 0
#pragma unroll
              for (int r = 0; r < RPW; ++r)
                if (to[i] == r) {
#pragma unroll
                  for (int x = 0; x < EPL; ++x) {
                    ak[r][x] = fmaf(we[i], (float)kx[i][x], ak[r][x]);
                    av[r][x] = fmaf(we[i], (float)vx[i][x], av[r][x]);
                  }
                  wsum[r] += we[i];
                }
        }
      }
    }
    __syncthreads();   // the lists are rewritten in the next round
  }
#pragma unroll
  for (int i = 0; i < RPW; ++i) {
    const int p = r0 + w * RPW + i;
    if (p < b && wsum[i] > 0.f) {      // nothing merged into a row: it stays bit for bit what the gather wrote
      const float inv = 1.f / (1.f + wsum[i]);
      __bf16* ko = k_out + (d.out_off + p) * D + lane * EPL;
      __bf16* vo = v_out + (d.out_off + p) * D + lane * EPL;
#pragma unroll
      for (int x = 0; x < EPL; ++x) {
        ko[x] = (__bf16)(((float)ko[x] + ak[i][x]) * inv);
        vo[x] = (__bf16)(((float)vo[x] + av[i][x]) * inv);
      }
    }
  }
}

template <int D>
void launch_t(hipStream_t s, const UnitDesc* descs, const int32_t* list, int n_list, int max_t_in, int max_out,
              const void* k_in, const void* v_in, const void* k_new, const void* v_new, int N_k, const int32_t* kept_idx,
              int64_t idx_stride, void* k_out, void* v_out, int32_t* nearest, float* weight, float* inv_norm,
              int64_t ws_stride) {
  typedef __bf16 T;
  hipLaunchKernelGGL(merge_norms<D>, dim3((max_out + kNormRows - 1) / kNormRows, n_list), dim3(kThreads), 0, s, descs, list,
                     (const T*)k_out, inv_norm, ws_stride);
#define HACK_NEAREST(PARTS_)                                                                                                   \
  hipLaunchKernelGGL((merge_nearest<D, PARTS_>), dim3((max_t_in + kNearRows / PARTS_ - 1) / (kNearRows / PARTS_), n_list),     \
                     dim3(kThreads), 0, s, descs, list, (const T*)k_in, (const T*)k_new, (const T*)k_out, N_k, kept_idx,       \
                     idx_stride, inv_norm, nearest, weight, ws_stride)
  if ((int64_t)((max_t_in + 31) / 32) * n_list <= kPartsGroups<D>) HACK_NEAREST(4);
  else HACK_NEAREST(1);
#undef HACK_NEAREST
  // list capacity of a wave of merge_apply: a quarter of the longest cache in whole 64-row steps, at most kScanPerWave
  const int cap = std::min(kScanPerWave, (max_t_in + 64 * kWaves - 1) / (64 * kWaves) * 64);
#define HACK_APPLY(ROWS_)                                                                                                   \
  hipLaunchKernelGGL((merge_apply<D, ROWS_>), dim3((max_out + ROWS_ - 1) / ROWS_, n_list), dim3(kThreads),                  \
                     (size_t)kWaves * cap * sizeof(uint32_t), s, descs, list, (const T*)k_in, (const T*)v_in, (const T*)k_new, \
                     (const T*)v_new, N_k, nearest, weight, ws_stride, (T*)k_out, (T*)v_out, cap)
  if ((int64_t)((max_out + 7) / 8) * n_list * max_t_in <= kApplyScan) HACK_APPLY(8);
  else HACK_APPLY(32);
#undef HACK_APPLY
}

}  // namespace

void launch_merge(hipStream_t s, int head_dim, const UnitDesc* descs, const int32_t* list, int n_list, int max_t_in,
                  int max_out, const void* k_in, const void* v_in, const void* k_new, const void* v_new, int N_k,
                  const int32_t* kept_idx, int64_t idx_stride, void* k_out, void* v_out, int32_t* nearest, float* weight,
                  float* inv_norm, int64_t ws_stride) {
  if (n_list <= 0 || max_out <= 0) return;
  if (head_dim == 64)
    launch_t<64>(s, descs, list, n_list, max_t_in, max_out, k_in, v_in, k_new, v_new, N_k, kept_idx, idx_stride, k_out,
                 v_out, nearest, weight, inv_norm, ws_stride);
  else
    launch_t<128>(s, descs, list, n_list, max_t_in, max_out, k_in, v_in, k_new, v_new, N_k, kept_idx, idx_stride, k_out,
                  v_out, nearest, weight, inv_norm, ws_stride);
}

}  // namespace hack
