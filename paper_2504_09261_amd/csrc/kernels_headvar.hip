// Attention variance of a head (Sec. 4.2, "Offline Head Classification via
// Attention Variance") on gfx950:
//     A = Softmax(scale * Q K^T)  (N_K queries x T_K keys, the final step over the
//     full cache),   sigma = sum_j Var_i(A[i, j])   (population variance).
// With c1_j = sum_i A_ij the sum of the column variances is
//     sigma = (1/N) sum_ij A_ij^2 - (1/N^2) sum_j c1_j^2,
// so no per-column state has to leave the chip: a first pass forms every query's
// softmax statistics (running maximum and normaliser), a second pass recomputes
// the scores tile by tile, turns them into probabilities and accumulates the sum
// of squares and each key's column sum.
//
// Both passes stream one operand (the keys in pass 1, the queries in pass 2) in
// 32-row blocks HBM -> LDS (global_load_lds, coalesced whole rows) through a ring
// shared by the four waves of a work-group, one barrier per block, and keep the
// other operand in registers: S^T = K Q^T with v_mfma_f32_32x32x16_bf16, so a
// lane owns one query column and 16 key rows.  (Fetching MFMA operands straight
// from global memory, one row per lane, runs the memory pipeline at a quarter of
// its coalesced rate.)  The sums that are subtracted from each other are kept in
// fp64.
//
// Both passes are bound by the matrix and the vector unit together: a pass needs per
// 32 x 32 scores 256 cycles of MFMA (D = 128) and 260 (pass 1) or 400 (pass 2) of
// vector work (an exponential takes 8).  Both therefore run one block ahead: a stage
// holds the MFMAs of block b + 1 and the softmax arithmetic of block b, interleaved by
// hand, one barrier a stage.  16 heads x batch 2, 4096 queries x 10521 keys, D = 128:
// pass 1 426 -> 365 us, pass 2 566 -> 475 us against blocks computed one after the other
// (under the profiler, which lengthens both), the call without it 873 -> 755 us.  Matrix cores 60 % busy in pass 1
// and 42 % in pass 2; the chip holds 1.67-1.74 GHz
// in this mix (power), so that fewer cycles buy less time than their share.  The
// steady loop holds no branch: with one, the compiler sinks the fp64 sums past it and spills.
#include <type_traits>

#include "device_util.h"
#include "hack_internal.h"

namespace hack {

namespace {

using namespace dev;

constexpr int kThreads = 256;          // 4 waves
constexpr int kWaves = 4;
constexpr int kRB1 = 2;                // 32-query blocks per wave in pass 1
constexpr int kRB2 = 2;                // 32-key blocks per wave in pass 2 (64 registers of fp64 sums per block)
constexpr int kTile1 = kWaves * 32 * kRB1;  // queries per work-group in pass 1
constexpr int kTile2 = kWaves * 32 * kRB2;  // keys per work-group in pass 2
constexpr int kRing = 4;               // LDS ring slots (32-row blocks)
constexpr float kFollowAbove = 256.f;  // pass 1: sum over 16 keys at which the reference follows the scores

// Element offset of MFMA operand fragment kk in a 32-row LDS slot: row col, chunk 2 kk + half.
template <int D>
__device__ __forceinline__ int frag_off(int col, int half, int kk) {
  return col * D + (((2 * kk + half) ^ swz_k<D>(col)) & (D / 8 - 1)) * 8;
}

// Pass 1: stats[(u*N_k + i)] = (m_i, sum_j 2^((s_ij - m_i) * c2)), s = raw dot product, c2 = scale*log2(e); m_i is a
// reference near the row's maximum: it follows the scores only when a block's sum exceeds kFollowAbove.
// A wave owns kRB1 blocks of 32 queries (registers); the keys stream through LDS.
template <int D>
__global__ __launch_bounds__(kThreads, 2) void hv_rowstats(
    const UnitDesc* __restrict__ descs, const __bf16* __restrict__ q, const __bf16* __restrict__ k_cache,
    int N_k, float scale, float2* __restrict__ stats, double* __restrict__ sigma) {
  using St = BlockStream<D, kWaves>;
  constexpr int KK = D / 16;
  __shared__ __attribute__((aligned(1024))) __bf16 ring[kRing][St::BLK];
  const UnitDesc d = descs[blockIdx.y];
  if (blockIdx.x == 0 && threadIdx.x == 0) sigma[d.unit] = 0.0;   // pass 2 adds to it (a launch that cleared it took 1 to 3 us)
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 31, half = lane >> 5;
  const int q0 = blockIdx.x * kTile1 + w * (32 * kRB1);   // may lie past N_k: the wave still copies and synchronises
  const int len = d.n_out;
  const int n_blocks = (len + 31) / 32, n_full = len / 32;
  St st;
  st.init(k_cache + d.out_off * D, len, &ring[0][0], lane, w);
  st.issue(0, 0);
  if (n_blocks > 1) st.issue(1, 1);
  if (n_blocks > 2) st.issue(2, 2);

  bf16x8 qf[kRB1][KK];
#pragma unroll
  for (int j = 0; j < kRB1; ++j) {
    // a block past the end repeats the last query; it is not stored
    const int qj = min(q0 + 32 * j, N_k - 1);
    load_frags<D>(q + ((int64_t)d.unit * N_k + qj) * D, min(32, N_k - qj), lane, qf[j]);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) asm volatile("" ::"v"(qf[j][kk]));   // waited for here, not inside the loop
  }
  int k_off[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) k_off[kk] = frag_off<D>(col, half, kk);
  const float c2 = scale * kLog2eF;
  float m[kRB1], mc[kRB1], l[kRB1];
#pragma unroll
  for (int j = 0; j < kRB1; ++j) l[j] = 0.f;

  auto scores = [&](const __bf16* slot, floatx16 (&sc)[kRB1]) {
#pragma unroll
    for (int j = 0; j < kRB1; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) sc[j][r] = 0.f;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const bf16x8 kf = *reinterpret_cast<const bf16x8*>(&slot[k_off[kk]]);
#pragma unroll
      for (int j = 0; j < kRB1; ++j) sc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[j][kk], sc[j], 0, 0, 0);
    }
  };
  auto mask = [&](floatx16 (&sc)[kRB1], int b) {   // rows of block b past the unit's end
    if ((b + 1) * 32 <= len) return;
#pragma unroll
    for (int j = 0; j < kRB1; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (b * 32 + c_row(r, half) >= len) sc[j][r] = -INFINITY;
  };
  auto block_max = [&](const floatx16& sc) {
    float mx = sc[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, sc[r]);
    return pair_max(mx);                       // finite: a block holds a valid key
  };
  auto block_sum = [&](const floatx16& sc, float ref) {
    float s0 = 0.f, s1 = 0.f;
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
      s0 += __builtin_amdgcn_exp2f(fmaf(sc[r], c2, -ref));
      s1 += __builtin_amdgcn_exp2f(fmaf(sc[r + 1], c2, -ref));
    }
    return s0 + s1;
  };
  // Stage b: on entry sc = scores of block b, on exit those of block b + 1 (unless b is the last block).
  // STEADY: blocks b + 1 .. b + 3 exist and are full.
  auto stage = [&](auto last_tag, auto steady_tag, int b, int next_slot, floatx16 (&sc)[kRB1]) __attribute__((always_inline)) {
    constexpr bool LAST = decltype(last_tag)::value, STEADY = decltype(steady_tag)::value;
    floatx16 sn[kRB1];
    if constexpr (!LAST) {
      if (STEADY || b + 2 < n_blocks) dma_wait_but<St::IPW>();   // this wave's part of block b + 1 has landed
      else dma_wait_but<0>();
      __syncthreads();                                // all of block b + 1 is visible; the slot of block b - 1 is free
      if (STEADY || b + 3 < n_blocks) st.issue(b + 3, (next_slot + 2) % kRing, STEADY);
      __builtin_amdgcn_sched_barrier(0);
    }
    // The order is fixed by hand: with each MFMA go the exponentials of a few scores and the sums of those before
    // them; operands are read two ahead.
    const __bf16* next = &ring[next_slot][0];
    constexpr int N = kRB1 * 16;       // scores per lane and block
    constexpr int STEPS = LAST ? N / 2 : kRB1 * KK;
    constexpr int PER = N / STEPS;     // scores per step
    float p[2][PER], part[kRB1][2] = {};
    bf16x8 kf[3];
    auto load_k = [&](int kk) { kf[kk % 3] = *reinterpret_cast<const bf16x8*>(&next[k_off[kk]]); };
    auto add_up = [&](int i) {
#pragma unroll
      for (int x = 0; x < PER; ++x) part[(i * PER + x) / 16][x & 1] += p[i & 1][x];
    };
    if constexpr (!LAST) {
      load_k(0);
      load_k(1);
#pragma unroll
      for (int j = 0; j < kRB1; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) sn[j][r] = 0.f;
    }
#pragma unroll
    for (int i = 0; i < STEPS; ++i) {
      if constexpr (!LAST) {
        const int kk = i / kRB1, j = i % kRB1;
        if (j == 0 && kk + 2 < KK) load_k(kk + 2);
        sn[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[kk % 3], qf[j][kk], sn[j], 0, 0, 0);
      }
#pragma unroll
      for (int x = 0; x < PER; ++x) {
        const int e = i * PER + x;
        p[i & 1][x] = __builtin_amdgcn_exp2f(fmaf(sc[e / 16][e % 16], c2, -mc[e / 16]));
      }
      if (i > 0) add_up(i - 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    add_up(STEPS - 1);
    float s[kRB1];
#pragma unroll
    for (int j = 0; j < kRB1; ++j) s[j] = part[j][0] + part[j][1];
    if (__any(!(fmaxf(s[0], s[kRB1 - 1]) < kFollowAbove))) {
#pragma unroll
      for (int j = 0; j < kRB1; ++j) {
        const float m_new = fmaxf(m[j], block_max(sc[j]));
        l[j] *= __builtin_amdgcn_exp2f((m[j] - m_new) * c2);
        m[j] = m_new;
        mc[j] = m_new * c2;
        s[j] = block_sum(sc[j], mc[j]);
      }
    }
#pragma unroll
    for (int j = 0; j < kRB1; ++j) l[j] += s[j];
    if constexpr (!LAST) {
      if (!STEADY) mask(sn, b + 1);
#pragma unroll
      for (int j = 0; j < kRB1; ++j) sc[j] = sn[j];
    }
  };

  dma_wait_but<0>();
  __syncthreads();
  floatx16 sc[kRB1];
  scores(&ring[0][0], sc);
  mask(sc, 0);
#pragma unroll
  for (int j = 0; j < kRB1; ++j) {
    m[j] = block_max(sc[j]);
    mc[j] = m[j] * c2;
  }
  int b = 0;
  for (; b + 6 < n_full; b += kRing) {
#pragma unroll
    for (int i = 0; i < kRing; ++i) stage(std::false_type{}, std::true_type{}, b + i, (i + 1) % kRing, sc);
  }
  for (; b + 1 < n_blocks; ++b) stage(std::false_type{}, std::false_type{}, b, (b + 1) % kRing, sc);
  stage(std::true_type{}, std::false_type{}, b, 0, sc);
#pragma unroll
  for (int j = 0; j < kRB1; ++j) {
    const float lj = pair_sum(l[j]);
    const int qi = q0 + 32 * j + col;
    if (half == 0 && qi < N_k) stats[(int64_t)d.unit * N_k + qi] = make_float2(m[j], lj);
  }
}

// Pass 2: sigma[u] += (1/N) sum_ij p_ij^2 - (1/N^2) sum_j (sum_i p_ij)^2 over this work-group's keys.
// A wave owns kRB2 blocks of 32 keys (registers); the queries and their pass-1
// statistics stream through LDS (every wave copies the 256 bytes of statistics
// of a block itself, so all waves issue the same number of copies per block).
template <int D>
__global__ __launch_bounds__(kThreads, 2) void hv_colmoments(
    const UnitDesc* __restrict__ descs, const __bf16* __restrict__ q, const __bf16* __restrict__ k_cache,
    int N_k, float scale, const float2* __restrict__ stats, double* __restrict__ sigma) {
  using St = BlockStream<D, kWaves>;
  constexpr int KK = D / 16;
  __shared__ __attribute__((aligned(1024))) __bf16 ring[kRing][St::BLK];
  __shared__ __attribute__((aligned(256))) float2 st_ring[kRing][kWaves][32];
  const UnitDesc d = descs[blockIdx.y];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 31, half = lane >> 5;
  const int len = d.n_out;
  if ((int)blockIdx.x * kTile2 >= len) return;   // whole work-group past the end of this unit
  const int t0 = blockIdx.x * kTile2 + w * (32 * kRB2);
  const int n_blocks = (N_k + 31) / 32, n_full = N_k / 32;
  St st;
  st.init(q + (int64_t)d.unit * N_k * D, N_k, &ring[0][0], lane, w);
  const float* stat_base = reinterpret_cast<const float*>(stats + (int64_t)d.unit * N_k);
  const unsigned st_lds = lds_addr_of(&st_ring[0][0][0]);
  // block b of the queries and its statistics: lane l copies float l of the
  // block's 64 (a query past the end repeats the last one; it is masked below)
  auto issue = [&](int b, int slot, bool full = false) {
    st.issue(b, slot, full);
    const int qi = min(b * 32 + (lane >> 1), N_k - 1);
    load_to_lds_dword(stat_base, (unsigned)(qi * 2 + (lane & 1)) * 4u, st_lds + (unsigned)((slot * kWaves + w) * 256));
  };
  issue(0, 0);
  if (n_blocks > 1) issue(1, 1);
  if (n_blocks > 2) issue(2, 2);

  // a wave whose keys all lie past the end of the unit still takes part in the copies and barriers
  bf16x8 kf[kRB2][KK];
  int nv[kRB2];
#pragma unroll
  for (int j = 0; j < kRB2; ++j) {
    const int tj = min(t0 + 32 * j, len - 1);   // a block past the end repeats the last key; nv = 0 leaves it out
    nv[j] = max(0, min(32, len - (t0 + 32 * j)));
    load_frags<D>(k_cache + (d.out_off + tj) * D, max(1, min(32, len - tj)), lane, kf[j]);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) asm volatile("" ::"v"(kf[j][kk]));   // waited for here, not inside the loop
  }
  int q_off[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) q_off[kk] = frag_off<D>(col, half, kk);
  const float c2 = scale * kLog2eF;
  double c1[kRB2][16];                 // per key row: sum_i p_ij over this lane's queries
  double s2[kRB2][2];                  // sum of p_ij^2 over this lane's queries and valid key rows
#pragma unroll
  for (int j = 0; j < kRB2; ++j) {
#pragma unroll
    for (int r = 0; r < 16; ++r) c1[j][r] = 0.0;
    s2[j][0] = s2[j][1] = 0.0;
  }
  auto scores = [&](const __bf16* slot, floatx16 (&sc)[kRB2]) {
#pragma unroll
    for (int j = 0; j < kRB2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) sc[j][r] = 0.f;
    // every query fragment feeds the MFMAs of all kRB2 key blocks and is then dropped
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const bf16x8 qf = *reinterpret_cast<const bf16x8*>(&slot[q_off[kk]]);
#pragma unroll
      for (int j = 0; j < kRB2; ++j) sc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[j][kk], qf, sc[j], 0, 0, 0);
    }
  };
  // p = 2^(s c2 - (m c2 + log2 l)): the normaliser rides in the exponent; queries past the end give 2^-inf = 0
  auto exponent = [&](float2 ml, int b, bool full) {
    const float e = fmaf(ml.x, c2, __builtin_amdgcn_logf(ml.y));
    return (full || b * 32 + col < N_k) ? e : INFINITY;
  };
  float mc = 0.f;   // of the block whose moments are next
  // Stage b as in pass 1: the scores of block b + 1 beside the moments of block b.  RAGGED: some of the wave's
  // keys lie past the unit's end; their probabilities are replaced by zero.
  auto stage = [&](auto last_tag, auto steady_tag, auto ragged_tag, int b, int slot, floatx16 (&sc)[kRB2]) __attribute__((always_inline)) {
    constexpr bool LAST = decltype(last_tag)::value, STEADY = decltype(steady_tag)::value, RAGGED = decltype(ragged_tag)::value;
    floatx16 sn[kRB2];
    if constexpr (!LAST) {
      if (STEADY || b + 2 < n_blocks) dma_wait_but<St::IPW + 1>();   // this wave's copies of block b + 1 have landed
      else dma_wait_but<0>();
      __syncthreads();                                      // all of block b + 1 is visible; the slot of block b - 1 is free
      if (STEADY || b + 3 < n_blocks) issue(b + 3, (slot + 3) % kRing, STEADY);
      __builtin_amdgcn_sched_barrier(0);
    }
    float2 ml;
    if constexpr (!LAST) ml = st_ring[(slot + 1) % kRing][w][col];
    // The order is fixed by hand (left to itself the scheduler forms every probability first and spills): with each
    // MFMA go the exponentials of two scores and the fp64 sums of the two before them; operands are read two ahead.
    const __bf16* next = &ring[(slot + 1) % kRing][0];
    constexpr int N = kRB2 * 16;       // scores per lane and block
    constexpr int STEPS = LAST ? N / 2 : kRB2 * KK;
    constexpr int PER = N / STEPS;     // scores per step
    float pf[2][PER];
    bf16x8 qf[3];
    auto load_q = [&](int kk) { qf[kk % 3] = *reinterpret_cast<const bf16x8*>(&next[q_off[kk]]); };
    auto add_up = [&](int i) {         // moments of the scores of step i
#pragma unroll
      for (int x = 0; x < PER; ++x) {
        const int e = i * PER + x, j = e / 16, r = e % 16;
        const double p = (double)pf[i & 1][x];
        c1[j][r] += p;
        s2[j][r & 1] = fma(p, p, s2[j][r & 1]);
      }
    };
    if constexpr (!LAST) {
      load_q(0);
      load_q(1);
#pragma unroll
      for (int j = 0; j < kRB2; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) sn[j][r] = 0.f;
    }
#pragma unroll
    for (int i = 0; i < STEPS; ++i) {
      if constexpr (!LAST) {
        const int kk = i / kRB2, j = i % kRB2;
        if (j == 0 && kk + 2 < KK) load_q(kk + 2);
        sn[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[j][kk], qf[kk % 3], sn[j], 0, 0, 0);
      }
#pragma unroll
      for (int x = 0; x < PER; ++x) {
        const int e = i * PER + x, j = e / 16, r = e % 16;
        pf[i & 1][x] = __builtin_amdgcn_exp2f(fmaf(sc[j][r], c2, -mc));
        if (RAGGED && c_row(r, half) >= nv[j]) pf[i & 1][x] = 0.f;
      }
      if (i > 0) add_up(i - 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    add_up(STEPS - 1);
    if constexpr (!LAST) {
#pragma unroll
      for (int j = 0; j < kRB2; ++j) sc[j] = sn[j];
      mc = exponent(ml, b + 1, STEADY);
    }
  };
  auto walk = [&](auto ragged_tag) __attribute__((always_inline)) {
    dma_wait_but<0>();
    __syncthreads();
    floatx16 sc[kRB2];
    scores(&ring[0][0], sc);
    mc = exponent(st_ring[0][w][col], 0, false);
    int b = 0;
    for (; b + 6 < n_full; b += kRing) {
#pragma unroll
      for (int i = 0; i < kRing; ++i) stage(std::false_type{}, std::true_type{}, ragged_tag, b + i, i, sc);
    }
    for (; b + 1 < n_blocks; ++b) stage(std::false_type{}, std::false_type{}, ragged_tag, b, b % kRing, sc);
    stage(std::true_type{}, std::false_type{}, ragged_tag, b, b % kRing, sc);
  };
  // the choice is the work-group's, so that all four waves meet at the same barriers
  if ((int)(blockIdx.x + 1) * kTile2 <= len) walk(std::false_type{});
  else walk(std::true_type{});

  // a half-wave holds 32 different queries of the same 16 key rows
  const double inv_n = 1.0 / (double)N_k;
  double acc = 0.0;
#pragma unroll
  for (int j = 0; j < kRB2; ++j) {
    acc += half_sum_f64(s2[j][0] + s2[j][1]) * inv_n;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const double c = half_sum_f64(c1[j][r]) * inv_n;
      acc = fma(-c, c, acc);   // all keys together: sum_j Var_i(A[i, j])
    }
  }
  // What the rounding of the two totals can leave where there is next to no variance: one query has none at all, and
  // a sum of variances is not negative.  (NaN stays NaN.)
  if (N_k == 1 || acc < 0.0) acc -= acc;
  if (col == 0 && t0 < len) atomicAdd(&sigma[d.unit], acc);
}

}  // namespace

void launch_head_variance(hipStream_t s, int head_dim, const UnitDesc* descs, int n_desc, int max_len, const void* q,
                          const void* k_cache, int N_k, float scale, float* stats, double* sigma) {
  if (n_desc <= 0) return;
  typedef __bf16 T;
  const dim3 g1((N_k + kTile1 - 1) / kTile1, n_desc), g2((max_len + kTile2 - 1) / kTile2, n_desc);
  if (head_dim == 64) {
    hipLaunchKernelGGL(hv_rowstats<64>, g1, dim3(kThreads), 0, s, descs, (const T*)q, (const T*)k_cache, N_k, scale,
                       (float2*)stats, sigma);
    hipLaunchKernelGGL(hv_colmoments<64>, g2, dim3(kThreads), 0, s, descs, (const T*)q, (const T*)k_cache, N_k, scale,
                       (const float2*)stats, sigma);
  } else {
    hipLaunchKernelGGL(hv_rowstats<128>, g1, dim3(kThreads), 0, s, descs, (const T*)q, (const T*)k_cache, N_k, scale,
                       (float2*)stats, sigma);
    hipLaunchKernelGGL(hv_colmoments<128>, g2, dim3(kThreads), 0, s, descs, (const T*)q, (const T*)k_cache, N_k,
                       scale, (const float2*)stats, sigma);
  }
}

}  // namespace hack
