// Attention of the current scale's queries over the ragged compressed cache
// (Preliminaries, attention equation: O = Softmax(scale * Q K^T) V, no mask
// inside a scale step) on gfx950.
//
// bf16, flash-style: one pass over K/V with an online softmax; a work item is a unit and 128 queries, four waves of 32, which share every
// block of 32 keys through LDS.  S^T = K Q^T and O^T += V^T P^T, so that a lane owns query columns: the softmax reductions are in-lane plus an
// exchange between lanes that hold the same query, the probabilities go from the accumulator registers straight into the B operand,
// and V^T comes from row-major V through the transposing LDS read (ds_read_b64_tr_b16).  K/V blocks travel HBM -> LDS directly (no
// register round trip) through a ring of four slots per tensor.
//   * attn_pipe, which serves the launches: 16x16x32 matrix instructions, scores, softmax and PV product of three blocks side by side.
//   * attn_mfma, a second implementation that tests and A/B timings select (HACK_ATTN_PIPE=0): 32x32x16 matrix instructions, one block ahead.
#include <cfloat>
#include <type_traits>

#include "device_util.h"
#include "hack_internal.h"

namespace hack {

namespace {

using namespace dev;

// ---------------------------------------------------------------------------
// bf16 MFMA path
// ---------------------------------------------------------------------------
constexpr int kKB = 32;      // keys per block (one LDS ring slot)
constexpr float kRescaleAbove = 65536.f;  // a block sum of probabilities at or above this moves the reference

// NW waves per work-group, each wave owns 32 queries; two work-groups share a CU.  The accumulator of v_mfma_f32_32x32x16_bf16 holds one query
// column and 16 key rows a lane, the other 16 are lane ^ 32's; registers 8s .. 8s+7 are two runs of four consecutive keys (C rows
// 8(r/4)+4h+r%4), the order in which V^T is read.  A swizzle of 16-byte chunks keeps both LDS reads free of bank conflicts.
//
// The loop runs over 32-key blocks and is software-pipelined by one block: while
// the vector ALU turns the scores of block b into probabilities, the matrix core
// already forms the scores of block b+1; then O^T += V^T P^T for block b.  (A
// wave issues in order, so matrix and vector work only overlap if independent
// instructions of both kinds sit next to each other in its own stream; on this
// chip ~4 simple VALU ops or ~2 exponentials hide under one 32x32x16 MFMA.)
// K and V blocks travel HBM -> LDS through two rings of kRing slots: the copy of
// block b+3 is issued at stage b into the slot block b-1 has just left, so a
// copy has two full stages to land and one barrier per stage both publishes
// block b+1 and frees the slot.
//
// The vector ALU is the scarce unit (per block a wave issues 16 MFMAs but also
// has to exponentiate 16 scores per lane), so the softmax is kept to
// fma + exp2 + bf16 pack + a bf16 dot2 for the row sum:
//   * the running reference m_run is only moved when a probability would leave
//     [0, 2^16): the exponentials are formed optimistically against the current
//     reference, and only if some lane's block sum says "too large" (or inf, as
//     in the very first block) is the max computed and everything rescaled;
//   * the row sum is taken over the bf16-rounded probabilities, the same numbers
//     the PV product uses.
constexpr int kRing = 4;     // LDS ring slots per tensor (32-key blocks)

template <int D, int NW>
__global__ __launch_bounds__(64 * NW, 2) void attn_mfma(
    const UnitDesc* __restrict__ descs, const AttnItem* __restrict__ items,
    const __bf16* __restrict__ q, const __bf16* __restrict__ k_cache,
    const __bf16* __restrict__ v_cache, int N_k, float scale,
    __bf16* __restrict__ out) {
  constexpr int KK = D / 16;        // MFMA steps over head_dim for S^T
  constexpr int MB = D / 32;        // 32-row blocks of O^T
  constexpr int CPR = D / 8;        // 16-byte chunks per row
  constexpr int RPI = 64 / CPR;     // block rows covered by one wave-wide copy instruction
  constexpr int IPW = (kKB / RPI) / NW;  // copy instructions per wave, block and tensor
  constexpr int BLK = kKB * D;      // elements per block and tensor
  static_assert(IPW >= 1, "a block must give every wave at least one copy instruction");

  const AttnItem it = items[blockIdx.x];
  if (it.desc < 0) return;
  const AttnItem& d = it;   // the item carries the descriptor fields read here
  const int len = d.n_out;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 31, half = lane >> 5;

  __shared__ __attribute__((aligned(1024))) __bf16 Ks[kRing][BLK];
  __shared__ __attribute__((aligned(1024))) __bf16 Vs[kRing][BLK];

  const __bf16* kg = k_cache + d.out_off * D;
  const __bf16* vg = v_cache + d.out_off * D;
  const int n_blocks = (len + kKB - 1) / kKB;

  // Block copies.  Lane l of copy instruction i of this wave fills LDS row
  // r = (w + i NW) RPI + l / CPR, chunk position c = l % CPR, from global chunk
  // c ^ f(r) of block row r; the byte offsets inside a full block are loop invariant.
  unsigned k_src[IPW], v_src[IPW];
#pragma unroll
  for (int i = 0; i < IPW; ++i) {
    const int r = (w + i * NW) * RPI + lane / CPR, c = lane % CPR;
    k_src[i] = (unsigned)(r * D + ((c ^ swz_k<D>(r)) & (CPR - 1)) * 8) * 2u;
    v_src[i] = (unsigned)(r * D + ((c ^ swz_v<D>(r)) & (CPR - 1)) * 8) * 2u;
  }
  const unsigned ks_lds = lds_addr_of(&Ks[0][0]), vs_lds = lds_addr_of(&Vs[0][0]);
  // Rows past the end of a ragged last block repeat the last valid row (finite
  // data); their scores are masked to -inf, so their probabilities are exactly 0.
  auto issue = [&](int b, int slot) {
    const int t0 = b * kKB;
    const __bf16* kb = kg + (int64_t)t0 * D;
    const __bf16* vb = vg + (int64_t)t0 * D;
    if (t0 + kKB <= len) {
#pragma unroll
      for (int i = 0; i < IPW; ++i) {
        const unsigned dst = (unsigned)((slot * BLK + (w + i * NW) * 512) * 2);
        load_to_lds(kb, k_src[i], ks_lds + dst);
        load_to_lds(vb, v_src[i], vs_lds + dst);
      }
    } else {
#pragma unroll
      for (int i = 0; i < IPW; ++i) {
        const int r = (w + i * NW) * RPI + lane / CPR, c = lane % CPR;
        const int rc = min(r, len - 1 - t0);
        const unsigned dst = (unsigned)((slot * BLK + (w + i * NW) * 512) * 2);
        load_to_lds(kb, (unsigned)(rc * D + ((c ^ swz_k<D>(r)) & (CPR - 1)) * 8) * 2u, ks_lds + dst);
        load_to_lds(vb, (unsigned)(rc * D + ((c ^ swz_v<D>(r)) & (CPR - 1)) * 8) * 2u, vs_lds + dst);
      }
    }
  };
  issue(0, 0);
  if (n_blocks > 1) issue(1, 1);
  if (n_blocks > 2) issue(2, 2);

  // Q fragments (B operand of S^T = K Q^T): query col, head-dim slice [16kk + 8h, +8).
  const int q0 = it.q_tile * (NW * 32) + w * 32;
  bf16x8 qf[KK];
  {
    const int qi = min(q0 + col, N_k - 1);
    const __bf16* qrow = q + ((int64_t)d.unit * N_k + qi) * D;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) qf[kk] = *reinterpret_cast<const bf16x8*>(qrow + 16 * kk + 8 * half);
    // Consume the fragments here so that their loads are waited for before the
    // main loop: a vmcnt wait inside the loop would also drain the block copies
    // that are meant to stay in flight.
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) asm volatile("" ::"v"(qf[kk]));
  }

  floatx16 o[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[mb][r] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  const float c2 = scale * kLog2eF;
  float mc = -INFINITY;   // m_run * c2

  // per-lane LDS element offsets of the operand reads (block-relative); the ring
  // slot is a compile-time immediate
  int k_off[KK];           // K operand: row col, chunk 2kk + half
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) k_off[kk] = col * D + (((2 * kk + half) ^ swz_k<D>(col)) & (CPR - 1)) * 8;
  const int g = lane >> 4, e = (lane >> 2) & 3, qd = lane & 3;
  int v_off[MB];           // V^T operand: row 4 half + e (+16 sg, +8), head-dim 32mb + 16(g&1) + 4qd
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
    v_off[mb] = (4 * half + e) * D + (((4 * mb + 2 * (g & 1) + (qd >> 1)) ^ swz_v<D>(e)) & (CPR - 1)) * 8 + 4 * (qd & 1);

  const bf16x2 ones2 = {(__bf16)1.0f, (__bf16)1.0f};

  // S^T of block b (32 keys x 32 queries) from ring slot SLOT.
  auto scores = [&](auto slot_tag, int b) -> floatx16 {
    constexpr int SLOT = decltype(slot_tag)::value;
    const __bf16* Kt = &Ks[SLOT][0];
    floatx16 sc;
#pragma unroll
    for (int r = 0; r < 16; ++r) sc[r] = 0.f;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const bf16x8 kf = *reinterpret_cast<const bf16x8*>(&Kt[k_off[kk]]);
      sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[kk], sc, 0, 0, 0);
    }
    return sc;
  };
  // ragged end: keys past the end get -inf
  auto mask_tail = [&](floatx16& sc, int b) {
    if ((b + 1) * kKB > len) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int key = b * kKB + 8 * (r >> 2) + 4 * half + (r & 3);
        if (key >= len) sc[r] = -INFINITY;
      }
    }
  };
  // probabilities of a block against the current reference (per lane: one query,
  // 16 keys; the partner lane l ^ 32 holds the other 16) and their sum
  auto probs = [&](const floatx16& sc, bf16x8 (&pf)[2]) -> float {
    float psum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) pf[r >> 3][r & 7] = (__bf16)__builtin_amdgcn_exp2f(fmaf(sc[r], c2, -mc));
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
      const bf16x2 pr = {pf[r >> 3][r & 7], pf[r >> 3][(r & 7) + 1]};
      psum = __builtin_amdgcn_fdot2_f32_bf16(pr, ones2, psum, false);
    }
    return psum;
  };
  // Some probability left the safe range (always so in the first block, where the
  // reference is -inf): move the reference to the running max, bring the
  // accumulators to the new scale and redo this block's probabilities.
  auto rescale = [&](const floatx16& sc, bf16x8 (&pf)[2]) -> float {
    float mx = sc[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, sc[r]);
    mx = pair_max(mx);
    const float m_new = fmaxf(m_run, mx);   // finite: the block holds a valid key
    const float a = __builtin_amdgcn_exp2f((m_run - m_new) * c2);
    l_run *= a;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int r = 0; r < 16; ++r) o[mb][r] *= a;
    m_run = m_new;
    mc = m_new * c2;
    return probs(sc, pf);
  };
  // O^T += V^T P^T for the block in ring slot SLOT
  auto pv = [&](auto slot_tag, const bf16x8 (&pf)[2]) {
    constexpr int SLOT = decltype(slot_tag)::value;
    const __bf16* Vt = &Vs[SLOT][0];
#pragma unroll
    for (int sg = 0; sg < 2; ++sg) {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        const __bf16* vp = &Vt[16 * sg * D + v_off[mb]];
        const bf16x4 v0 = lds_read_tr(vp);
        const bf16x4 v1 = lds_read_tr(vp + 8 * D);
        bf16x8 vf;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          vf[i] = v0[i];
          vf[4 + i] = v1[i];
        }
        o[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, pf[sg], o[mb], 0, 0, 0);
      }
    }
  };

  // Stage b (ring slot S = b % kRing): sc holds the scores of block b on entry
  // and those of block b+1 on exit.  LAST: block b is the unit's last one.
  // TAIL: block b+1 may be the ragged last block (its scores then need the mask,
  // whose branch would keep the scheduler from mixing matrix and vector work).
  auto stage = [&](auto slot_tag, auto last_tag, auto tail_tag, int b, floatx16& sc) {
    constexpr int S = decltype(slot_tag)::value;
    constexpr bool LAST = decltype(last_tag)::value;
    constexpr bool TAIL = decltype(tail_tag)::value;
    using S1 = std::integral_constant<int, (S + 1) % kRing>;
    // everything but the copy group issued one stage ago (block b+2) has landed
    if (b + 2 < n_blocks) dma_wait_but<2 * IPW>();
    else dma_wait_but<0>();
    __syncthreads();   // block b+1 is visible to every wave; the slot of block b-1 is free
    if (b + 3 < n_blocks) issue(b + 3, (S + 3) % kRing);
    __builtin_amdgcn_sched_barrier(0);
    floatx16 sn;
    if (!LAST) sn = scores(S1{}, b + 1);
    bf16x8 pf[2];
    float psum = probs(sc, pf);
    if (!LAST) {
      // the K fragment reads first, then one MFMA of the next block's scores and a
      // slice of this block's softmax arithmetic, and so on
      __builtin_amdgcn_sched_group_barrier(0x100, KK, 0);
#pragma unroll
      for (int i = 0; i < KK; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 48 / KK, 0);
      }
    }
    if (!LAST && TAIL) mask_tail(sn, b + 1);
    if (__any(!(psum < kRescaleAbove))) psum = rescale(sc, pf);
    l_run += psum;
    pv(slot_tag, pf);
    if (!LAST) sc = sn;
  };

  using R0 = std::integral_constant<int, 0>;
  using R1 = std::integral_constant<int, 1>;
  using R2 = std::integral_constant<int, 2>;
  using R3 = std::integral_constant<int, 3>;
  using No = std::false_type;
  using Yes = std::true_type;

  // block 0 has landed -> its scores
  if (n_blocks > 2) dma_wait_but<4 * IPW>();
  else if (n_blocks > 1) dma_wait_but<2 * IPW>();
  else dma_wait_but<0>();
  __syncthreads();
  floatx16 sc = scores(R0{}, 0);
  mask_tail(sc, 0);

  // main loop: four stages whose next blocks are all full
  int b = 0;
  for (; b + 5 < n_blocks; b += 4) {
    stage(R0{}, No{}, No{}, b, sc);
    stage(R1{}, No{}, No{}, b + 1, sc);
    stage(R2{}, No{}, No{}, b + 2, sc);
    stage(R3{}, No{}, No{}, b + 3, sc);
  }
  // the remaining 1..5 blocks, one stage at a time (b is a multiple of 4 here)
  for (; b < n_blocks; ++b) {
    const bool last = (b + 1 == n_blocks);
    switch (b & 3) {
      case 0: if (last) stage(R0{}, Yes{}, Yes{}, b, sc); else stage(R0{}, No{}, Yes{}, b, sc); break;
      case 1: if (last) stage(R1{}, Yes{}, Yes{}, b, sc); else stage(R1{}, No{}, Yes{}, b, sc); break;
      case 2: if (last) stage(R2{}, Yes{}, Yes{}, b, sc); else stage(R2{}, No{}, Yes{}, b, sc); break;
      default: if (last) stage(R3{}, Yes{}, Yes{}, b, sc); else stage(R3{}, No{}, Yes{}, b, sc); break;
    }
  }

  // ---- normalise and store: lane holds query col, head-dim rows 32mb + 8(r/4) + 4h + r%4 ----
  const float l = pair_sum(l_run);
  const float inv = 1.f / l;
  const int qi = q0 + col;
  if (qi < N_k) {
    __bf16* orow = out + ((int64_t)d.unit * N_k + qi) * D;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
      for (int r4 = 0; r4 < 4; ++r4) {
        bf16x4 pk;
#pragma unroll
        for (int i = 0; i < 4; ++i) pk[i] = (__bf16)(o[mb][4 * r4 + i] * inv);
        *reinterpret_cast<bf16x4*>(orow + 32 * mb + 8 * r4 + 4 * half) = pk;
      }
    }
  }
}


// ---------------------------------------------------------------------------
// bf16 MFMA path, deeper software pipeline (the kernel that serves the large steps)
// ---------------------------------------------------------------------------
// The work item of attn_mfma above, with 16x16x32 MFMAs: the chip runs these launches at its power limit, where the bare 16x16x32
// instruction on random operands sustains 2.07 PFLOP/s (at 2.03 GHz) and the 32x32x16 one 1.83 (at 1.78 GHz).  A wave holds 32 queries as two
// tiles of 16, S^T of a block as 2x2 tiles: a lane has one query column and four keys of each, P^T goes from the accumulators into the B operand of
// O^T += V^T P^T in that order of keys, and V^T is read from LDS in the same order.  Row sums are one more tile of that product, with a V^T of ones
// (the bf16-rounded probabilities, summed in float32): between MFMAs a bf16 dot product adds 17 cycles, a multiply-add half a cycle.
// A stage (one barrier) holds three independent strands:
//     S(b+1)   the score MFMAs of the next block          (matrix core)
//     PV(b-1)  O^T += V^T P^T of the previous block       (matrix core)
//     softmax(b): multiply-adds, exponentials, packing    (vector ALU)
// in slots of one MFMA, one LDS read and a share of the vector work, in the order written: an MFMA takes 8 cycles of the issue port that
// vector instructions share and leaves 8 of its 16, so work that bunches up stands still in the matrix core.  Operands are read a step
// (eight slots) ahead, across stages too.
// The probabilities of block b wait in registers for one stage; the check "did a probability leave the safe range" travels beside
// the last MFMAs, and the rare rescale that follows it sits at the end of the stage, after PV(b-1) has been added, so a rescale
// always meets accumulators that are complete up to block b-1.
// LDS: four slots per tensor.  K(j) is read from the end of stage j-2 on through stage j-1, V(j) from the end of stage j on through
// stage j+1.  The barrier in the middle of stage b publishes K(b+2) and V(b); behind it the copies K(b+4) and V(b+2) go into the
// slots of K(b) and V(b-2), which every wave finished reading in stage b-1.  Each copy has two stages to land.
// Measured, us a launch of whole items, 32x32x16 in a three-slot ring / this: head_dim 128, 32 units of 4096 queries over 10521 keys 613 / 568
// (1.24 PFLOP/s), 128 units of 4096 over 3010 or 6020 1226 / 1120, 64 units of 4096 over 1579 or 4735 384 / 356, 32 units of 4096 over 1943 or 3885
// 205 / 187; 576 queries over 1497 31.9 / 29.7.  Counters at the first of them: 1021 / 983 thousand shader cycles (747 a stage and SIMD, the matrix core
// busy in 73 % of them, 66 % before), so 1.67 / 1.73 GHz.  Of this, at the first two: with the order of a stage left to the compiler 580 and 1141, with row
// sums by dot products 574 and 1147.  The accumulators pass a branch in every stage and must not be cut into pieces there (compiled without
// -amdgpu-codegenprepare-break-large-phis=false they do not fit the registers: 8840 us).

// Reference: 2^15 above the running maximum, so that the exponent's top bit says that a probability reached 2 (or inf, as in the very
// first block): bf16 and float32 keep their precision down to 2^-126, 2^-111 of a row's largest probability.
constexpr float kHeadroom = 15.f;

// The vector work of a stage: 16 scores a lane become probabilities; conversions take two of them.  Listed in the order of issue with
// a fixed distance between dependent operations, and dealt out over the stage's MFMAs by their issue time.
struct SoftmaxOp {
  enum Kind { kFma, kExp, kPack } kind;
  int index;   // element; of a pack, the first of two
};
struct SoftmaxOrder {
  static constexpr int kOps = 40, kCycles = 16 * 4 + 16 * 8 + 8 * 4;
  SoftmaxOp op[kOps];
  constexpr SoftmaxOrder() : op() {
    int n = 0;
    op[n++] = SoftmaxOp{SoftmaxOp::kFma, 0};
    op[n++] = SoftmaxOp{SoftmaxOp::kFma, 1};
    for (int j = 0; j < 16; ++j) {
      op[n++] = SoftmaxOp{SoftmaxOp::kExp, j};
      if (j + 2 < 16) op[n++] = SoftmaxOp{SoftmaxOp::kFma, j + 2};
      if (j >= 2 && j % 2 == 0) op[n++] = SoftmaxOp{SoftmaxOp::kPack, j - 2};
    }
    op[n++] = SoftmaxOp{SoftmaxOp::kPack, 14};
  }
  // operations in front of MFMA slot s of n
  static constexpr int before(int s, int n) {
    if (s >= n) return kOps;
    const SoftmaxOrder o;
    int c = 0, t = 0;
    while (t < kOps) {
      c += o.op[t].kind == SoftmaxOp::kExp ? 8 : 4;
      if (c * n > kCycles * s) break;
      ++t;
    }
    return t;
  }
};
constexpr SoftmaxOrder kSoftmaxOrder;

template <int I, int N, typename F>
__device__ __forceinline__ void for_range(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    for_range<I + 1, N>(f);
  }
}

// STREAM = false: work-group i serves work item items[i] (one query tile of one unit, all of its keys).
// STREAM = true: work-group i serves the segments segs[seg_begin[i] .. seg_begin[i+1]), one after the
// other.  A segment is a run of 32-key blocks [blk0, blk1) of one work item; the host cuts the
// concatenation of all work items of a launch into as many equal runs as the device holds work-groups
// at once, so every work-group gets the same number of blocks whatever the lengths of the units are.
// A segment that covers its work item completely stores the output rows as usual (part < 0).
// Otherwise it leaves its reference, normaliser and unnormalised O^T (float32) in slot `part` of the
// partial-result arrays and draws a ticket from the work item's counter; the work-group that draws
// the last of the item's n_parts tickets (every other part has been stored and published by then)
// adds the parts first_part .. first_part + n_parts - 1 up and stores the output rows, then leaves the
// counter at zero for the next launch.  Nobody waits for anybody.
//
// KS = 2: two groups of NW waves hold the same queries and walk the two halves of the unit's blocks, each through rings of
// its own but from the same barriers, and exchange half of their unnormalised O^T through LDS at the end: a lone
// work-group's stage is a chain of latencies that two waves a SIMD overlap.  128 KiB of LDS, so one work-group a compute unit.
template <int D, int NW, int KS, bool STREAM>
__global__ __launch_bounds__(64 * NW * KS, 2) void attn_pipe(
    const UnitDesc* __restrict__ descs, const AttnItem* __restrict__ items,
    const AttnSeg* __restrict__ segs, const int32_t* __restrict__ seg_begin,
    const __bf16* __restrict__ q, const __bf16* __restrict__ k_cache,
    const __bf16* __restrict__ v_cache, int N_k, float scale,
    __bf16* __restrict__ out, float* part_o, float* part_ml, unsigned* part_count) {
  constexpr int KC = D / 32;        // MFMA steps over head_dim for S^T
  constexpr int MT = D / 16;        // 16-row tiles of O^T
  constexpr int RPI = 512 / D;      // block rows covered by one wave-wide copy instruction
  constexpr int IPW = (kKB / RPI) / NW;  // copy instructions per wave, block and tensor
  constexpr int BLK = kKB * D;      // elements per block and tensor
  constexpr int NS = 4;             // ring slots per tensor
  static_assert(IPW >= 1, "a block must give every wave at least one copy instruction");
  static_assert(KS == 1 || (KS == 2 && !STREAM), "whole work items only when the keys are split");

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int w = KS == 1 ? wave : wave % NW, ks = KS == 1 ? 0 : wave / NW;   // 32 queries and half of the keys of this wave

  __shared__ __attribute__((aligned(1024))) __bf16 K_ring[KS][NS][BLK];
  __shared__ __attribute__((aligned(1024))) __bf16 V_ring[KS][NS][BLK];
  __bf16 (&Ks)[NS][BLK] = K_ring[ks];
  __bf16 (&Vs)[NS][BLK] = V_ring[ks];
  __shared__ float2 ml_sh[KS == 2 ? 2 * NW * 32 : 1];
  __shared__ int last_ticket;

  int seg_lo = blockIdx.x, seg_hi = blockIdx.x + 1;
  if (STREAM) {
    seg_lo = seg_begin[blockIdx.x];
    seg_hi = seg_begin[blockIdx.x + 1];
  }
  for (int si = seg_lo; si < seg_hi; ++si) {
  // The lane index is re-read per segment behind a compiler barrier: values derived from it that
  // only the ragged paths need are then formed where they are used instead of being carried
  // through the main loop in registers.
  int lane = tid & 63;
  if (STREAM) asm volatile("" : "+v"(lane));
  const int col = lane & 15, g = lane >> 4;
  AttnSeg sg;
  AttnItem d;      // unit, n_out, out_off of the work item
  if (STREAM) {
    sg = segs[si];
    const UnitDesc ud = descs[sg.desc];
    d.unit = ud.unit; d.n_out = ud.n_out; d.out_off = ud.out_off;
  } else {
    d = items[si];
    if (d.desc < 0) return;
    sg = AttnSeg{d.desc, d.q_tile, 0, 0x3fffffff, -1, 0, 0, 0};
  }
  if (KS == 2) {   // the first half of the blocks, the larger one if they are odd, and the rest (the host sees to it that there is one)
    const int h = ((d.n_out + kKB - 1) / kKB + 1) / 2;
    sg.blk0 = ks == 0 ? 0 : h;
    sg.blk1 = ks == 0 ? h : 0x3fffffff;
  }
  const int key0 = sg.blk0 * kKB;                                               // first key of the segment
  const int len = (int)min((int64_t)sg.blk1 * kKB, (int64_t)d.n_out) - key0;    // its keys

  const __bf16* kg = k_cache + (d.out_off + key0) * D;
  const __bf16* vg = v_cache + (d.out_off + key0) * D;
  const int n_blocks = (len + kKB - 1) / kKB;
  // LDS layout of a block: rows in groups of four, a group's 64-byte pieces row after row (piece c of row r at
  // (r / 4) 8D + 256 c + 64 (r % 4)), the 16-byte chunks of a piece permuted by the group: chunk x holds x ^ (group & 3) in K and
  // x ^ 2 (group & 1) in V.  A phase of the V reads (8 rows x 32 bytes) then covers all banks; a phase of the K reads takes four lanes each of
  // all four groups, two of them at the same chunks (SQ_LDS_BANK_CONFLICT a third of SQ_LDS_IDX_ACTIVE; with x ^ (group & 2 ? 3 : 0) none, and no
  // faster: 580 us for 578 over 10521 keys).  The lanes of a copy read whole 64-byte pieces, and all operands of a block stand at constant distances
  // from one address in K and two in V.
  // The copy instructions of a block are 16 rows apart: same lane offsets, another base.
  static_assert(IPW == 1 || NW * RPI == 16, "lane offsets are those of the first instruction");
  constexpr int GPI = RPI / 4;                     // groups of four rows covered by one copy instruction
  auto copy_src = [&](int ln, int first_row, int n_rows, bool is_v) -> unsigned {   // lane ln's source in the copy from first_row on
    const int cg = w * GPI + (GPI == 2 ? ln >> 5 : 0), row = min(first_row + 4 * cg + ((ln >> 2) & 3), n_rows - 1);
    const int flip = is_v ? 2 * (cg & 1) : cg & 3;
    return (unsigned)(row * D + (4 * ((ln >> 4) & (D / 32 - 1)) + ((ln & 3) ^ flip)) * 8) * 2u;
  };
  unsigned k_src[IPW], v_src[IPW];
#pragma unroll
  for (int i = 0; i < IPW; ++i) {
    k_src[i] = copy_src(lane, i * (NW * RPI), kKB, false);
    v_src[i] = copy_src(lane, i * (NW * RPI), kKB, true);
  }
  const unsigned ks_lds = lds_addr_of(&Ks[0][0]), vs_lds = lds_addr_of(&Vs[0][0]);
  // Block 0 is the unit's last one, ragged or not, blocks 1 .. n_blocks - 1 are the full ones in front of it: what is particular about
  // a ragged block (rows past the end repeat the last valid row, their scores are masked to -inf) stays in front of the main loop.
  // Copies past the last block repeat it into slots that nobody reads any more, so that every stage issues and awaits as many.
  const unsigned last_full = (unsigned)max(n_blocks - 2, 0);
  unsigned k_at = 0, v_at = 0;             // the next blocks to copy (their byte offsets do not fit 32 bits)
  auto issue_next = [&](const __bf16* base, unsigned& at, const unsigned (&src)[IPW], unsigned lds, int slot) {
    const __bf16* gb = base + (uint64_t)at * BLK;
#pragma unroll
    for (int i = 0; i < IPW; ++i) load_to_lds(gb, src[i], lds + (unsigned)((slot * BLK + (w + i * NW) * 512) * 2));
    at = min(at + 1, last_full);
  };
  auto issue_k = [&](int slot) { issue_next(kg, k_at, k_src, ks_lds, slot); };
  auto issue_v = [&](int slot) { issue_next(vg, v_at, v_src, vs_lds, slot); };
  {
    const int t0 = (n_blocks - 1) * kKB;
#pragma unroll
    for (int i = 0; i < IPW; ++i) {
      load_to_lds(kg + (int64_t)t0 * D, copy_src(lane, i * (NW * RPI), len - t0, false), ks_lds + (unsigned)((w + i * NW) * 1024));
      load_to_lds(vg + (int64_t)t0 * D, copy_src(lane, i * (NW * RPI), len - t0, true), vs_lds + (unsigned)((w + i * NW) * 1024));
    }
  }
  if (n_blocks > 1) {
    issue_k(1);
    issue_k(2);
    issue_k(3);
    issue_v(1);
  }

  // Q fragments (B operand of S^T = K Q^T): query 16 qt + col, head-dim slice [32kc + 8g, +8).
  const int q0 = sg.q_tile * (NW * 32) + w * 32;
  bf16x8 qf[2][KC];
#pragma unroll
  for (int qt = 0; qt < 2; ++qt) {
    const int qi = min(q0 + 16 * qt + col, N_k - 1);
    const __bf16* qrow = q + ((int64_t)d.unit * N_k + qi) * D;
#pragma unroll
    for (int kc = 0; kc < KC; ++kc) qf[qt][kc] = *reinterpret_cast<const bf16x8*>(qrow + 32 * kc + 8 * g);
  }
  // Consumed here so that their loads are waited for before the main loop (a vmcnt
  // wait inside the loop would also drain the block copies meant to stay in flight).
  // The copies issued above are older than these loads and have landed with them.
#pragma unroll
  for (int kc = 0; kc < KC; ++kc) asm volatile("" ::"v"(qf[0][kc]), "v"(qf[1][kc]));

  floatx4 o[MT][2];        // O^T: head-dim 16mt + 4g + r, query 16qt + col
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) o[mt][0] = o[mt][1] = floatx4{0.f, 0.f, 0.f, 0.f};
  floatx4 ls[2] = {floatx4{0.f, 0.f, 0.f, 0.f}, floatx4{0.f, 0.f, 0.f, 0.f}};   // row sums of P (equal in all four rows)
  const float c2 = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, scale * kLog2eF)));
  // Reference: probabilities are 2^(c2 s - mc).  Finite from the start: keys whose score is -inf get a probability of 0 also where nothing
  // else has been seen, and whatever finite score comes first is far too large for it.
  float mc[2] = {-FLT_MAX, -FLT_MAX};

  const int e = col >> 2, qd = col & 3;
  const int k_off = e * 4 * D + (col & 3) * 32 + (g ^ e) * 8;   // K operand: row 16kt + col, chunk 4kc + g
  // V^T operand: rows 4g + e and 16 + 4g + e, head-dim 16mt + 4qd; even and odd mt
  const int v_even = g * 4 * D + e * 32 + (2 * (g & 1) + (qd >> 1)) * 8 + 4 * (qd & 1), v_odd = v_even ^ 16;
  bf16x8 ones;
#pragma unroll
  for (int j = 0; j < 8; ++j) ones[j] = (__bf16)1.0f;
  asm volatile("" : "+v"(ones));   // stays in registers

  // Scores of a block: sc[kt][qt], keys 16kt + 4g + r, query 16qt + col.
  struct Scores { floatx4 t[2][2]; };
  // Probabilities of a block's 32 keys for one query column, in the order of the B operand of the PV product: element j of lane
  // group g is key 4g + j (j < 4) or 16 + 4g + j - 4, and the V^T operand is read in the same order.
  auto probs = [&](const Scores& sc, int qt, bf16x8& pf) {
#pragma unroll
    for (int j = 0; j < 8; ++j) pf[j] = (__bf16)__builtin_amdgcn_exp2f(fmaf(sc.t[j >> 2][qt][j & 3], c2, -mc[qt]));
  };
  // Some probability reached 2 (or is inf, as in the very first block): the exponent field's top bit is set
  auto too_large = [&](const bf16x8 (&pf)[2]) -> bool {
    const uintx4 a = __builtin_bit_cast(uintx4, pf[0]), b = __builtin_bit_cast(uintx4, pf[1]);
    return (((a[0] | a[1] | a[2]) | a[3] | b[0]) | b[1] | b[2] | b[3]) & 0x40004000u;
  };
  auto rescale = [&](const Scores& sc, bf16x8 (&pf)[2]) {
#pragma unroll
    for (int qt = 0; qt < 2; ++qt) {
      float mx = sc.t[0][qt][0];
#pragma unroll
      for (int j = 1; j < 8; ++j) mx = fmaxf(mx, sc.t[j >> 2][qt][j & 3]);
      const float m_new = fmaxf(mc[qt], fmaf(quad_max(mx), c2, kHeadroom));
      const float a = __builtin_amdgcn_exp2f(mc[qt] - m_new);
      mc[qt] = m_new;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        ls[qt][r] *= a;
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) o[mt][qt][r] *= a;
      }
      probs(sc, qt, pf[qt]);
    }
  };
  auto k_frag = [&](const __bf16* Kt, int kt, int kc) -> bf16x8 { return *reinterpret_cast<const bf16x8*>(&Kt[16 * kt * D + 128 * kc + k_off]); };
  auto v_half = [&](const __bf16* Vt, int mt, int h) -> bf16x4 {   // keys 16h + 4g ..
    return lds_read_tr(&Vt[16 * h * D + 128 * (mt >> 1) + (mt & 1 ? v_odd : v_even)]);
  };
  // Operands of step i of a stage: head-dim slice i of S^T and two head-dim tiles of O^T.  Four tiles each, one operand of an MFMA kept for the next.
  struct Frags {
    bf16x8 k[2];
    bf16x4 v[2][2];
  };
  auto load_frag = [&](Frags& f, const __bf16* Kt, const __bf16* Vt, int i, int part) {   // one LDS read, parts 0 .. 5
    if (part < 2) f.k[part] = k_frag(Kt, part, i);
    else f.v[(part >> 1) - 1][part & 1] = v_half(Vt, 2 * i + (part >> 1) - 1, part & 1);
  };
  auto joined = [](const bf16x4 (&v)[2]) { return bf16x8{v[0][0], v[0][1], v[0][2], v[0][3], v[1][0], v[1][1], v[1][2], v[1][3]}; };
  auto qk = [&](Scores& sn, const Frags& f, int kc, int n) {
    const int kt = n >> 1, qt = kt ^ (n & 1);
    sn.t[kt][qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.k[kt], qf[qt][kc], sn.t[kt][qt], 0, 0, 0);
  };
  auto pv = [&](const Frags& f, const bf16x8 (&p)[2], int i, int n) {
    const int m = n >> 1, qt = m ^ (n & 1);
    o[2 * i + m][qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(joined(f.v[m]), p[qt], o[2 * i + m][qt], 0, 0, 0);
  };
  auto row_sums = [&](const bf16x8 (&p)[2], int qt) { ls[qt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, p[qt], ls[qt], 0, 0, 0); };

  bf16x8 P[2][2];   // probabilities of block b in P[b & 1]: those of the previous block wait for their PV product
  Frags pre;      // operands of the next stage's first step

  // Stage b, ring slot S = b % 4 (compile time).  On entry sc = scores of block b and
  // pp = probabilities of block b-1; on exit sc = scores of block b+1, pp = those of block b.
  // FIRST: b == 0 (no previous block).
  auto stage = [&](auto slot_tag, auto first_tag, Scores& sc) {
    constexpr int S = decltype(slot_tag)::value;
    constexpr bool FIRST = decltype(first_tag)::value;
    const __bf16* const Kt = &Ks[(S + 1) % NS][0];
    const __bf16* const Vt = &Vs[(S + 3) % NS][0];
    Scores sn;
#pragma unroll
    for (int i = 0; i < 4; ++i) sn.t[i >> 1][i & 1] = floatx4{0.f, 0.f, 0.f, 0.f};
    bf16x8 (&pp)[2] = P[(S + 1) & 1], (&pf)[2] = P[S & 1];
    Frags f = pre, nx;
    float x[16];
    auto vec_op = [&](auto t_tag) {
      constexpr SoftmaxOp op = kSoftmaxOrder.op[decltype(t_tag)::value];
      constexpr int j = op.index, qt = (j >> 3) & 1, jj = j & 7;
      if constexpr (op.kind == SoftmaxOp::kFma) x[j] = fmaf(sc.t[jj >> 2][qt][jj & 3], c2, -mc[qt]);
      else if constexpr (op.kind == SoftmaxOp::kExp) x[j] = __builtin_amdgcn_exp2f(x[j]);
      else { pf[qt][jj] = (__bf16)x[j]; pf[qt][jj + 1] = (__bf16)x[j + 1]; }
    };
    constexpr int SLOTS = 8 * KC + 2, VEC_SLOTS = SLOTS - 3 * KC / 4;   // the vector work ends early: its test travels beside the last MFMAs
    bool large = false;
    // one MFMA, one LDS read, a share of the vector work
    auto slot = [&](auto s_tag) {
      constexpr int T = decltype(s_tag)::value, I = T / 8 < KC ? T / 8 : KC - 1, N = T - 8 * I;   // the last step has two more
      // one wait for both K operands (lgkmcnt(4)) and one for both of V^T (lgkmcnt(2)) instead of one for each
      if constexpr (N == 0) __builtin_amdgcn_s_waitcnt(0xC47F);
      if constexpr (N == 4) __builtin_amdgcn_s_waitcnt(0xC27F);
      if constexpr (N < 4) qk(sn, f, I, N);
      else if constexpr (N < 8) { if (!FIRST) pv(f, pp, I, N - 4); }
      else { if (!FIRST) row_sums(pp, N - 8); }
      for_range<SoftmaxOrder::before(T, VEC_SLOTS), SoftmaxOrder::before(T + 1, VEC_SLOTS)>(vec_op);
      if constexpr (T == VEC_SLOTS) large = __any(too_large(pf));
      if constexpr (N < 2 || (N >= 4 && N < 8)) {
        constexpr int P = N < 2 ? N : N - 2;
        if constexpr (I + 1 < KC) load_frag(nx, Kt, Vt, I + 1, P);
        else load_frag(nx, &Ks[(S + 2) % NS][0], &Vs[S][0], 0, P);
      }
      if constexpr (N == 7 && I + 1 < KC) f = nx;
      __builtin_amdgcn_sched_barrier(0);
    };
    for_range<0, 4 * KC>(slot);
    wait_and_sync<2 * IPW>();   // K(b+2) and V(b) have landed: everything but what the previous stage issued
    issue_k(S);              // K(b+4)
    issue_v((S + 2) % NS);   // V(b+2)
    __builtin_amdgcn_sched_barrier(0);
    for_range<4 * KC, SLOTS>(slot);
    pre = nx;
    if (__builtin_expect(large, 0)) rescale(sc, pf);
    sc = sn;
  };

  // block 0 has landed (see the Q fragments above) -> its scores
  dma_wait_but<0>();
  __syncthreads();
  Scores sc;
#pragma unroll
  for (int i = 0; i < 4; ++i) sc.t[i >> 1][i & 1] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int kc = 0; kc < KC; ++kc) {
    Frags f;
    for (int n = 0; n < 2; ++n) load_frag(f, &Ks[0][0], nullptr, kc, n);
    for (int n = 0; n < 4; ++n) qk(sc, f, kc, n);
  }
  for (int n = 0; n < 2; ++n) load_frag(pre, &Ks[1][0], nullptr, 0, n);
  for (int n = 2; n < 6; ++n) load_frag(pre, nullptr, &Vs[0][0], 0, n);
#pragma unroll
  for (int kt = 0; kt < 2; ++kt)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if ((n_blocks - 1) * kKB + 16 * kt + 4 * g + r >= len) sc.t[kt][0][r] = sc.t[kt][1][r] = -INFINITY;

  using No = std::false_type;
  using Yes = std::true_type;
  if (n_blocks > 1) {
    stage(std::integral_constant<int, 0>{}, Yes{}, sc);
    for (int b = 1;; b += 4) {
      if (b >= n_blocks - 1) break;
      stage(std::integral_constant<int, 1>{}, No{}, sc);
      if (b + 1 >= n_blocks - 1) break;
      stage(std::integral_constant<int, 2>{}, No{}, sc);
      if (b + 2 >= n_blocks - 1) break;
      stage(std::integral_constant<int, 3>{}, No{}, sc);
      if (b + 3 >= n_blocks - 1) break;
      stage(std::integral_constant<int, 0>{}, No{}, sc);
    }
  }
  // the last block: its probabilities, its PV product and the one of the block before
  auto pv_block = [&](const __bf16* Vt, const bf16x8 (&p)[2]) {
#pragma unroll
    for (int i = 0; i < KC; ++i) {
      Frags f;
      for (int n = 2; n < 6; ++n) load_frag(f, nullptr, Vt, i, n);
      for (int n = 0; n < 4; ++n) pv(f, p, i, n);
    }
    row_sums(p, 0);
    row_sums(p, 1);
  };
  if (n_blocks > 1) {
    const bool odd = n_blocks & 1;   // the block before the last has an odd number
    const bf16x8 pl[2] = {odd ? P[1][0] : P[0][0], odd ? P[1][1] : P[0][1]};
    pv_block(&Vs[(n_blocks - 2) % NS][0], pl);
  }
  wait_and_sync<0>();
  probs(sc, 0, P[0][0]);
  probs(sc, 1, P[0][1]);
  if (__any(too_large(P[0]))) rescale(sc, P[0]);
  pv_block(&Vs[(n_blocks - 1) % NS][0], P[0]);

  // ---- normalise and store: a lane holds head-dim 16mt + 4g .. +4 of queries 16qt + col ----
  float l[2] = {ls[0][0], ls[1][0]};
  if constexpr (KS == 2) {
    // The waves (w, 0) and (w, 1) hold the same queries over the two halves of the keys: each adds up and stores half of
    // the head-dim, what the other one needs goes through the rings, which nobody reads any more.
    if (ks == 1 && (((d.n_out + kKB - 1) / kKB) & 1)) __syncthreads();   // this half had one stage less
    constexpr int HT = MT / 2;   // head-dim tiles of a half
    float4* const xo = reinterpret_cast<float4*>(ks == 0 ? &K_ring[0][0][0] : &V_ring[0][0][0]) + w * HT * 2 * 64 + lane;
    const float4* const xi = reinterpret_cast<const float4*>(ks == 0 ? &V_ring[0][0][0] : &K_ring[0][0][0]) + w * HT * 2 * 64 + lane;
    __syncthreads();
    if (g < 2) ml_sh[wave * 32 + 16 * g + col] = make_float2(g ? mc[1] : mc[0], g ? l[1] : l[0]);
    auto finish = [&](auto half_tag) {
      constexpr int MINE = decltype(half_tag)::value * HT, THEIRS = HT - MINE;
#pragma unroll
      for (int m = 0; m < HT; ++m)
#pragma unroll
        for (int qt = 0; qt < 2; ++qt)
          xo[(m * 2 + qt) * 64] = make_float4(o[THEIRS + m][qt][0], o[THEIRS + m][qt][1], o[THEIRS + m][qt][2], o[THEIRS + m][qt][3]);
      __syncthreads();
#pragma unroll
      for (int qt = 0; qt < 2; ++qt) {
        const float2 ml = ml_sh[(wave ^ NW) * 32 + 16 * qt + col];
        const float M = fmaxf(mc[qt], ml.x);
        float f = __builtin_amdgcn_exp2f(mc[qt] - M), h = __builtin_amdgcn_exp2f(ml.x - M);
        const float inv = 1.f / fmaf(f, l[qt], h * ml.y);
        f *= inv;
        h *= inv;
        const int qi = q0 + 16 * qt + col;
        __bf16* orow = out + ((int64_t)d.unit * N_k + min(qi, N_k - 1)) * D;
#pragma unroll
        for (int m = 0; m < HT; ++m) {
          const float4 x = xi[(m * 2 + qt) * 64];
          bf16x4 pk;
          pk[0] = (__bf16)fmaf(h, x.x, f * o[MINE + m][qt][0]);
          pk[1] = (__bf16)fmaf(h, x.y, f * o[MINE + m][qt][1]);
          pk[2] = (__bf16)fmaf(h, x.z, f * o[MINE + m][qt][2]);
          pk[3] = (__bf16)fmaf(h, x.w, f * o[MINE + m][qt][3]);
          if (qi < N_k) *reinterpret_cast<bf16x4*>(orow + 16 * (MINE + m) + 4 * g) = pk;
        }
      }
    };
    if (ks == 0) finish(std::integral_constant<int, 0>{});
    else finish(std::integral_constant<int, 1>{});
    return;
  }
  bool store = true;
  if (STREAM && sg.part >= 0) {
    // Partial result, register-major (every store instruction of a wave writes 512 contiguous bytes).
    // The parts of a work item come from work-groups on different XCDs, whose L2 caches are not kept
    // coherent with each other, so parts and tickets travel as device-scope relaxed atomics (stores
    // that write through, loads that do not take a stale line), 8 bytes each; a device-scope fence
    // would instead write back and invalidate the whole L2 at every segment end.  Order is kept by
    // hand: a work-group draws its ticket only after every store of its part has been acknowledged.
    constexpr int QT = NW * 32;
    typedef unsigned long long u64;
    auto pack2 = [](float a, float b) -> u64 {
      return (u64)__builtin_bit_cast(unsigned, a) | ((u64)__builtin_bit_cast(unsigned, b) << 32);
    };
    {
      u64* po = reinterpret_cast<u64*>(part_o + (int64_t)sg.part * (QT * D)) + (w * MT * 4) * 64 + lane;
#pragma unroll
      for (int i = 0; i < MT * 4; ++i)
        __hip_atomic_store(po + i * 64, pack2(o[i >> 2][(i >> 1) & 1][2 * (i & 1)], o[i >> 2][(i >> 1) & 1][2 * (i & 1) + 1]),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (g < 2)   // reference in log2 units and normaliser
        __hip_atomic_store(reinterpret_cast<u64*>(part_ml + (int64_t)sg.part * (2 * QT)) + w * 32 + 16 * g + col,
                           pack2(g ? mc[1] : mc[0], g ? l[1] : l[0]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this thread's stores have been acknowledged
    __syncthreads();                                    // ... and so have the whole work-group's
    if (tid == 0)
      last_ticket = (__hip_atomic_fetch_add(&part_count[sg.counter], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                     (unsigned)(sg.n_parts - 1)) ? 1 : 0;
    __syncthreads();
    store = last_ticket != 0;
    if (store) {
      // every other part was acknowledged before its ticket was drawn, and all tickets before this one
      auto part_ml_of = [&](int p, int qt) -> u64 {
        return __hip_atomic_load(reinterpret_cast<const u64*>(part_ml + (int64_t)(sg.first_part + p) * (2 * QT)) + w * 32 + 16 * qt + col,
                                 __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      };
      float M[2] = {-INFINITY, -INFINITY};
      for (int p = 0; p < sg.n_parts; ++p)
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) M[qt] = fmaxf(M[qt], __builtin_bit_cast(float, (unsigned)part_ml_of(p, qt)));
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) o[mt][0] = o[mt][1] = floatx4{0.f, 0.f, 0.f, 0.f};
      l[0] = l[1] = 0.f;
      for (int p = 0; p < sg.n_parts; ++p) {   // in slot order: the sum does not depend on who adds it up
        float f[2];
#pragma unroll
        for (int qt = 0; qt < 2; ++qt) {
          const u64 ml = part_ml_of(p, qt);
          f[qt] = __builtin_amdgcn_exp2f(__builtin_bit_cast(float, (unsigned)ml) - M[qt]);
          l[qt] = fmaf(f[qt], __builtin_bit_cast(float, (unsigned)(ml >> 32)), l[qt]);
        }
        const u64* po = reinterpret_cast<const u64*>(part_o + (int64_t)(sg.first_part + p) * (QT * D)) + (w * MT * 4) * 64 + lane;
#pragma unroll
        for (int i = 0; i < MT * 4; ++i) {
          const int mt = i >> 2, qt = (i >> 1) & 1, r = 2 * (i & 1);
          const u64 v2 = __hip_atomic_load(po + i * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          o[mt][qt][r] = fmaf(f[qt], __builtin_bit_cast(float, (unsigned)v2), o[mt][qt][r]);
          o[mt][qt][r + 1] = fmaf(f[qt], __builtin_bit_cast(float, (unsigned)(v2 >> 32)), o[mt][qt][r + 1]);
        }
      }
      if (tid == 0)   // as the next launch expects it
        __hip_atomic_store(&part_count[sg.counter], 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
#pragma unroll
  for (int qt = 0; qt < 2; ++qt) {
    const float inv = 1.f / l[qt];
    const int qi = q0 + 16 * qt + col;
    if (store && qi < N_k) {
      __bf16* orow = out + ((int64_t)d.unit * N_k + qi) * D;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        bf16x4 pk;
#pragma unroll
        for (int r = 0; r < 4; ++r) pk[r] = (__bf16)(o[mt][qt][r] * inv);
        *reinterpret_cast<bf16x4*>(orow + 16 * mt + 4 * g) = pk;
      }
    }
  }
  if (STREAM && si + 1 < seg_hi) __syncthreads();   // every wave has left the ring before the next segment refills it
  }  // segments
}

}  // namespace


template <int D, int NW>
static void launch_mfma_t(hipStream_t s, const UnitDesc* descs, const AttnItem* items, int n_items,
                          const void* q, const void* k_cache, const void* v_cache, int N_k,
                          float scale, void* out, int kernel) {
  typedef __bf16 T;
  if constexpr (D == 128) {
    if (kernel == kAttnHalves) {
      hipLaunchKernelGGL((attn_pipe<D, NW, 2, false>), dim3(n_items), dim3(128 * NW), 0, s, descs, items, nullptr, nullptr,
                         (const T*)q, (const T*)k_cache, (const T*)v_cache, N_k, scale, (T*)out, nullptr, nullptr, nullptr);
      return;
    }
  }
  if (kernel != kAttnPlain)
    hipLaunchKernelGGL((attn_pipe<D, NW, 1, false>), dim3(n_items), dim3(64 * NW), 0, s, descs, items, nullptr, nullptr,
                       (const T*)q, (const T*)k_cache, (const T*)v_cache, N_k, scale, (T*)out, nullptr, nullptr, nullptr);
  else
    hipLaunchKernelGGL((attn_mfma<D, NW>), dim3(n_items), dim3(64 * NW), 0, s, descs, items,
                       (const T*)q, (const T*)k_cache, (const T*)v_cache, N_k, scale, (T*)out);
}

void launch_attn(hipStream_t s, int head_dim, const UnitDesc* descs, const AttnItem* items, int n_items, const void* q,
                 const void* k_cache, const void* v_cache, int N_k, float scale, void* out, int bf16_kernel) {
  if (n_items <= 0) return;
  if (head_dim == 64) launch_mfma_t<64, 4>(s, descs, items, n_items, q, k_cache, v_cache, N_k, scale, out, bf16_kernel);
  else launch_mfma_t<128, 4>(s, descs, items, n_items, q, k_cache, v_cache, N_k, scale, out, bf16_kernel);
}

// Work-groups of the streamed bf16 kernel that the current device holds at once.
int attn_stream_slots(int head_dim) {
  int dev = 0, cus = 0, blocks = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  const hipError_t e = head_dim == 64
      ? hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, attn_pipe<64, 4, 1, true>, 256, 0)
      : hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, attn_pipe<128, 4, 1, true>, 256, 0);
  if (e != hipSuccess) return 0;
  return blocks * cus;
}

void launch_attn_stream(hipStream_t s, int head_dim, const UnitDesc* descs, const AttnSeg* segs, const int32_t* seg_begin,
                        int n_groups, const void* q, const void* k_cache, const void* v_cache, int N_k, float scale,
                        void* out, float* part_o, float* part_ml, unsigned* part_count) {
  if (n_groups <= 0) return;
  typedef __bf16 T;
  if (head_dim == 64)
    hipLaunchKernelGGL((attn_pipe<64, 4, 1, true>), dim3(n_groups), dim3(256), 0, s, descs, nullptr, segs, seg_begin,
                       (const T*)q, (const T*)k_cache, (const T*)v_cache, N_k, scale, (T*)out, part_o, part_ml, part_count);
  else
    hipLaunchKernelGGL((attn_pipe<128, 4, 1, true>), dim3(n_groups), dim3(256), 0, s, descs, nullptr, segs, seg_begin,
                       (const T*)q, (const T*)k_cache, (const T*)v_cache, N_k, scale, (T*)out, part_o, part_ml, part_count);
}

}  // namespace hack
