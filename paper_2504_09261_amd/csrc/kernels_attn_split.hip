// Attention for scale steps with few queries (Preliminaries, attention
// equation: O = Softmax(scale * Q K^T) V, no mask inside a scale step) on gfx950.
//
// The first scale steps of a next-scale schedule have a handful to a few
// hundred queries per unit: tiles of 128 queries leave most of the chip idle
// and every work-group walks the whole cache alone.  Here a work item is
// (unit, 32 queries) and its four waves split the KEYS: wave w takes the 32-key
// blocks w, w+4, ... with a private online softmax, and the four partial
// results (running max, normaliser, unnormalised O) are merged through LDS at
// the end.  There is no work-group barrier inside the loop: K and V blocks
// travel HBM -> LDS directly (global_load_lds, whole rows, so the copies are
// fully coalesced) into one private K slot and one private V slot per wave; the
// copy of the next K block is issued as soon as the score MFMAs have read the
// current one, the copy of the next V block as soon as the PV MFMAs have read
// theirs.  K fragments are read with ds_read_b128, V^T through the transposing
// LDS read, with the same bank-conflict-free swizzles as the large-step kernel.
// Optionally the kernel also performs the cache update of the step (cache-update
// equation of the Preliminaries): keys are then read from the virtual
// concatenation [cached rows | rows of the current scale] and work item t
// copies rows [32t, 32t+32) of the current scale behind the unit's cached rows,
// so a step that does not compress needs a single launch.  A step that compresses
// (GATHER) reads keys and values in place through the units' lists of kept rows,
// and further work-groups of the launch move those rows: one launch less, and the
// move beside the attention (one 256^2 image, four compressing steps of 60 units,
// 120 -> 111 us; odd sides 128 -> 121 us).  A wave copies the list entries of its next-but-one
// block into an LDS ring of its own; all but one block of a unit lie wholly in the
// cached or wholly in the new rows, so their rows are a wave-uniform base plus 32 bits.
// The 128-query kernel gains nothing from the same: each of its work items pays 4 us for
// the way through the list, and beside matrix work that already draws all the power the
// chip may take, the moving work-groups cost what they cost alone (1024^2 schedules
// 784 / 1267 / 3326 us as separate launches, 763 / 1254 / 3355 fused).
#include <type_traits>

#include "device_util.h"
#include "hack_internal.h"

namespace hack {

namespace {

using namespace dev;

constexpr int kKB = 32;        // keys per block
constexpr int kQTile = 32;     // queries per work item

// fuse != 0: keys are [rows in_off .. in_off+len_in of the cache | the unit's n_new
// rows of k_new / v_new], and those new rows are also written behind the cached
// ones (k_app / v_app / pos_app are the cache arrays, which k_cache / v_cache then
// alias: reads stay below row len_in, writes at or above it).
// fuse == 0: keys are rows [out_off, out_off + n_out) of the cache.
template <int D, bool GATHER, int kWaves>   // kWaves waves per work-group = key splits
__global__ __launch_bounds__(64 * kWaves, D == 64 ? 4 : 2) void attn_split(
    const UnitDesc* __restrict__ descs, const AttnItem* __restrict__ items, const __bf16* __restrict__ q,
    const __bf16* k_cache, const __bf16* v_cache, const __bf16* k_new, const __bf16* v_new, __bf16* k_app,
    __bf16* v_app, int32_t* pos_app, int pos_new, int fuse, int N_k, float scale, __bf16* __restrict__ out, GatherArgs ga) {
  constexpr int KK = D / 16;        // MFMA steps over head_dim for S^T
  constexpr int MB = D / 32;        // 32-row blocks of O^T
  constexpr int CPR = D / 8;        // 16-byte chunks per row
  constexpr int RPI = 64 / CPR;     // block rows covered by one wave-wide copy instruction
  constexpr int IPB = kKB / RPI;    // copy instructions per V block
  constexpr int BLK = kKB * D;      // elements per block

  constexpr int XI = GATHER ? 1 : 0;   // list copies per block
  // list entries of this wave's blocks w, w + kWaves, ...: block b in slot (b / kWaves) % 4 (a copy also fills the 32 words behind it)
  __shared__ __attribute__((aligned(256))) int idx_ring[GATHER ? kWaves : 1][GATHER ? 4 * 2 * kKB : 1];
  if constexpr (GATHER) {
    const int mover = (int)blockIdx.x - ((int)gridDim.x - ga.n_moves);
    if (mover >= 0) {
      move_rows<D / 8, 64 * kWaves>(descs, ga, mover, N_k);
      return;
    }
  }
  const AttnItem it = items[blockIdx.x];
  if (it.desc < 0) return;
  const AttnItem& d = it;   // the item carries the descriptor fields read here
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 31, half = lane >> 5;

  const int total = d.n_out;                       // keys attended over
  const int len_c = fuse ? d.len_in : d.n_out;     // of which come from the cache
  const int64_t base = fuse ? d.in_off : d.out_off;
  const int64_t new_row0 = (int64_t)d.unit * N_k;  // first row of the unit in q / k_new / v_new / out
  const int q0 = it.q_tile * kQTile;

  // per wave one K slot [0] and one V slot [1]; after the loop the pair holds the
  // wave's unnormalised O^T (same size)
  __shared__ __attribute__((aligned(1024))) __bf16 Vs[kWaves][2][BLK];
  __shared__ float m_sh[kWaves][32], l_sh[kWaves][32];

  // Block b of K (slot 0) or V (slot 1) into this wave's LDS: lane l of copy
  // instruction i fills LDS row r = i RPI + l / CPR, chunk position c = l % CPR, from
  // global chunk c ^ swz(r) of key row b*32 + r.  A block that lies wholly in the
  // cache or wholly in the new rows is a contiguous piece of memory: uniform base
  // plus loop-invariant lane offsets.  The ragged last block and a block that
  // straddles the two sources take per-lane addresses (rows past the end repeat
  // the last key; their scores are masked): a uniform row of either source plus 32
  // bits.  The first scales' only block is ragged: formed from 64-bit row numbers those addresses stood 1 us in front of it
  // (head_dim 128, four steps of 32 units 25.2 -> 23.8 us), and copying 32 rows where there are 1 to 21 half a microsecond
  // (with a one-block unit stored straight from its wave's registers 24.0 -> 23.3; one 256^2 image 91.3 -> 90.3).
  const unsigned vs_lds = lds_addr_of(&Vs[0][0][0]);
  unsigned k_src[IPB], v_src[IPB];
#pragma unroll
  for (int i = 0; i < IPB; ++i) {
    const int r = i * RPI + lane / CPR, c = lane % CPR;
    k_src[i] = (unsigned)(r * D + ((c ^ swz_k<D>(r)) & (CPR - 1)) * 8) * 2u;
    v_src[i] = (unsigned)(r * D + ((c ^ swz_v<D>(r)) & (CPR - 1)) * 8) * 2u;
  }
  const unsigned k_lds = vs_lds + (unsigned)((w * 2 + 0) * BLK * 2), v_lds = vs_lds + (unsigned)((w * 2 + 1) * BLK * 2);
  auto issue = [&](auto k_tag, bool first, int b, const __bf16* cache, const __bf16* fresh, const unsigned (&src)[IPB], unsigned lds) {
    constexpr bool IS_K = decltype(k_tag)::value;
    const int j0 = b * kKB;
    const __bf16* blk = nullptr;
    if (j0 + kKB <= len_c) blk = cache + (base + j0) * D;
    else if (j0 >= len_c && j0 + kKB <= total) blk = fresh + (new_row0 + (j0 - len_c)) * D;
    if (blk != nullptr) {
#pragma unroll
      for (int i = 0; i < IPB; ++i) load_to_lds(blk, src[i], lds + (unsigned)(i * 1024));
    } else {
      const __bf16* const in_cache = cache + (base + j0) * D;                 // row j0 of the unit, were it cached
      const __bf16* const in_fresh = fresh + (new_row0 + (j0 - len_c)) * D;   // ... or a new one
      const int last = total - 1 - j0;
      // The loop below counts a block's copies in flight.  In front of it only the rows there are travel; what the K slot holds
      // behind them is masked, and the V slot is cleared.
      const int n = first ? min(IPB, last / RPI + 1) : IPB;
#pragma unroll 1
      for (int i = 0; i < n; ++i) {
        const int r = i * RPI + lane / CPR, rc = min(r, last);
        const unsigned off = (unsigned)(rc * D + (((lane % CPR) ^ (IS_K ? swz_k<D>(r) : swz_v<D>(r))) & (CPR - 1)) * 8) * 2u;
        load_to_lds(reinterpret_cast<const char*>(j0 + rc < len_c ? in_cache : in_fresh) + off, lds + (unsigned)(i * 1024));
      }
      if (!IS_K) {
        uintx4* slot = reinterpret_cast<uintx4*>(&Vs[w][1][0]) + lane;
#pragma unroll 1
        for (int i = n; i < IPB; ++i) slot[i * 64] = uintx4{0u, 0u, 0u, 0u};
      }
    }
  };
  const int n_blocks = (total + kKB - 1) / kKB;
  const int32_t* list = nullptr;
  int seam = 0;
  const char *kc = nullptr, *vc = nullptr, *kn = nullptr, *vn = nullptr;   // row 0 of the list's numbering in the two homes
  if constexpr (GATHER) {
    const bool gather = d.mode == MOVE_GATHER;
    list = gather ? ga.kept + (int64_t)d.unit * ga.kept_stride : ga.iota;
    seam = gather ? ga.seam[d.unit] : d.len_in;
    const int64_t rc = d.in_off * (D * 2), rn = (new_row0 - d.len_in) * (D * 2);
    kc = reinterpret_cast<const char*>(k_cache) + rc;
    vc = reinterpret_cast<const char*>(v_cache) + rc;
    kn = static_cast<const char*>(ga.k_new) + rn;
    vn = static_cast<const char*>(ga.v_new) + rn;
  }
  int* const ring = &idx_ring[GATHER ? w : 0][0];
  const unsigned ring_lds = lds_addr_of(ring);
  auto issue_x = [&](int b) {   // b = w + kWaves i; past the end: entries of the last block
    const int b0 = min(b, n_blocks - 1);
    load_to_lds_dword(list + b0 * kKB, (unsigned)(min(lane, total - 1 - b0 * kKB) * 4), ring_lds + (unsigned)(((b / kWaves) & 3) * 2 * kKB * 4));
  };
  auto issue_rows = [&](int b, const char* cached, const char* fresh, const unsigned (&src)[IPB], unsigned lds) {
    const int j0 = b * kKB;
    const int* x = ring + ((b / kWaves) & 3) * 2 * kKB + lane / CPR;
    if (j0 + kKB <= seam || j0 >= seam) {
      const char* base = j0 >= seam ? fresh : cached;
#pragma unroll
      for (int i = 0; i < IPB; ++i) load_to_lds(base, (unsigned)x[i * RPI] * (unsigned)(D * 2) + (src[i] & (D * 2 - 1)), lds + (unsigned)(i * 1024));
    } else {
#pragma unroll
      for (int i = 0; i < IPB; ++i) {
        const int j = x[i * RPI];
        load_to_lds((j < d.len_in ? cached : fresh) + (int64_t)j * (D * 2) + (src[i] & (D * 2 - 1)), lds + (unsigned)(i * 1024));
      }
    }
  };
  auto issue_k = [&](int b, bool first = false) {
    if constexpr (GATHER) {
      issue_x(b + 2 * kWaves);
      issue_rows(b, kc, kn, k_src, k_lds);
    } else {
      issue(std::true_type{}, first, b, k_cache, k_new, k_src, k_lds);
    }
  };
  auto issue_v = [&](int b, bool first = false) {
    if constexpr (GATHER) issue_rows(b, vc, vn, v_src, v_lds);
    else issue(std::false_type{}, first, b, v_cache, v_new, v_src, v_lds);
  };

  if (w < n_blocks) {
    if constexpr (GATHER) {
      issue_x(w);
      issue_x(w + kWaves);
      dma_wait_but<0>();
    }
    issue_k(w, true);
    issue_v(w, true);
  }

  // Cache update of this tile's rows: loaded behind the first K and V blocks, stored when the loop is done (stored at
  // once they would put a memory round trip in front of everything else: one 256^2 image 99.6 against 96.5 us).
  constexpr int LPR = D / 8;                               // 16-byte pieces per row
  constexpr int APP = (kQTile * LPR + 64 * kWaves - 1) / (64 * kWaves);   // pieces per thread
  uintx4 app_k[APP], app_v[APP];
  const int n_app = fuse ? min(kQTile, N_k - q0) * LPR : 0;
  if (!GATHER && fuse) {
#pragma unroll
    for (int i = 0; i < APP; ++i) {
      const int e = min(tid + i * 64 * kWaves, n_app - 1);
      app_k[i] = (reinterpret_cast<const uintx4*>(k_new) + (new_row0 + q0) * LPR)[e];
      app_v[i] = (reinterpret_cast<const uintx4*>(v_new) + (new_row0 + q0) * LPR)[e];
    }
  }

  // Q fragments (B operand): query col, head-dim slice [16kk + 8 half, +8)
  bf16x8 qf[KK];
  {
    const __bf16* qrow = q + (new_row0 + min(q0 + col, N_k - 1)) * D;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) qf[kk] = *reinterpret_cast<const bf16x8*>(qrow + 16 * kk + 8 * half);
    // consumed here so that the compiler's wait for them sits before the loop,
    // whose vector-memory waits are all placed by hand
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) asm volatile("" ::"v"(qf[kk]));
  }
  dma_wait_but<0>();   // first K and V blocks (and everything above) have landed

  floatx16 o[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[mb][r] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  const float c2 = scale * kLog2eF;

  // V^T operand reads: row 4 half + e (+16 sg, +8), head-dim 32mb + 16(g&1) + 4qd
  const int g = lane >> 4, e = (lane >> 2) & 3, qd = lane & 3;
  int v_off[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
    v_off[mb] = (4 * half + e) * D + (((4 * mb + 2 * (g & 1) + (qd >> 1)) ^ swz_v<D>(e)) & (CPR - 1)) * 8 + 4 * (qd & 1);
  int k_off[KK];   // K operand reads: row col, chunk 2kk + half
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) k_off[kk] = col * D + (((2 * kk + half) ^ swz_k<D>(col)) & (CPR - 1)) * 8;
  const bf16x2 ones2 = {(__bf16)1.0f, (__bf16)1.0f};

  // Vector-memory traffic of a wave inside the loop, all hand-issued copies, in
  // order: ... K(b), V(b) | K(next) after the score MFMAs of b, V(next) after the
  // PV MFMAs of b.  Copies complete in order, so "all but the newest IPB
  // instructions" is K(b) at the top of an iteration and V(b) before its PV.
  const __bf16* Kt = &Vs[w][0][0];
  const __bf16* Vt = &Vs[w][1][0];
  for (int b = w; b < n_blocks; b += kWaves) {
    const bool more = b + kWaves < n_blocks;
    dma_wait_but<IPB>();                 // K(b) has landed (V(b) may still be in flight)
    // S^T of block b: per lane one query column and 16 key rows
    floatx16 sc;
#pragma unroll
    for (int r = 0; r < 16; ++r) sc[r] = 0.f;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
      const bf16x8 kf = *reinterpret_cast<const bf16x8*>(&Kt[k_off[kk]]);
      sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[kk], sc, 0, 0, 0);
    }
    // the MFMAs above have consumed every K read, so the slot may be refilled;
    // nothing below moves above this point
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    if (more) issue_k(b + kWaves);
    if ((b + 1) * kKB > total) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if (b * kKB + 8 * (r >> 2) + 4 * half + (r & 3) >= total) sc[r] = -INFINITY;
    }
    float mx = sc[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, sc[r]);
    mx = pair_max(mx);                       // finite: the block holds a valid key
    const float m_new = fmaxf(m_run, mx);
    if (__any(m_new != m_run)) {
      const float a = __builtin_amdgcn_exp2f((m_run - m_new) * c2);   // first block: exp2(-inf) = 0
      l_run *= a;
      if (b != w) {   // nothing has been added up in front of the first block
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[mb][r] *= a;
      }
      m_run = m_new;
    }
    const float mc = m_run * c2;
    bf16x8 pf[2];
#pragma unroll
    for (int r = 0; r < 16; ++r) pf[r >> 3][r & 7] = (__bf16)__builtin_amdgcn_exp2f(fmaf(sc[r], c2, -mc));
    // the row sum is taken over the rounded probabilities, the numbers the PV product uses
    float psum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
      const bf16x2 pr = {pf[r >> 3][r & 7], pf[r >> 3][(r & 7) + 1]};
      psum = __builtin_amdgcn_fdot2_f32_bf16(pr, ones2, psum, false);
    }
    l_run += psum;
    if (more) dma_wait_but<IPB + XI>();  // V(b) has landed (K(next) and list entries may still be in flight)
    else dma_wait_but<0>();
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
    // every V read has been consumed by an MFMA above: the slot may be refilled
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    if (more) issue_v(b + kWaves);
  }
  dma_wait_but<0>();   // nothing is outstanding when the slots are reused below
  auto append = [&] {
    if (!GATHER && fuse) {
      uintx4* kd = reinterpret_cast<uintx4*>(k_app) + (d.in_off + d.len_in + q0) * LPR;
      uintx4* vd = reinterpret_cast<uintx4*>(v_app) + (d.in_off + d.len_in + q0) * LPR;
#pragma unroll
      for (int i = 0; i < APP; ++i) {
        const int e = tid + i * 64 * kWaves;
        if (e < n_app) {
          kd[e] = app_k[i];
          vd[e] = app_v[i];
        }
      }
      if (pos_app != nullptr && tid < n_app / LPR) pos_app[d.in_off + d.len_in + q0 + tid] = pos_new + q0 + tid;
    }
  };
  const int qi = q0 + col;
  __bf16* orow = out + (new_row0 + min(qi, N_k - 1)) * D;

  // A unit of one block (the first scales): wave 0 holds the whole result.
  if (n_blocks == 1) {
    if (w == 0) {
      const float inv = 1.f / pair_sum(l_run);
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          bf16x4 pk;
#pragma unroll
          for (int i = 0; i < 4; ++i) pk[i] = (__bf16)(o[mb][4 * r4 + i] * inv);
          if (qi < N_k) *reinterpret_cast<bf16x4*>(orow + 32 * mb + 8 * r4 + 4 * half) = pk;
        }
    }
    append();
    return;
  }
  append();

  // ---- merge the partial results ----
  // This wave's copies have all landed and its LDS reads are done: its two slots
  // become its O^T partial, four registers of a lane together, lanes contiguous (b128 accesses, a quarter of the
  // instructions of a register at a time).
  l_run = pair_sum(l_run);
  float4* mine = reinterpret_cast<float4*>(&Vs[w][0][0]) + lane;
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4)
      mine[(mb * 4 + r4) * 64] = make_float4(o[mb][4 * r4], o[mb][4 * r4 + 1], o[mb][4 * r4 + 2], o[mb][4 * r4 + 3]);
  if (half == 0) {
    m_sh[w][col] = m_run;
    l_sh[w][col] = l_run;
  }
  __syncthreads();
  // wave w finishes registers [w CH, (w+1) CH) of the 16 MB per lane; register
  // 16 mb + r of lane (col, half) is head-dim 32mb + 8(r/4) + 4 half + r%4 of query col
  constexpr int CH = 16 * MB / kWaves;
  static_assert(CH % 4 == 0, "whole groups of four registers");
  const float4* const part = reinterpret_cast<const float4*>(&Vs[0][0][0]) + w * (CH / 4) * 64 + lane;
  constexpr int kPart = 2 * BLK * 2 / 16;   // float4 per partial result
  float M = -INFINITY;
#pragma unroll
  for (int x = 0; x < kWaves; ++x) M = fmaxf(M, m_sh[x][col]);   // finite: wave 0 saw block 0
  float f[kWaves], L = 0.f;
#pragma unroll
  for (int x = 0; x < kWaves; ++x) {
    f[x] = __builtin_amdgcn_exp2f((m_sh[x][col] - M) * c2);       // a wave without blocks: exp2(-inf) = 0
    L = fmaf(f[x], l_sh[x][col], L);
  }
  float4 acc[CH / 4];
#pragma unroll
  for (int i4 = 0; i4 < CH / 4; ++i4) {
    acc[i4] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int x = 0; x < kWaves; ++x) {
      const float4 p = part[x * kPart + i4 * 64];
      acc[i4].x = fmaf(f[x], p.x, acc[i4].x);
      acc[i4].y = fmaf(f[x], p.y, acc[i4].y);
      acc[i4].z = fmaf(f[x], p.z, acc[i4].z);
      acc[i4].w = fmaf(f[x], p.w, acc[i4].w);
    }
  }
  const float inv = 1.f / L;
#pragma unroll
  for (int i4 = 0; i4 < CH / 4; ++i4) {
    const int reg0 = w * CH + 4 * i4;
    const bf16x4 pk = {(__bf16)(acc[i4].x * inv), (__bf16)(acc[i4].y * inv), (__bf16)(acc[i4].z * inv), (__bf16)(acc[i4].w * inv)};
    const int mb = reg0 >> 4, r4 = (reg0 & 15) >> 2;
    if (qi < N_k) *reinterpret_cast<bf16x4*>(orow + 32 * mb + 8 * r4 + 4 * half) = pk;
  }
}

}  // namespace

int attn_split_q_tile_rows() { return kQTile; }

#define HACK_SPLIT(D_, G_, ...)                                                                                  \
  do {                                                                                                           \
    if (eight) hipLaunchKernelGGL((attn_split<D_, G_, 8>), dim3(n), dim3(512), 0, s, descs, items, __VA_ARGS__); \
    else hipLaunchKernelGGL((attn_split<D_, G_, 4>), dim3(n), dim3(256), 0, s, descs, items, __VA_ARGS__);       \
  } while (0)

void launch_attn_split(hipStream_t s, int head_dim, const UnitDesc* descs, const AttnItem* items, int n_items,
                       const void* q, const void* k_cache, const void* v_cache, const void* k_new, const void* v_new,
                       void* k_app, void* v_app, int32_t* pos_app, int pos_new, bool append, bool eight, int N_k, float scale,
                       void* out) {
  const int n = n_items;
  if (n <= 0) return;
  typedef __bf16 T;
  if (head_dim == 64)
    HACK_SPLIT(64, false, (const T*)q, (const T*)k_cache, (const T*)v_cache, (const T*)k_new, (const T*)v_new, (T*)k_app, (T*)v_app,
               pos_app, pos_new, append ? 1 : 0, N_k, scale, (T*)out, GatherArgs{});
  else
    HACK_SPLIT(128, false, (const T*)q, (const T*)k_cache, (const T*)v_cache, (const T*)k_new, (const T*)v_new, (T*)k_app, (T*)v_app,
               pos_app, pos_new, append ? 1 : 0, N_k, scale, (T*)out, GatherArgs{});
}

void launch_attn_split_gather(hipStream_t s, int head_dim, const UnitDesc* descs, const AttnItem* items, int n_items,
                              const GatherArgs& g, const void* q, const void* k_cache, const void* v_cache, int N_k,
                              float scale, void* out) {
  const int n = n_items + g.n_moves;
  if (n <= 0) return;
  typedef __bf16 T;
  const bool eight = g.eight;
  if (head_dim == 64)
    HACK_SPLIT(64, true, (const T*)q, (const T*)k_cache, (const T*)v_cache, nullptr, nullptr, nullptr, nullptr, nullptr, 0, 0, N_k,
               scale, (T*)out, g);
  else
    HACK_SPLIT(128, true, (const T*)q, (const T*)k_cache, (const T*)v_cache, nullptr, nullptr, nullptr, nullptr, nullptr, 0, 0, N_k,
               scale, (T*)out, g);
}
#undef HACK_SPLIT

}  // namespace hack
