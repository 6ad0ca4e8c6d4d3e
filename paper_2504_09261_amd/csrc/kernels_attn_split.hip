// Attention for scale steps with few queries (Preliminaries, attention
// equation: O = Softmax(scale * Q K^T) V, no mask inside a scale step) on gfx950.
//
// The first scale steps of a next-scale schedule have a handful to a few
// hundred queries per unit: tiles of 128 queries leave most of the chip idle
// and every work-group walks the whole cache alone.  Here a work item is
// (unit, 32 queries), a work-group takes one or half of one (sixteen_queries), and its four or eight waves split the KEYS: wave w
// of four takes the 32-key blocks w, w+4, ... with a private online softmax, and the partial
// results (reference, normaliser, unnormalised O) are merged through LDS at
// the end.  There is no work-group barrier inside the loop: K and V blocks
// travel HBM -> LDS directly (global_load_lds, whole rows, so the copies are
// fully coalesced) into one private K slot and one private V slot per wave; the
// copy of the next K block is issued as soon as the score MFMAs have read the
// current one, the copy of the next V block as soon as the PV MFMAs have read
// theirs.  K fragments are read with ds_read_b128, V^T through the transposing
// LDS read, with swizzles free of bank conflicts.  S^T = K Q^T and O^T += V^T P^T in 16x16x32 matrix instructions; row sums are one
// more tile of the latter, against ones.
// The queries come through LDS too: read straight from memory into the operand registers of all waves, 32 rows x 32 bytes an instruction, they
// kept the memory pipeline busy for longer than a block takes (in-kernel time stamps, 32 units of 256 queries over 521 keys, head_dim 128: 1.1 us
// of 10.5).  With that and the first block of V awaited behind the first scores, us a launch, before / now: head_dim 128, 32 units, queries over
// keys: 4 over 5 4.0 / 3.1, 64 over 121 5.4 / 4.5, 144 over 265 8.0 / 6.9, 256 over 521 10.2 / 9.0, 400 over 921 16.9 / 14.2; head_dim 64: 60 units, 64 over 155
// 5.2 / 4.1, 256 over 306 7.4 / 6.5, 960 units, 36 over 91 11.6 / 9.9, 27 units, 1369 over 640 19.4 / 18.2.  What is left is a chain: at 121 keys some 0.3 us for the
// item, 0.6 to issue the copies, 0.4 until they have landed, 0.8 the block and 0.7 the merge (first passes through the code), in front of it the launch.
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
#include <cfloat>
#include <type_traits>

#include "device_util.h"
#include "hack_internal.h"
#include "split_stage.h"

namespace hack {

namespace {

using namespace dev;

constexpr int kKB = 32;        // keys per block
constexpr int kItemRows = 32;  // queries per work item

// fuse != 0: keys are [rows in_off .. in_off+len_in of the cache | the unit's n_new
// rows of k_new / v_new], and those new rows are also written behind the cached
// ones (k_app / v_app / pos_app are the cache arrays, which k_cache / v_cache then
// alias: reads stay below row len_in, writes at or above it).
// fuse == 0: keys are rows [out_off, out_off + n_out) of the cache.
// NQ tiles of 16 queries a work-group (2: a work item, 1: half of one), kWaves waves = key splits.
template <int D, bool GATHER, int NQ, int kWaves>
__global__ __launch_bounds__(64 * kWaves, D == 64 ? 4 : 2) void attn_split(
    const UnitDesc* __restrict__ descs, const AttnItem* __restrict__ items, const __bf16* __restrict__ q,
    const __bf16* k_cache, const __bf16* v_cache, const __bf16* k_new, const __bf16* v_new, __bf16* k_app,
    __bf16* v_app, int32_t* pos_app, int pos_new, int fuse, int N_k, float scale, __bf16* __restrict__ out, GatherArgs ga) {
  constexpr int KC = D / 32;        // MFMA steps over head_dim for S^T
  constexpr int MT = D / 16;        // 16-row tiles of O^T
  constexpr int CPR = D / 8;        // 16-byte chunks per row
  constexpr int RPI = 64 / CPR;     // block rows covered by one wave-wide copy instruction
  constexpr int IPB = kKB / RPI;    // copy instructions per block and tensor
  constexpr int BLK = kKB * D;      // elements per block
  constexpr int QROWS = 16 * NQ;    // queries of this work-group

  constexpr int XI = GATHER ? 1 : 0;   // list copies per block
  // list entries of this wave's blocks w, w + kWaves, ...: block b in slot (b / kWaves) % 4
  __shared__ __attribute__((aligned(256))) int idx_ring[GATHER ? kWaves : 1][GATHER ? 4 * kKB : 1];
  if constexpr (GATHER) {
    const int mover = (int)blockIdx.x - ((int)gridDim.x - ga.n_moves);
    if (mover >= 0) {
      move_rows<D / 8, 64 * kWaves>(descs, ga, mover, N_k);
      return;
    }
  }
  // The halves of an item follow each other on its XCD (work-group id mod 8).
  const AttnItem it = items[NQ == 1 ? (blockIdx.x >> 4) * 8 + (blockIdx.x & 7) : blockIdx.x];
  const int q0 = it.q_tile * kItemRows + (NQ == 1 ? 16 * ((blockIdx.x >> 3) & 1) : 0);
  if (it.desc < 0 || q0 >= N_k) return;
  const AttnItem& d = it;   // the item carries the descriptor fields read here
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 15, g = lane >> 4;

  const int total = d.n_out;                       // keys attended over
  const int len_c = fuse ? d.len_in : d.n_out;     // of which come from the cache
  const int64_t base = fuse ? d.in_off : d.out_off;
  const int64_t new_row0 = (int64_t)d.unit * N_k;  // first row of the unit in q / k_new / v_new / out

  // [0]: K, [1]: V; after the loop a wave's pair holds its unnormalised O^T
  __shared__ __attribute__((aligned(1024))) __bf16 ring[kWaves][2][BLK];
  __shared__ __attribute__((aligned(1024))) __bf16 q_sh[QROWS * D];
  __shared__ float m_sh[kWaves][QROWS], l_sh[kWaves][QROWS];

  // Block b of K or V into this wave's LDS: lane l of copy
  // instruction i fills LDS row r = i RPI + l / CPR, chunk position c = l % CPR, from
  // global chunk c ^ swz(r) of key row b*32 + r.  A block that lies wholly in the
  // cache or wholly in the new rows is a contiguous piece of memory: uniform base
  // plus loop-invariant lane offsets.  The ragged last block and a block that
  // straddles the two sources take per-lane addresses (rows past the end repeat
  // the last key; their scores are masked): a uniform row of either source plus 32
  // bits.  The first scales' only block is ragged: formed from 64-bit row numbers those addresses stood 1 us in front of it
  // (head_dim 128, four steps of 32 units 25.2 -> 23.8 us), and copying 32 rows where there are 1 to 21 half a microsecond
  // (with a one-block unit stored straight from its wave's registers 24.0 -> 23.3; one 256^2 image 91.3 -> 90.3).
  // Copies KP (K) or VP (V) apart differ by whole rows only.
  constexpr int KP = D == 128 ? 4 : 2, VP = D == 128 ? 2 : 1;
  unsigned k_src[KP], v_src[VP];
#pragma unroll
  for (int i = 0; i < KP; ++i) {
    const int r = i * RPI + lane / CPR, c = lane % CPR;
    k_src[i] = (unsigned)(r * D + ((c ^ swz_k<D>(r)) & (CPR - 1)) * 8) * 2u;
    if (i < VP) v_src[i] = (unsigned)(r * D + ((c ^ swz_v16<D>(r)) & (CPR - 1)) * 8) * 2u;
  }
  auto lds_of = [&](int wave, int v) { return lds_addr_of(&ring[0][0][0]) + (unsigned)((wave * 2 + v) * BLK * 2); };
  // first: in front of the loop, which counts a block's copies in flight; only the rows there are travel then, of these the
  // copies i0, i0 + di, ...; what the K slot holds behind them is masked, and the V slot is cleared.
  auto issue = [&](auto k_tag, bool first, int i0, int di, int b, const __bf16* cache, const __bf16* fresh, const auto& src, unsigned lds) {
    constexpr bool IS_K = decltype(k_tag)::value;
    const int j0 = b * kKB;
    const __bf16* blk = nullptr;
    if (j0 + kKB <= len_c) blk = cache + (base + j0) * D;
    else if (j0 >= len_c && j0 + kKB <= total) blk = fresh + (new_row0 + (j0 - len_c)) * D;
    if (blk != nullptr && di == 1) {
#pragma unroll
      for (int i = 0; i < IPB; ++i) {
        constexpr int P = IS_K ? KP : VP;
        load_to_lds(blk + i / P * (P * RPI * D), src[i % P], lds + (unsigned)(i * 1024));
      }
    } else {
      const __bf16* const in_cache = cache + (base + j0) * D;                 // row j0 of the unit, were it cached
      const __bf16* const in_fresh = fresh + (new_row0 + (j0 - len_c)) * D;   // ... or a new one
      const int last = total - 1 - j0;
      auto row_copy = [&](int i) {
        const int r = i * RPI + lane / CPR, rc = min(r, last);
        const unsigned off = (unsigned)(rc * D + (((lane % CPR) ^ (IS_K ? swz_k<D>(r) : swz_v16<D>(r))) & (CPR - 1)) * 8) * 2u;
        load_to_lds(reinterpret_cast<const char*>(j0 + rc < len_c ? in_cache : in_fresh) + off, lds + (unsigned)(i * 1024));
      };
      if (!first) {
#pragma unroll
        for (int i = 0; i < IPB; ++i) row_copy(i);
        return;
      }
      const int n = min(IPB, last / RPI + 1);
#pragma unroll 1
      for (int i = i0; i < n; i += di) row_copy(i);
      if (!IS_K) {
        uintx4* slot = reinterpret_cast<uintx4*>(&ring[0][0][0]) + (lds - lds_of(0, 0)) / 16 + lane;
#pragma unroll 1
        for (int i = n + (i0 - n % di + di) % di; i < IPB; i += di) slot[i * 64] = uintx4{0u, 0u, 0u, 0u};
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
  int* const xring = &idx_ring[GATHER ? w : 0][0];
  const unsigned ring_lds = lds_addr_of(xring);
  auto issue_x = [&](int b) {   // b = w + kWaves i; past the end: entries of the last block
    const int b0 = min(b, n_blocks - 1);
    if (lane < kKB)
      load_to_lds_dword(list + b0 * kKB, (unsigned)(min(lane, total - 1 - b0 * kKB) * 4), ring_lds + (unsigned)(((b / kWaves) & 3) * kKB * 4));
  };
  auto issue_rows = [&](int i0, int di, int b, const char* cached, const char* fresh, const auto& src, unsigned lds) {
    constexpr int P = sizeof(src) / sizeof(src[0]);
    const int j0 = b * kKB;
    const int* x = xring + ((b / kWaves) & 3) * kKB + lane / CPR;
    if (j0 + kKB <= seam || j0 >= seam) {
      const char* base = j0 >= seam ? fresh : cached;
#pragma unroll
      for (int i = 0; i < IPB; ++i)
        if (di == 1 || i % di == i0)
          load_to_lds(base, (unsigned)x[i * RPI] * (unsigned)(D * 2) + (src[i % P] & (D * 2 - 1)), lds + (unsigned)(i * 1024));
    } else {
#pragma unroll
      for (int i = 0; i < IPB; ++i) {
        if (di != 1 && i % di != i0) continue;
        const int j = x[i * RPI];
        load_to_lds((j < d.len_in ? cached : fresh) + (int64_t)j * (D * 2) + (src[i % P] & (D * 2 - 1)), lds + (unsigned)(i * 1024));
      }
    }
  };
  auto issue_k = [&](int b, unsigned lds, bool first = false, int i0 = 0, int di = 1) {
    if constexpr (GATHER) issue_rows(i0, di, b, kc, kn, k_src, lds);
    else issue(std::true_type{}, first, i0, di, b, k_cache, k_new, k_src, lds);
  };
  auto issue_v = [&](int b, unsigned lds, bool first = false, int i0 = 0, int di = 1) {
    if constexpr (GATHER) issue_rows(i0, di, b, vc, vn, v_src, lds);
    else issue(std::false_type{}, first, i0, di, b, v_cache, v_new, v_src, lds);
  };

  // The queries travel through LDS as well, row col of tile qt in the K layout: one row a lane, straight from memory into the
  // operand registers of every wave, they take the memory pipeline at a quarter of its rate.
  {
    const char* const qbase = reinterpret_cast<const char*>(q + (new_row0 + q0) * D);
    const int last = min(QROWS, N_k - q0) - 1;
#pragma unroll
    for (int i = 0; i < QROWS / RPI; ++i)
      if (i % kWaves == w) {
        const int r = i * RPI + lane / CPR;
        load_to_lds(qbase, (unsigned)(min(r, last) * D + (((lane % CPR) ^ swz_k<D>(r)) & (CPR - 1)) * 8) * 2u, lds_addr_of(q_sh) + (unsigned)(i * 1024));
      }
  }

  // The first scales' units have one block: all waves copy and score it, and each forms a share of the head-dim.
  const bool lone = n_blocks == 1;
  if (lone) {
    if constexpr (GATHER) {
      if (lane < kKB) load_to_lds_dword(list, (unsigned)(min(lane, total - 1) * 4), ring_lds);
      dma_wait_but<0>();
    }
    issue_k(0, lds_of(0, 0), true, w, kWaves);
    issue_v(0, lds_of(0, 1), true, w, kWaves);
  } else if (w < n_blocks) {
    if constexpr (GATHER) {
      issue_x(w);
      issue_x(w + kWaves);
      dma_wait_but<0>();
    }
    if constexpr (GATHER) issue_x(w + 2 * kWaves);
    issue_k(w, lds_of(w, 0), true);
    issue_v(w, lds_of(w, 1), true);
  }

  // Cache update of this tile's rows: loaded behind the first K and V blocks, stored when the loop is done (stored at
  // once they would put a memory round trip in front of everything else: one 256^2 image 99.6 against 96.5 us).
  constexpr int LPR = D / 8;                               // 16-byte pieces per row
  constexpr int APP = (QROWS * LPR + 64 * kWaves - 1) / (64 * kWaves);   // pieces per thread
  uintx4 app_k[APP], app_v[APP];
  const int n_app = fuse ? min(QROWS, N_k - q0) * LPR : 0;
  if (!GATHER && fuse) {
#pragma unroll
    for (int i = 0; i < APP; ++i) {
      const int e = min(tid + i * 64 * kWaves, n_app - 1);
      app_k[i] = (reinterpret_cast<const uintx4*>(k_new) + (new_row0 + q0) * LPR)[e];
      app_v[i] = (reinterpret_cast<const uintx4*>(v_new) + (new_row0 + q0) * LPR)[e];
    }
  }

  SplitStage<D, NQ> att;
  att.init(scale, lane);

  // The queries and the first K block have landed; what was issued behind them, the first V block and the rows to append, may still be
  // on its way.  A wave that has issued fewer copies (a ragged block, a share of the only block, none) waits for all of them.
  if (lone || (w + 1) * kKB > total) dma_wait_but<0>();
  else if (!GATHER && fuse) dma_wait_but<IPB + 2 * APP>();
  else dma_wait_but<IPB>();
  __syncthreads();     // ... of every wave
  // Q fragments (B operand of S^T = K Q^T): query 16 qt + col, head-dim slice [32 c + 8 g, +8)
  bf16x8 qf[NQ][KC];
#pragma unroll
  for (int qt = 0; qt < NQ; ++qt)
#pragma unroll
    for (int c = 0; c < KC; ++c) qf[qt][c] = *reinterpret_cast<const bf16x8*>(&q_sh[16 * qt * D + att.k_off[c]]);

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
  auto store = [&](int mt, int qt, const floatx4& x, float inv) {
    const int qi = q0 + 16 * qt + col;
    if (qi < N_k) att.store(out + (new_row0 + qi) * D, mt, x, inv);
  };

  if (lone) {
    floatx4 sc[2][NQ];
    bf16x8 pf[NQ];
    att.scores(&ring[0][0][0], qf, sc);
    att.mask(sc, 0, total);
    att.follow(sc, true);
    att.probs(sc, pf);
    att.row_sums(pf);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
      if (mt % kWaves == w) {
        att.pv(&ring[0][1][0], pf, mt);
#pragma unroll
        for (int qt = 0; qt < NQ; ++qt) store(mt, qt, att.o[mt][qt], 1.f / att.ls[qt][0]);
      }
    append();
    return;
  }

  // Vector-memory traffic of a wave inside the loop, all hand-issued copies, in
  // order: ... K(b), V(b) | K(next) after the score MFMAs of b, V(next) after the
  // PV MFMAs of b.  Copies complete in order, so "all but the newest IPB
  // instructions" is K(b) at the top of an iteration and V(b) before its PV.
  for (int b = w; b < n_blocks; b += kWaves) {
    const bool more = b + kWaves < n_blocks;
    dma_wait_but<IPB>();                 // K(b) has landed (V(b) may still be in flight)
    floatx4 sc[2][NQ];
    att.scores(&ring[w][0][0], qf, sc);
    // the MFMAs above have consumed every K read, so the slot may be refilled;
    // nothing below moves above this point
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    if (more) {
      if constexpr (GATHER) issue_x(b + 3 * kWaves);
      issue_k(b + kWaves, lds_of(w, 0));
    }
    att.mask(sc, b, total);
    bf16x8 pf[NQ];
    att.follow(sc, b == w);
    att.probs(sc, pf);
    if (more) dma_wait_but<IPB + XI>();  // V(b) has landed (K(next) and list entries may still be in flight)
    else dma_wait_but<0>();
    att.row_sums(pf);
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) att.pv(&ring[w][1][0], pf, mt);
    // every V read has been consumed by an MFMA above: the slot may be refilled
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    if (more) issue_v(b + kWaves, lds_of(w, 1));
  }
  dma_wait_but<0>();   // nothing is outstanding when the slots are reused below
  append();

  // ---- merge the partial results ----
  // This wave's copies have all landed and its LDS reads are done: its pair of slots becomes its O^T partial, four registers of a
  // lane together, lanes contiguous (b128 accesses, a quarter of the instructions of a register at a time).
  constexpr int kPart = 2 * BLK * 2 / 16;   // float4 per wave
  static_assert(NQ * MT * 64 <= kPart && kWaves % NQ == 0, "partial results fit the slots");
  float4* mine = reinterpret_cast<float4*>(&ring[w][0][0]) + lane;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) mine[(mt * NQ + qt) * 64] = make_float4(att.o[mt][qt][0], att.o[mt][qt][1], att.o[mt][qt][2], att.o[mt][qt][3]);
  if (g == 0) {
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) {
      m_sh[w][16 * qt + col] = att.mc[qt];
      l_sh[w][16 * qt + col] = att.ls[qt][0];
    }
  }
  __syncthreads();
  // wave w finishes query tile w % NQ, head-dim tiles w / NQ, w / NQ + kWaves / NQ, ...
  const int qt = w % NQ;
  float M = -FLT_MAX;
#pragma unroll
  for (int x = 0; x < kWaves; ++x) M = fmaxf(M, m_sh[x][16 * qt + col]);
  float f[kWaves], L = 0.f;
#pragma unroll
  for (int x = 0; x < kWaves; ++x) {
    f[x] = __builtin_amdgcn_exp2f(m_sh[x][16 * qt + col] - M);   // a wave without blocks has summed nothing
    L = fmaf(f[x], l_sh[x][16 * qt + col], L);
  }
  const float inv = 1.f / L;
  const float4* const part = reinterpret_cast<const float4*>(&ring[0][0][0]) + lane;
#pragma unroll
  for (int m = 0; m < MT; m += kWaves / NQ) {
    const int mt = m + w / NQ;
    if (mt >= MT) break;
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int x = 0; x < kWaves; ++x) {
      const float4 p = part[x * kPart + (mt * NQ + qt) * 64];
      acc[0] = fmaf(f[x], p.x, acc[0]);
      acc[1] = fmaf(f[x], p.y, acc[1]);
      acc[2] = fmaf(f[x], p.z, acc[2]);
      acc[3] = fmaf(f[x], p.w, acc[3]);
    }
    store(mt, qt, acc, inv);
  }
}

}  // namespace

int attn_split_q_tile_rows() { return kItemRows; }

// Which launches take 16 queries a work-group.  A launch of few work-groups is a chain of latencies over a few blocks: half of the queries
// halve a wave's matrix and vector work, the partial results and the merge, and twice as many work-groups share it out; where compute units
// have more than one of them to do anyway, they copy K and V twice as often.  Measured, us a launch, 32 / 16 queries, work items of 32: head_dim
// 128, four waves, keys: 32 items of 21 3.4 / 3.1, 64 of 121 5.1 / 4.5, 128 of 300 7.0 / 6.0, 192 of 400 and 200 8.1 / 8.1, 6.1 / 5.9; 224 of 521 9.1 / 9.3,
// 416 of 921 14.2 / 21.7; 64, four waves: 120 of 155 4.7 / 4.1, 256 of 400 6.3 / 5.8, 300 of 300 and 600 6.0 / 5.7, 7.8 / 7.9, 360 of 271 6.2 / 5.9; 448 of 450
// 7.4 / 8.5.  Eight waves (longer caches), head_dim 128: 64 of 1500 11.2 / 9.9, 96 of 1500 11.5 / 10.9, but a step that compresses to as many 30.5 / 32.0
// (the work-groups that move its rows find no room); 64: 128 of 1500 8.6 / 7.1, 160 8.5 / 10.3.
static bool sixteen_queries(int head_dim, bool eight, int n_items) {
  if (eight) return n_items <= (head_dim == 64 ? 128 : 64);
  return n_items <= (head_dim == 64 ? 384 : 192);
}

template <int D, bool GATHER, typename... Args>
static void launch_split(hipStream_t s, bool eight, int n_items, int n_moves, Args... args) {
  const bool half = n_items % 8 == 0 && sixteen_queries(D, eight, n_items);   // items come dealt to eight XCDs
  const dim3 grid((half ? 2 * n_items : n_items) + n_moves), block(eight ? 512 : 256);
  if (half && eight) hipLaunchKernelGGL((attn_split<D, GATHER, 1, 8>), grid, block, 0, s, args...);
  else if (half) hipLaunchKernelGGL((attn_split<D, GATHER, 1, 4>), grid, block, 0, s, args...);
  else if (eight) hipLaunchKernelGGL((attn_split<D, GATHER, 2, 8>), grid, block, 0, s, args...);
  else hipLaunchKernelGGL((attn_split<D, GATHER, 2, 4>), grid, block, 0, s, args...);
}

void launch_attn_split(hipStream_t s, int head_dim, const UnitDesc* descs, const AttnItem* items, int n_items,
                       const void* q, const void* k_cache, const void* v_cache, const void* k_new, const void* v_new,
                       void* k_app, void* v_app, int32_t* pos_app, int pos_new, bool append, bool eight, int N_k, float scale,
                       void* out) {
  if (n_items <= 0) return;
  typedef __bf16 T;
#define HACK_ARGS s, eight, n_items, 0, descs, items, (const T*)q, (const T*)k_cache, (const T*)v_cache, (const T*)k_new, (const T*)v_new, (T*)k_app, \
                  (T*)v_app, pos_app, pos_new, append ? 1 : 0, N_k, scale, (T*)out, GatherArgs{}
  if (head_dim == 64) launch_split<64, false>(HACK_ARGS);
  else launch_split<128, false>(HACK_ARGS);
#undef HACK_ARGS
}

void launch_attn_split_gather(hipStream_t s, int head_dim, const UnitDesc* descs, const AttnItem* items, int n_items,
                              const GatherArgs& g, const void* q, const void* k_cache, const void* v_cache, int N_k,
                              float scale, void* out) {
  if (n_items + g.n_moves <= 0) return;
  typedef __bf16 T;
#define HACK_ARGS s, g.eight, n_items, g.n_moves, descs, items, (const T*)q, (const T*)k_cache, (const T*)v_cache, (const T*)nullptr, (const T*)nullptr, \
                  (T*)nullptr, (T*)nullptr, (int32_t*)nullptr, 0, 0, N_k, scale, (T*)out, g
  if (head_dim == 64) launch_split<64, true>(HACK_ARGS);
  else launch_split<128, true>(HACK_ARGS);
#undef HACK_ARGS
}

}  // namespace hack
