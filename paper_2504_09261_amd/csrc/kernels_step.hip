// A whole compressing step of short units in one launch on gfx950: importance (Sec. 4.4, subset attention), selection (f_C, f_S),
// compaction K^ = K[I,:], V^ = V[I,:], and the attention of the current scale over it (Preliminaries, attention equation).
//
// A work-group of eight waves belongs to one unit.  It scores all of the unit's keys and ranks them (score_unit and select_rows, as score_select does),
// copies the kept rows of K and V into LDS at once, through the list that it has just formed there, stores its share of them behind each other
// where the next step expects them, and attends for its queries over the rows in LDS: eight waves = query tiles x key splits, the
// splits merged at the end as in attn_split.  A unit that keeps everything takes all of its rows instead, and stores the new ones.
// Work-groups of one unit (whole_step_queries says how many there are) repeat its scores and selection and share out queries and rows.
//
// These steps are chains of latencies.  As launches of their own (score and selection, then attention and moves, which start with the
// table, the list, the rows from memory again) they took 6.8 + 3.8 us at 60 units of 64 queries over 166 keys, 102 kept, and 23.0 + 39.7 us at 480 units of 256
// over 562, 306 kept (kernel trace); in one 8.4 and 48.7.  In-kernel time stamps, thousands of cycles: 60 units of 169 queries over 424 keys, 255 kept, four
// splits: scores 11.7, selection 5.4, row copies 2.0, waiting for them 0.4, moves 0.8, attention 2.7, merge 3.3 (a launch of 15.0 us); 480 units of 256 over 562, 306
// kept, no splits: 16.3, 5.8, 2.8, 1.1, 2.0, 12.1, stores 1.0.  What is left is mostly the scores' vector work and the barriers of the ranking.
#include <cfloat>

#include "device_util.h"
#include "hack_internal.h"
#include "score_device.h"
#include "select_device.h"
#include "split_stage.h"

namespace hack {

namespace {

using namespace dev;

constexpr int kNW = 8;   // waves

// TILES: score tiles of 32 keys a wave, NQ: 16-query tiles a wave, S: key splits, so that a work-group has 8 / S query tiles of 16 NQ.
// Grid: x = XCD (unit mod 8) + 8 work-group of the unit, y = unit / 8, so that the work-groups of a unit share an L2.
template <int D, int TILES, int NQ, int S>
__global__ __launch_bounds__(64 * kNW, D == 64 && TILES <= 2 && NQ == 1 ? 4 : 2) void step_units(
    const UnitDesc* __restrict__ descs, const __bf16* __restrict__ q, const int32_t* __restrict__ q_rows, const __bf16* k_cache,
    const __bf16* v_cache, const __bf16* k_new, const __bf16* v_new, WholeStep st, CachePtrs cache, int pos_new, int N_k, float scale,
    __bf16* __restrict__ out, int32_t* __restrict__ kept_idx, int64_t idx_stride) {
  constexpr int KC = D / 32, MT = D / 16, CPR = D / 8, RPI = 64 / CPR;
  constexpr int PER = TILES <= 2 ? 1 : 2;
  extern __shared__ __attribute__((aligned(1024))) char region[];
  __shared__ __attribute__((aligned(1024))) __bf16 q_lds[32 * D];
  __shared__ double red[kNW][kMaxObs], inv_s[kNW][kMaxObs];
  __shared__ uint32_t keys[256 * TILES];
  __shared__ SelectShared<64 * kNW, 11, 11> sh;

  const int di = blockIdx.y * 8 + (blockIdx.x & 7), part = blockIdx.x >> 3, parts = gridDim.x >> 3;
  if (di >= st.n_units) return;
  const UnitDesc d = descs[di];
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint32_t* const list = reinterpret_cast<uint32_t*>(region + st.region);
  const bool comp = !st.moved && d.mode == MOVE_GATHER;
  const int64_t new0 = (int64_t)d.unit * N_k;
  // wave w holds query tile w / S of the work-group's, key split w % S
  const int tile = w / S, split = w % S;
  const int col = lane & 15, g = lane >> 4;
  const int q0 = (part * (kNW / S) + tile) * 16 * NQ;
  bf16x8 qf[NQ][KC];
  auto load_q = [&] {
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) {
      const __bf16* qrow = q + (new0 + min(q0 + 16 * qt + col, N_k - 1)) * D;
#pragma unroll
      for (int c = 0; c < KC; ++c) qf[qt][c] = *reinterpret_cast<const bf16x8*>(qrow + 32 * c + 8 * g);
    }
  };

  if (comp) {
    score_unit<D, kNW, TILES>(d, q, q_rows, st.n_obs, N_k, scale, k_cache, k_new, reinterpret_cast<char (*)[8192]>(region), red, inv_s, keys, q_lds,
                              st.fault);
    load_q();   // the queries land behind the selection
    uint32_t* const hist = reinterpret_cast<uint32_t*>(region);
    clear_hist<64 * kNW, 11, 11>(hist, tid);
    __syncthreads();
    uint32_t key[PER];
    unsigned in_seg = 0;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const int j = tid * PER + e;
      key[e] = 0;
      if (j >= d.sel_lo && j < d.sel_hi) {
        in_seg |= 1u << e;
        key[e] = keys[j];
      }
    }
    select_rows<64 * kNW, PER, 11, 11, true>(d, key, in_seg, hist, sh, part == 0 ? kept_idx + (int64_t)d.unit * idx_stride : nullptr, nullptr, list);
    __syncthreads();
  } else {
    load_q();
  }

  // ---- the unit's rows into LDS, in the layouts of attn_split; rows past the end repeat the last one, and where no copy reaches V is
  // cleared (their scores are masked, their probabilities zero) ----
  const int n = d.n_out, n32 = (n + 31) / 32 * 32;
  __bf16* const Kh = reinterpret_cast<__bf16*>(region);
  __bf16* const Vh = Kh + (int64_t)n32 * D;
  // Entry s of the unit's numbering is row s of either home; a copy whose rows are all of one home takes a uniform base and 32 bits.
  const int home = st.moved ? n : d.len_in;   // entries below are cached rows
  const int64_t rc = (st.moved ? d.out_off : d.in_off) * (D * 2), rn = (new0 - home) * (D * 2);
  const char* const kc = reinterpret_cast<const char*>(k_cache) + rc;
  const char* const vc = reinterpret_cast<const char*>(v_cache) + rc;
  const char* const kn = reinterpret_cast<const char*>(k_new) + rn;
  const char* const vn = reinterpret_cast<const char*>(v_new) + rn;
  const int n_c = (n + RPI - 1) / RPI;        // copies per tensor
  auto entry = [&](int i) -> int { return comp ? (int)list[i] : i; };
  const unsigned k_lds = lds_addr_of(Kh), v_lds = lds_addr_of(Vh);
  auto copy = [&](int i, int s) {
    const int r = i * RPI + lane / CPR, c = lane % CPR;
    const unsigned at = (unsigned)s * (unsigned)(D * 2);
    const unsigned ko = at + (unsigned)(((c ^ swz_k<D>(r)) & (CPR - 1)) * 16), vo = at + (unsigned)(((c ^ swz_v16<D>(r)) & (CPR - 1)) * 16);
    const bool fresh = s >= home;
    if (!__any(fresh)) {
      load_to_lds(kc, ko, k_lds + (unsigned)(i * 1024));
      load_to_lds(vc, vo, v_lds + (unsigned)(i * 1024));
    } else if (__all(fresh)) {
      load_to_lds(kn, ko, k_lds + (unsigned)(i * 1024));
      load_to_lds(vn, vo, v_lds + (unsigned)(i * 1024));
    } else {
      load_to_lds((fresh ? kn : kc) + ko, k_lds + (unsigned)(i * 1024));
      load_to_lds((fresh ? vn : vc) + vo, v_lds + (unsigned)(i * 1024));
    }
  };
  constexpr int AHEAD = 4;   // list entries read together
  for (int i = w; i < n_c; i += AHEAD * kNW) {
    int s[AHEAD];
#pragma unroll
    for (int x = 0; x < AHEAD; ++x) s[x] = entry(min((i + x * kNW) * RPI + lane / CPR, n - 1));
#pragma unroll
    for (int x = 0; x < AHEAD; ++x)
      if (i + x * kNW < n_c) copy(i + x * kNW, s[x]);
  }
  {
    uint4* const z = reinterpret_cast<uint4*>(Vh + (int64_t)n_c * RPI * D);
    for (int e = tid; e < (n32 - n_c * RPI) * CPR; e += 64 * kNW) z[e] = make_uint4(0u, 0u, 0u, 0u);
  }
  // this work-group's share of the rows that move: rows [m0, m1) of the unit's n_mv
  const int n_mv = st.moved ? 0 : comp ? n : d.n_new, share = (n_mv + parts - 1) / parts;
  const int m0 = min(part * share, n_mv), m1 = min(m0 + share, n_mv);
  const int first = comp ? 0 : d.len_in;                       // LDS row of the first that moves
  const int64_t dst0 = comp ? d.out_off : d.in_off + d.len_in;
  int pos[2] = {0, 0};
  if (cache.pos != nullptr) {
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      const int i = m0 + tid + x * 64 * kNW;
      if (i < m1) {
        const int s = entry(first + i);
        pos[x] = s < d.len_in ? cache.pos[d.in_off + s] : pos_new + (s - d.len_in);
      }
    }
  }

  SplitStage<D, NQ> att;
  att.init(scale, lane);
#pragma unroll
  for (int qt = 0; qt < NQ; ++qt)
#pragma unroll
    for (int c = 0; c < KC; ++c) asm volatile("" ::"v"(qf[qt][c]));
  dma_wait_but<0>();
  __syncthreads();   // the unit's rows have landed

  // ---- rows that move ----
  for (int x = tid; x < (m1 - m0) * CPR; x += 64 * kNW) {
    const int i = m0 + x / CPR, c = x % CPR, r = first + i;
    const uint4 kr = *reinterpret_cast<const uint4*>(&Kh[r * D + ((c ^ swz_k<D>(r)) & (CPR - 1)) * 8]);
    const uint4 vr = *reinterpret_cast<const uint4*>(&Vh[r * D + ((c ^ swz_v16<D>(r)) & (CPR - 1)) * 8]);
    static_cast<uint4*>(cache.k)[(dst0 + i) * CPR + c] = kr;
    static_cast<uint4*>(cache.v)[(dst0 + i) * CPR + c] = vr;
  }
  if (cache.pos != nullptr) {
#pragma unroll
    for (int x = 0; x < 2; ++x) {
      const int i = m0 + tid + x * 64 * kNW;
      if (i < m1) cache.pos[dst0 + i] = pos[x];
    }
  }

  // ---- attention ----
  const int n_blocks = n32 / 32;
  if (q0 < N_k) {
    for (int b = split; b < n_blocks; b += S) {
      const __bf16* const Kt = Kh + b * 32 * D;
      const __bf16* const Vt = Vh + b * 32 * D;
      floatx4 sc[2][NQ];
      bf16x8 pf[NQ];
      att.scores(Kt, qf, sc);
      att.mask(sc, b, n);
      att.follow(sc, b == split);
      att.probs(sc, pf);
      att.row_sums(pf);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) att.pv(Vt, pf, mt);
    }
  }
  auto store = [&](int mt, int qt, const floatx4& x, float inv) {
    const int qi = q0 + 16 * qt + col;
    if (qi < N_k) att.store(out + (new0 + qi) * D, mt, x, inv);
  };
  if constexpr (S == 1) {
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) {
      const float inv = 1.f / att.ls[qt][0];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) store(mt, qt, att.o[mt][qt], inv);
    }
    return;
  }
  // ---- merge of the S splits of a query tile ----
  float* const m_sh = reinterpret_cast<float*>(&red[0][0]);     // [wave][16 NQ]
  float* const l_sh = reinterpret_cast<float*>(&inv_s[0][0]);
  __syncthreads();   // the rows have been read
  float4* const mine = reinterpret_cast<float4*>(region) + w * (NQ * MT * 64) + lane;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) mine[(mt * NQ + qt) * 64] = make_float4(att.o[mt][qt][0], att.o[mt][qt][1], att.o[mt][qt][2], att.o[mt][qt][3]);
  if (g == 0) {
#pragma unroll
    for (int qt = 0; qt < NQ; ++qt) {
      m_sh[w * 32 + 16 * qt + col] = att.mc[qt];
      l_sh[w * 32 + 16 * qt + col] = att.ls[qt][0];
    }
  }
  __syncthreads();
  const int w0 = tile * S;   // first wave of the tile
  const float4* const pp = reinterpret_cast<const float4*>(region) + w0 * (NQ * MT * 64) + lane;
  float f[NQ][S], inv[NQ];
#pragma unroll
  for (int qt = 0; qt < NQ; ++qt) {
    float m[S], M = -FLT_MAX, L = 0.f;
#pragma unroll
    for (int x = 0; x < S; ++x) m[x] = m_sh[(w0 + x) * 32 + 16 * qt + col];
#pragma unroll
    for (int x = 0; x < S; ++x) M = fmaxf(M, m[x]);
#pragma unroll
    for (int x = 0; x < S; ++x) {
      f[qt][x] = __builtin_amdgcn_exp2f(m[x] - M);
      L = fmaf(f[qt][x], l_sh[(w0 + x) * 32 + 16 * qt + col], L);
    }
    inv[qt] = 1.f / L;
  }
  // split x of the tile finishes the groups x, x + S, ... of its NQ MT
#pragma unroll
  for (int y = 0; y < NQ * MT; y += S) {
    const int group = y + split;
    if (NQ * MT % S != 0 && group >= NQ * MT) break;
    floatx4 acc = {0.f, 0.f, 0.f, 0.f};
    const int qt = NQ == 1 ? 0 : group % NQ;
#pragma unroll
    for (int x = 0; x < S; ++x) {
      const float4 p = pp[(x * NQ * MT + group) * 64];
      const float fx = NQ == 1 || qt == 0 ? f[0][x] : f[NQ - 1][x];
      acc[0] = fmaf(fx, p.x, acc[0]);
      acc[1] = fmaf(fx, p.y, acc[1]);
      acc[2] = fmaf(fx, p.z, acc[2]);
      acc[3] = fmaf(fx, p.w, acc[3]);
    }
    store(group / NQ, qt, acc, NQ == 1 || qt == 0 ? inv[0] : inv[NQ - 1]);
  }
}

}  // namespace

void launch_step_units(hipStream_t s, int head_dim, const UnitDesc* descs, WholeStep st, const void* q, const CachePtrs& cache, const void* k_new,
                       const void* v_new, int pos_new, int N_k, float scale, void* out, int32_t* kept, int64_t kept_stride) {
  typedef __bf16 T;
  const int rows = (st.max_rows + 31) / 32 * 32;
  st.region = (int)whole_step_region(head_dim, st.max_rows);
  const dim3 grid(8 * ((N_k + st.queries - 1) / st.queries), (st.n_units + 7) / 8);
  const size_t lds = st.region + rows * 4;
#define HACK_STEP(D_, T_, Q_, S_)                                                                                                              \
  hipLaunchKernelGGL((step_units<D_, T_, Q_, S_>), grid, dim3(64 * kNW), lds, s, descs, (const T*)q, st.q_rows, (const T*)cache.k, (const T*)cache.v, \
                     (const T*)k_new, (const T*)v_new, st, cache, pos_new, N_k, scale, (T*)out, kept, kept_stride)
#define HACK_STEP_Q(D_, T_)                                \
  switch (st.queries) {                                    \
    case 16: HACK_STEP(D_, T_, 1, 8); break;               \
    case 32: HACK_STEP(D_, T_, 1, 4); break;               \
    case 64: HACK_STEP(D_, T_, 2, 4); break;               \
    case 128: HACK_STEP(D_, T_, 2, 2); break;              \
    default: HACK_STEP(D_, T_, 2, 1); break;               \
  }
  if (head_dim == 64) {
    if (st.max_t <= 256) HACK_STEP_Q(64, 1)
    else if (st.max_t <= 512) HACK_STEP_Q(64, 2)
    else HACK_STEP_Q(64, 4)
  } else {
    if (st.max_t <= 256) HACK_STEP_Q(128, 1)
    else if (st.max_t <= 512) HACK_STEP_Q(128, 2)
    else HACK_STEP_Q(128, 4)
  }
#undef HACK_STEP_Q
#undef HACK_STEP
}

}  // namespace hack
