// float32 attention of the current scale over the ragged cache (Preliminaries,
// attention equation: O = Softmax(scale * Q K^T) V, no mask inside a scale step)
// on gfx950, with v_mfma_f32_16x16x4_f32 (float32 products and sums throughout).
//
// The float32 schedules are small (hundreds of keys, a few hundred queries, a few
// dozen units): what bounds a launch is the chain of dependent work of one
// work-group, not the chip's arithmetic.  So a work item is (unit, 16 R queries)
// and its NW waves split the KEYS: wave w takes the 16-key blocks w, w + NW, ...
// with a private online softmax; the partial results meet in LDS at the end.  There
// is no barrier and no LDS traffic inside the loop: operands go from global memory
// (L2) straight into the registers the MFMAs read.
//   * S^T = K Q^T.  The order in which the contraction runs over the head
//     dimension is free as long as both operands agree, so lane (i, g) = (l % 16,
//     l / 16) feeds step 4 c + e with element 16 c + 4 g + e of row i: one 16-byte
//     load per four steps, 64 contiguous bytes per row and load instruction.
//   * C register r of lane (i, g) is key 4 g + r of query i, which is exactly the B
//     operand of O^T += V^T P^T for the key set {4 g + r : g}: step r takes register r.
//   * The rows of V^T may be taken in any order too: MFMA e covers the head-dim rows
//     4 i + e (+ 64 m), so one 16-byte load of V row 4 g + r feeds four MFMAs, whole
//     256-byte row pieces are read per instruction, and the four results of a register
//     are four consecutive outputs of a query (16-byte stores).
// R = 1 with 8 waves for launches of up to 384 such items (one work-group per compute
// unit, or little more: the depth of a wave's key loop is what lasts), beyond that R = 2
// with 4 waves, which reads K and V half as often per query.  Measured, us a launch,
// R = 1 / R = 2: head_dim 64, 256 items of 306 keys 8.5 / 11.2, 512 items 13.7 / 11.9, 800
// items of 700 keys 42 / 36; head_dim 128: 13.7 / 18.3, 26.2 / 19.8, 81 / 69; at 64 units x
// 1024 queries x 2000 keys R = 2 reaches 90 (d = 64) and 108 TFLOP/s (d = 128) of the 157
// the float32 matrix rate allows.  The rows to append loaded with the operands instead of behind the loop, and units of one block (the first
// scales) stored without the merge: launches over 1 to 14 keys 4.4 -> 3.5 us (kernel trace), a 680-token schedule 105.3 -> 103.4.  One query per lane with K/V rows broadcast from LDS, the
// form this replaces, took 135 us on average over the ten launches of a 680-token
// schedule (16 heads x 64, batch 1); the whole schedule went from 1699 to 379 us.
#include "device_util.h"
#include "hack_internal.h"

namespace hack {

namespace {

using namespace dev;

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;

constexpr int kKB = 16;   // keys per block

// all-reduce over the four 16-lane rows of a wave (lanes i, i + 16, i + 32, i + 48)
__device__ __forceinline__ float rows_max(float v) {
  const unsigned u = __builtin_bit_cast(unsigned, v);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return pair_max(fmaxf(__builtin_bit_cast(float, (unsigned)r[0]), __builtin_bit_cast(float, (unsigned)r[1])));
}
__device__ __forceinline__ float rows_sum(float v) {
  const unsigned u = __builtin_bit_cast(unsigned, v);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return pair_sum(__builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]));
}

// fuse != 0: keys are [rows in_off .. in_off + len_in of the cache | the unit's N_k rows
// of k_new / v_new], and work item t also writes its rows of the current scale (and
// their position ids) behind the cached ones (k_app / v_app / pos_app, which k_cache /
// v_cache then alias: reads stay below row len_in, writes at or above it).
// fuse == 0: keys are rows [out_off, out_off + n_out) of the cache.
// GATHER (fuse == 0): keys are the rows the unit keeps, read in place through its list, whose entries are loaded a block
// ahead; ga.n_moves further work-groups move those rows (as in the bf16 key-split kernel).  A step less one launch: the 680-token
// schedule 130.9 -> 124.3 us; single compressing steps of 8 to 64 units, 78 to 414 keys, 0 to 2 us of 35 to 100 less.
// kCache: fuse == 0 is known, for hack_attn with 16 queries a work item.  Where the kernel does not know it, every key's row is looked for in two homes, and
// rows to append are held through the loop: head_dim 128, 36 units of 3 queries over 1230 keys 34.8 -> 33.8 us, 34 of 2 over 2315 54.2 -> 53.4,
// 200 random launches of 16 and 32 queries 0.98 of the time; with 32 queries it gains nothing (332 units of 17 over 757 keys 71.3 / 74.6).  The store
// of one-block units without the merge, worth 10 to 20 % to those, still costs few long units 2 to 4 % (36 of 3 over 1230 without it 33.4).
enum : int { kFuse = 0, kCache = 1, kGather = 2 };
template <int D, int R, int NW, int MODE>
__global__ __launch_bounds__(64 * NW, 2) void attn_f32(
    const AttnItem* __restrict__ items, const float* __restrict__ q, const float* k_cache, const float* v_cache,
    const float* k_new, const float* v_new, float* k_app, float* v_app, int32_t* pos_app, int pos_new, int may_fuse, int N_k,
    float scale, float* __restrict__ out, const UnitDesc* __restrict__ descs, GatherArgs ga) {
  constexpr bool GATHER = MODE == kGather;
  const int fuse = MODE == kFuse ? may_fuse : 0;
  constexpr int C = D / 16;          // 16-byte pieces of a K / Q row per lane
  constexpr int M = D / 64;          // 16-byte pieces of a V row per lane
  constexpr int QT = 16 * R;         // queries per work item
  constexpr int NG = R * M * 4;      // groups of four output registers per lane

  if constexpr (GATHER) {
    const int mover = (int)blockIdx.x - ((int)gridDim.x - ga.n_moves);
    if (mover >= 0) {
      move_rows<D / 4, 64 * NW>(descs, ga, mover, N_k);
      return;
    }
  }
  const AttnItem it = items[blockIdx.x];
  if (it.desc < 0) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i = lane & 15, g = lane >> 4;

  const int total = it.n_out;                     // keys attended over
  const int len_c = fuse ? it.len_in : it.n_out;  // of which come from the cache
  const int64_t base = fuse ? it.in_off : it.out_off;
  const int64_t new_row0 = (int64_t)it.unit * N_k;   // first row of the unit in q / k_new / v_new / out
  const int q0 = it.q_tile * QT;

  __shared__ floatx4 o_sh[NW][NG][64];
  __shared__ float m_sh[NW][QT], l_sh[NW][QT];

  const int n_blocks = (total + kKB - 1) / kKB;
  // ---- Q operands ----
  floatx4 qf[R][C];
  if (w < n_blocks) {
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const float* qrow = q + (new_row0 + min(q0 + 16 * j + i, N_k - 1)) * D + 4 * g;
#pragma unroll
      for (int c = 0; c < C; ++c) qf[j][c] = *reinterpret_cast<const floatx4*>(qrow + 16 * c);
    }
  }

  // key row in its home; rows past the end repeat the last one (their scores are masked)
  const int32_t* list = nullptr;
  if constexpr (GATHER) list = it.mode == MOVE_GATHER ? ga.kept + (int64_t)it.unit * ga.kept_stride : ga.iota;
  auto entry = [&](int key) -> int {
    const int j = min(key, total - 1);
    if constexpr (GATHER) return list[j];
    else return j;
  };
  const int64_t cache0 = GATHER ? it.in_off : base;
  const int home = GATHER ? it.len_in : len_c;   // entries below are cached rows
  auto row_of = [&](const float* cache, const float* fresh, int x) -> const float* {
    if constexpr (MODE == kCache) return cache + (cache0 + x) * D;
    else return x < home ? cache + (cache0 + x) * D : fresh + (new_row0 + (x - home)) * D;
  };
  floatx4 kf[C], vf[4][M];
  int xk = 0, xv[4];   // entries of the next K block, of this V block
  auto entry_k = [&](int b) { xk = entry(b * kKB + i); };
  auto entries_v = [&](int b) {
#pragma unroll
    for (int r = 0; r < 4; ++r) xv[r] = entry(b * kKB + 4 * g + r);
  };
  auto load_k = [&]() {
    const float* p = row_of(k_cache, k_new, xk) + 4 * g;
#pragma unroll
    for (int c = 0; c < C; ++c) kf[c] = *reinterpret_cast<const floatx4*>(p + 16 * c);
  };
  auto load_v = [&]() {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float* p = row_of(v_cache, v_new, xv[r]) + 4 * i;
#pragma unroll
      for (int m = 0; m < M; ++m) vf[r][m] = *reinterpret_cast<const floatx4*>(p + 64 * m);
    }
  };

  // Cache update of this tile's rows: loaded behind the first operands, stored when the loop is done (loaded there they put a memory
  // round trip in front of the merge).
  constexpr int LPR = D / 4;                                       // 16-byte pieces per row
  constexpr int APP = (QT * LPR + 64 * NW - 1) / (64 * NW);        // pieces per thread
  uint4 app_k[APP], app_v[APP];
  const int n_app = !GATHER && fuse ? min(QT, N_k - q0) * LPR : 0;

  floatx4 o[R][M][4];   // [query block][64-row block of O^T][MFMA e]: C register r of lane (i, g) is O[query i][64 m + 16 g + 4 r + e]
  float m_run[R], l_run[R];
#pragma unroll
  for (int j = 0; j < R; ++j) {
    m_run[j] = -INFINITY;
    l_run[j] = 0.f;
#pragma unroll
    for (int m = 0; m < M; ++m)
#pragma unroll
      for (int e = 0; e < 4; ++e) o[j][m][e] = floatx4{0.f, 0.f, 0.f, 0.f};
  }
  const float c2 = scale * kLog2eF;

  if (w < n_blocks) {
    entry_k(w);
    entries_v(w);
    load_k();
  }
  if (!GATHER && fuse) {
#pragma unroll
    for (int x = 0; x < APP; ++x) {
      const int e = min(tid + x * 64 * NW, n_app - 1);
      app_k[x] = (reinterpret_cast<const uint4*>(k_new) + (new_row0 + q0) * LPR)[e];
      app_v[x] = (reinterpret_cast<const uint4*>(v_new) + (new_row0 + q0) * LPR)[e];
    }
  }
  for (int b = w; b < n_blocks; b += NW) {
    const bool more = b + NW < n_blocks;
    load_v();   // lands behind the score MFMAs
    if (more) {
      entry_k(b + NW);
      entries_v(b + NW);
    }
    floatx4 sc[R];
#pragma unroll
    for (int j = 0; j < R; ++j) sc[j] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int j = 0; j < R; ++j) sc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][e], qf[j][c][e], sc[j], 0, 0, 0);
    if (more) load_k();   // lands behind the softmax and the value MFMAs
    if ((b + 1) * kKB > total) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (b * kKB + 4 * g + r >= total)
#pragma unroll
          for (int j = 0; j < R; ++j) sc[j][r] = -INFINITY;
    }
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const float mx = rows_max(fmaxf(fmaxf(sc[j][0], sc[j][1]), fmaxf(sc[j][2], sc[j][3])));
      const float m_new = fmaxf(m_run[j], mx);   // finite: the block holds a valid key
      if (__any(m_new != m_run[j])) {
        const float a = __builtin_amdgcn_exp2f((m_run[j] - m_new) * c2);   // first block: exp2(-inf) = 0
        l_run[j] *= a;
#pragma unroll
        for (int m = 0; m < M; ++m)
#pragma unroll
          for (int e = 0; e < 4; ++e) o[j][m][e] *= a;
        m_run[j] = m_new;
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        sc[j][r] = __builtin_amdgcn_exp2f((sc[j][r] - m_run[j]) * c2);
        l_run[j] += sc[j][r];
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int m = 0; m < M; ++m)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int j = 0; j < R; ++j)
            o[j][m][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[r][m][e], sc[j][r], o[j][m][e], 0, 0, 0);
  }

  if (!GATHER && fuse) {
    uint4* kd = reinterpret_cast<uint4*>(k_app) + (it.in_off + it.len_in + q0) * LPR;
    uint4* vd = reinterpret_cast<uint4*>(v_app) + (it.in_off + it.len_in + q0) * LPR;
#pragma unroll
    for (int x = 0; x < APP; ++x) {
      const int e = tid + x * 64 * NW;
      if (e < n_app) {
        kd[e] = app_k[x];
        vd[e] = app_v[x];
      }
    }
    if (pos_app != nullptr && tid < n_app / LPR) pos_app[it.in_off + it.len_in + q0 + tid] = pos_new + q0 + tid;
  }

  // A unit of one block (the first scales): wave 0 holds the whole result.
  if (n_blocks == 1) {
    if (w == 0) {
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const float inv = 1.f / rows_sum(l_run[j]);
        const int qi = q0 + 16 * j + i;
        if (qi < N_k) {
#pragma unroll
          for (int m = 0; m < M; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r)
              *reinterpret_cast<floatx4*>(out + (new_row0 + qi) * D + 64 * m + 16 * g + 4 * r) =
                  floatx4{o[j][m][0][r], o[j][m][1][r], o[j][m][2][r], o[j][m][3][r]} * inv;
        }
      }
    }
    return;
  }

  // ---- merge the waves' partial results ----
#pragma unroll
  for (int j = 0; j < R; ++j) {
    const float l = rows_sum(l_run[j]);
    if (g == 0) {
      m_sh[w][16 * j + i] = m_run[j];
      l_sh[w][16 * j + i] = l;
    }
#pragma unroll
    for (int m = 0; m < M; ++m)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        o_sh[w][(j * M + m) * 4 + r][lane] = floatx4{o[j][m][0][r], o[j][m][1][r], o[j][m][2][r], o[j][m][3][r]};
  }
  __syncthreads();
  for (int x = w; x < NG; x += NW) {   // wave w finishes register groups w, w + NW, ...
    const int j = x / (4 * M), m = (x >> 2) % M, r = x & 3;
    const int qc = 16 * j + i;
    float top = -INFINITY;
#pragma unroll
    for (int y = 0; y < NW; ++y) top = fmaxf(top, m_sh[y][qc]);   // finite: wave 0 saw block 0
    floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
    float L = 0.f;
#pragma unroll
    for (int y = 0; y < NW; ++y) {
      const float f = __builtin_amdgcn_exp2f((m_sh[y][qc] - top) * c2);   // a wave without blocks: exp2(-inf) = 0
      L = fmaf(f, l_sh[y][qc], L);
      const floatx4 part = o_sh[y][x][lane];
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[e] = fmaf(f, part[e], acc[e]);
    }
    const float inv = 1.f / L;
    if (q0 + qc < N_k)
      *reinterpret_cast<floatx4*>(out + (new_row0 + q0 + qc) * D + 64 * m + 16 * g + 4 * r) = acc * inv;
  }
}

template <int D, int R, int NW>
void launch_gather_t(hipStream_t s, const UnitDesc* descs, const AttnItem* items, int n_items, const GatherArgs& g, const void* q,
                     const void* k_cache, const void* v_cache, int N_k, float scale, void* out) {
  typedef float T;
  hipLaunchKernelGGL((attn_f32<D, R, NW, kGather>), dim3(n_items + g.n_moves), dim3(64 * NW), 0, s, items, (const T*)q,
                     (const T*)k_cache, (const T*)v_cache, (const T*)g.k_new, (const T*)g.v_new, nullptr, nullptr, nullptr, 0, 0, N_k,
                     scale, (T*)out, descs, g);
}

template <int D, int R, int NW>
void launch_t(hipStream_t s, const AttnItem* items, int n_items, const void* q, const void* k_cache, const void* v_cache,
              const void* k_new, const void* v_new, void* k_app, void* v_app, int32_t* pos_app, int pos_new, int fuse, int N_k,
              float scale, void* out) {
  typedef float T;
#define HACK_ATTN(MODE_)                                                                                                             \
  hipLaunchKernelGGL((attn_f32<D, R, NW, MODE_>), dim3(n_items), dim3(64 * NW), 0, s, items, (const T*)q, (const T*)k_cache,          \
                     (const T*)v_cache, (const T*)k_new, (const T*)v_new, (T*)k_app, (T*)v_app, pos_app, pos_new, fuse, N_k,          \
                     scale, (T*)out, nullptr, GatherArgs{})
  if constexpr (R == 1) {
    if (!fuse) {
      HACK_ATTN(kCache);
      return;
    }
  }
  HACK_ATTN(kFuse);
#undef HACK_ATTN
}

}  // namespace

int attn_f32_q_tile_rows(int n_units, int N_k) { return (int64_t)n_units * ((N_k + 15) / 16) <= kAttnF32SmallItems ? 16 : 32; }

void launch_attn_f32(hipStream_t s, int head_dim, const AttnItem* items, int n_items, int q_tile_rows, const void* q,
                     const void* k_cache, const void* v_cache, const void* k_new, const void* v_new, void* k_app, void* v_app,
                     int32_t* pos_app, int pos_new, int fuse, int N_k, float scale, void* out) {
  if (n_items <= 0) return;
#define HACK_ARGS s, items, n_items, q, k_cache, v_cache, k_new, v_new, k_app, v_app, pos_app, pos_new, fuse, N_k, scale, out
  if (head_dim == 64) {
    if (q_tile_rows == 16) launch_t<64, 1, 8>(HACK_ARGS);
    else launch_t<64, 2, 4>(HACK_ARGS);
  } else {
    if (q_tile_rows == 16) launch_t<128, 1, 8>(HACK_ARGS);
    else launch_t<128, 2, 4>(HACK_ARGS);
  }
#undef HACK_ARGS
}

void launch_attn_f32_gather(hipStream_t s, int head_dim, const UnitDesc* descs, const AttnItem* items, int n_items, int q_tile_rows,
                            const GatherArgs& g, const void* q, const void* k_cache, const void* v_cache, int N_k, float scale,
                            void* out) {
  if (n_items + g.n_moves <= 0) return;
#define HACK_ARGS s, descs, items, n_items, g, q, k_cache, v_cache, N_k, scale, out
  if (head_dim == 64) {
    if (q_tile_rows == 16) launch_gather_t<64, 1, 8>(HACK_ARGS);
    else launch_gather_t<64, 2, 4>(HACK_ARGS);
  } else {
    if (q_tile_rows == 16) launch_gather_t<128, 1, 8>(HACK_ARGS);
    else launch_gather_t<128, 2, 4>(HACK_ARGS);
  }
#undef HACK_ARGS
}

}  // namespace hack
