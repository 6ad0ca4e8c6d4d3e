// Device-side helpers shared by the gfx950 MFMA kernels of this library
// (attention, score, head variance, merge): vector types, the HBM -> LDS copy
// and its wait, the LDS swizzles, lane-pair exchanges and the accumulator
// layout of v_mfma_f32_32x32x16_bf16.  HIP device code only.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hack_internal.h"

namespace hack {
namespace dev {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short shortx4;
typedef __attribute__((__vector_size__(4 * sizeof(unsigned)))) unsigned uintx4;

constexpr float kLog2eF = 1.4426950408889634f;

// ---- LDS layout -------------------------------------------------------------
// Tiles go from HBM straight into LDS (one contiguous KiB per wave instruction),
// so LDS rows cannot be padded; bank conflicts are avoided by a swizzle instead:
// the 16-byte chunk at position c of LDS row r holds global chunk c ^ f(r).  The
// LDS moves 256 bytes per clock (64 banks of 4 bytes), so one phase of a b128
// read covers 16 consecutive lanes (16 rows at one chunk position) and one phase
// of a transposing b64 read covers 32 lanes (4 rows x 64 bytes); f spreads those
// over all 16 chunk slots of 256 bytes:
//   D=128 (256-byte rows): f_K(r) = r & 15,        f_V(r) = 4 (r & 3)
//   D=64  (128-byte rows): f_K(r) = (r >> 1) & 7,  f_V(r) = 4 ((r >> 1) & 1)
// (measured: SQ_LDS_BANK_CONFLICT / SQ_LDS_IDX_ACTIVE was exactly 0.5 with the
// 32-bank variants r & 7 and 2 (r & 3), and is 0 with these).
// swz_k: tiles read as MFMA A/B operands with ds_read_b128 (row = lane % 32).
// swz_v: tiles read with the transposing ds_read_b64_tr_b16 (V^T operand).
template <int D> __device__ __forceinline__ int swz_k(int r) { return D == 128 ? (r & 15) : ((r >> 1) & 7); }
template <int D> __device__ __forceinline__ int swz_v(int r) { return D == 128 ? 4 * (r & 3) : 4 * ((r >> 1) & 1); }

// swz_v16: V tiles read as operands of v_mfma_f32_16x16x32_bf16, whose transposing reads cover 8 rows x 32 bytes a phase.
template <int D> __device__ __forceinline__ int swz_v16(int r) { return D == 128 ? 2 * (r & 7) : 2 * ((r >> 1) & 3); }

__device__ __forceinline__ unsigned lds_addr_of(const void* p) {
  return (unsigned)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

// Transposing LDS read: four consecutive rows of one 16-bit column group per lane.
__device__ __forceinline__ bf16x4 lds_read_tr(const __bf16* p) {
  shortx4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) shortx4*)(p));
  return __builtin_bit_cast(bf16x4, v);
}

// ---- HBM -> LDS copies ------------------------------------------------------
// One KiB (dwordx4) or 256 bytes (dword) per wave instruction without a register
// round trip: lane l writes LDS bytes [lds_addr + 16 l, +16) resp. [lds_addr + 4 l, +4).
// Issued from inline assembly so that the compiler does not wait for the copy
// before unrelated LDS reads (it would otherwise drain every outstanding copy
// before the next ds_read, which serialises load and compute); dma_wait_but<N>()
// is the matching wait, placed by hand before the barrier that publishes a tile.
// lds_addr is wave-uniform.
// per-lane source address:
__device__ __forceinline__ void load_to_lds(const void* src, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(lds_addr) : "memory", "m0");
}
// wave-uniform base address + per-lane byte offset (no per-lane 64-bit address
// arithmetic: the offsets inside a full tile are loop invariant):
__device__ __forceinline__ void load_to_lds(const void* base, unsigned voff, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(base), "s"(lds_addr) : "memory", "m0");
}
__device__ __forceinline__ void load_to_lds_dword(const void* base, unsigned voff, unsigned lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" ::"v"(voff), "s"(base), "s"(lds_addr) : "memory", "m0");
}
// Waits until at most N of this wave's vector-memory loads are outstanding.
// Loads return in order, so everything issued before the newest N has landed.
template <int N> __device__ __forceinline__ void dma_wait_but() {
  __builtin_amdgcn_sched_barrier(0);   // keep the consumers of the tile below the wait, the producers above
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// The same wait, and a barrier that does not wait for LDS reads: what was read before it must not be overwritten before the next one.
template <int N> __device__ __forceinline__ void wait_and_sync() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(N) : "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// Between LDS words that lanes of a wave write and other lanes of the same wave read (or the other way round): the
// hardware carries out a wave's LDS operations in order, this keeps the compiler from changing that order.  No
// instruction is emitted.
__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// ---- lane-pair exchanges ----------------------------------------------------
// The 32x32 accumulator splits a column over the lane pair (l, l ^ 32); one VALU
// swap instead of an LDS permute brings the two halves together.
__device__ __forceinline__ float pair_max(float v) {
  const unsigned u = __builtin_bit_cast(unsigned, v);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__builtin_bit_cast(float, (unsigned)r[0]), __builtin_bit_cast(float, (unsigned)r[1]));
}
__device__ __forceinline__ float pair_sum(float v) {
  const unsigned u = __builtin_bit_cast(unsigned, v);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __builtin_bit_cast(float, (unsigned)r[0]) + __builtin_bit_cast(float, (unsigned)r[1]);
}
// The 16x16 accumulator splits a column over the lanes l % 16 of all four rows of 16.
__device__ __forceinline__ float quad_max(float v) {
  const unsigned u = __builtin_bit_cast(unsigned, v);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return pair_max(fmaxf(__builtin_bit_cast(float, (unsigned)r[0]), __builtin_bit_cast(float, (unsigned)r[1])));
}
// The larger value, NaN if either is: v_maximum3_f32 takes operands as they come, where fmaxf has results of matrix instructions and lane swaps
// passed through a v_max of their own first (13 -> 7 instructions for the largest of a quad's 8 scores a lane).
__device__ __forceinline__ float maximum(float a, float b) { return __builtin_elementwise_maximum(a, b); }
__device__ __forceinline__ float quad_maximum(float v) {
  const unsigned u = __builtin_bit_cast(unsigned, v);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const unsigned m = __builtin_bit_cast(unsigned, maximum(__builtin_bit_cast(float, (unsigned)r[0]), __builtin_bit_cast(float, (unsigned)r[1])));
  const auto s = __builtin_amdgcn_permlane32_swap(m, m, false, false);
  return maximum(__builtin_bit_cast(float, (unsigned)s[0]), __builtin_bit_cast(float, (unsigned)s[1]));
}
// the partner lane's value
__device__ __forceinline__ unsigned pair_other(unsigned u) {
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  // after the swap r[0] holds, in lanes >= 32, what lanes < 32 had, and r[1] the converse
  return (threadIdx.x & 32) ? (unsigned)r[0] : (unsigned)r[1];
}

__device__ __forceinline__ double shfl_xor_f64(double v, int m) {
  int lo = __double2loint(v), hi = __double2hiint(v);
  lo = __shfl_xor(lo, m, 64);
  hi = __shfl_xor(hi, m, 64);
  return __hiloint2double(hi, lo);
}

// All-reduce sum over the 32 lanes of a half-wave, fp64, without touching LDS
// memory: two quad permutes, the two row mirrors (DPP moves of both dwords),
// then a swizzle across the 16-lane rows.
template <int CTRL>
__device__ __forceinline__ double dpp_mov_f64(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double half_sum_f64(double v) {
  v += dpp_mov_f64<0xB1>(v);
  v += dpp_mov_f64<0x4E>(v);
  v += dpp_mov_f64<0x141>(v);
  v += dpp_mov_f64<0x140>(v);
  const int lo = __builtin_amdgcn_ds_swizzle(__double2loint(v), 0x401F);
  const int hi = __builtin_amdgcn_ds_swizzle(__double2hiint(v), 0x401F);
  return v + __hiloint2double(hi, lo);
}

// ---- cache update beside another kernel's work --------------------------------
// A work-group takes one item: kMoveItemRows rows of a unit go to where the next step expects them.  All loads of a
// thread (up to 16 pieces of K and of V, their positions) are in flight before its first store.
template <int LPR, int THREADS>   // 16-byte pieces per row
__device__ __forceinline__ void move_rows(const UnitDesc* __restrict__ descs, const GatherArgs& g, int item, int N_k) {
  constexpr int RPP = THREADS / LPR, PASSES = kMoveItemRows / RPP;   // rows per pass
  const int lane = threadIdx.x % LPR;
  const MoveItem it = g.moves[item];
  const UnitDesc d = descs[it.desc];
  const bool gather = d.mode == MOVE_GATHER;
  const int n_rows = gather ? d.n_out : d.n_new;
  const int r0 = it.row0 + (int)threadIdx.x / LPR;
  int s[PASSES];
#pragma unroll
  for (int p = 0; p < PASSES; ++p) {
    const int i = min(r0 + p * RPP, n_rows - 1);
    s[p] = gather ? g.kept[(int64_t)d.unit * g.kept_stride + i] : d.len_in + i;
  }
  uintx4 kr[PASSES], vr[PASSES];
  int pos[PASSES];
#pragma unroll
  for (int p = 0; p < PASSES; ++p) {
    const bool cached = s[p] < d.len_in;
    const int64_t row = cached ? d.in_off + s[p] : (int64_t)d.unit * N_k + (s[p] - d.len_in);
    kr[p] = (static_cast<const uintx4*>(cached ? g.cache.k : g.k_new))[row * LPR + lane];
    vr[p] = (static_cast<const uintx4*>(cached ? g.cache.v : g.v_new))[row * LPR + lane];
    pos[p] = g.pos_new + (s[p] - d.len_in);
    if (cached && g.cache.pos != nullptr) pos[p] = g.cache.pos[row];
  }
  const int64_t dst0 = gather ? d.out_off : d.in_off + d.len_in;
#pragma unroll
  for (int p = 0; p < PASSES; ++p) {
    const int i = r0 + p * RPP;
    if (i < n_rows) {
      static_cast<uintx4*>(g.cache.k)[(dst0 + i) * LPR + lane] = kr[p];
      static_cast<uintx4*>(g.cache.v)[(dst0 + i) * LPR + lane] = vr[p];
      if (g.cache.pos != nullptr && lane == 0) g.cache.pos[dst0 + i] = pos[p];
    }
  }
}

// ---- accumulator layout -----------------------------------------------------
// C = A B with v_mfma_f32_32x32x16_bf16: A operand row = lane % 32, B operand
// column = lane % 32, both holding the 8 contraction elements [16 kk + 8 (lane / 32), +8)
// at step kk.  C register r of lane l is row 8 (r / 4) + 4 (l / 32) + r % 4, column l % 32.
__device__ __forceinline__ int c_row(int r, int half) { return 8 * (r >> 2) + 4 * half + (r & 3); }

// ---- streamed and resident MFMA operands --------------------------------------
// Streams the 32-row blocks of a row-major [n_rows, D] bf16 matrix into an LDS
// ring of 32-row slots (swz_k layout); the WAVES waves of the work-group each copy
// their share of a block (IPW instructions).  Rows past the end repeat the last row.
template <int D, int WAVES>
struct BlockStream {
  static constexpr int CPR = D / 8;               // 16-byte chunks per row
  static constexpr int RPI = 64 / CPR;            // rows per copy instruction
  static constexpr int IPW = (32 / RPI) / WAVES; // copy instructions per wave and block
  static constexpr int BLK = 32 * D;              // elements per block
  const __bf16* base;
  int n_rows, lane, w;
  unsigned lds0;
  unsigned src[IPW];
  __device__ __forceinline__ void init(const __bf16* base_, int n_rows_, const __bf16* ring, int lane_, int w_) {
    base = base_; n_rows = n_rows_; lane = lane_; w = w_;
    lds0 = lds_addr_of(ring);
#pragma unroll
    for (int i = 0; i < IPW; ++i) {
      const int r = (w + i * WAVES) * RPI + lane / CPR, c = lane % CPR;
      src[i] = (unsigned)(r * D + ((c ^ swz_k<D>(r)) & (CPR - 1)) * 8) * 2u;
    }
  }
  // full: the caller knows that all 32 rows of the block exist
  __device__ __forceinline__ void issue(int b, int slot, bool full = false) const {
    const int r0 = b * 32;
    const __bf16* blk = base + (int64_t)r0 * D;
    if (full || r0 + 32 <= n_rows) {
#pragma unroll
      for (int i = 0; i < IPW; ++i)
        load_to_lds(blk, src[i], lds0 + (unsigned)((slot * BLK + (w + i * WAVES) * 512) * 2));
    } else {
#pragma unroll
      for (int i = 0; i < IPW; ++i) {
        const int r = (w + i * WAVES) * RPI + lane / CPR, c = lane % CPR;
        const int rc = min(r, n_rows - 1 - r0);
        load_to_lds(blk, (unsigned)(rc * D + ((c ^ swz_k<D>(r)) & (CPR - 1)) * 8) * 2u,
                       lds0 + (unsigned)((slot * BLK + (w + i * WAVES) * 512) * 2));
      }
    }
  }
};

// Operand fragment of a 32-row block starting at `base` (row-major, D elements per
// row): lane l takes row min(l%32, n_valid-1) (rows past the end repeat the last
// valid one), elements [16kk + 8(l/32), +8) at MFMA step kk.
template <int D>
__device__ __forceinline__ void load_frags(const __bf16* base, int n_valid, int lane, bf16x8 (&f)[D / 16]) {
  const int row = min(lane & 31, n_valid - 1);
  const __bf16* p = base + (int64_t)row * D + 8 * (lane >> 5);
#pragma unroll
  for (int kk = 0; kk < D / 16; ++kk) f[kk] = *reinterpret_cast<const bf16x8*>(p + 16 * kk);
}

// Operand fragment kk of the block in an LDS slot: row lane%32, chunk 2kk + lane/32
template <int D>
__device__ __forceinline__ bf16x8 lds_frag(const __bf16* slot, int col, int half, int kk) {
  constexpr int CPR = D / 8;
  return *reinterpret_cast<const bf16x8*>(&slot[col * D + (((2 * kk + half) ^ swz_k<D>(col)) & (CPR - 1)) * 8]);
}

}  // namespace dev
}  // namespace hack
