// Internal declarations shared by the host side (hack_api.cpp) and the HIP
// kernels of the gfx950 library.  Nothing here is part of the C ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "attn_plan.h"

namespace hack {

// Per-unit launch table entry, built on the host from the caller's host arrays
// and uploaded once per distinct table.  One unit = one (batch, head) pair.
struct alignas(16) UnitDesc {
  int64_t in_off;   // first row of the unit's input rows in the cache arrays
  int64_t out_off;  // first row of its output rows (gather target / attention source)
  int32_t len_in;   // cache rows before this step (L)
  int32_t n_new;    // rows of the current scale that virtually follow them (0 or N_k)
  int32_t n_out;    // rows to produce (gather) or rows attended over
  int32_t keep_a;   // select: rows [0, keep_a) are always kept
  int32_t sel_lo;   // select: ranked segment [sel_lo, sel_hi)
  int32_t sel_hi;
  int32_t sel_m;    // select: how many rows of the ranked segment are kept
  int32_t keep_b;   // select: rows [keep_b, T_in) are always kept
  int32_t mode;     // move kernel: MOVE_* below
  int32_t unit;     // unit id u = b*H + h (rows of q/k_new/out start at u*N_k)
  int32_t pad0;
  int32_t pad1;
};
static_assert(sizeof(UnitDesc) == 64, "UnitDesc must stay 64 bytes");

enum : int32_t { MOVE_NONE = 0, MOVE_APPEND = 1, MOVE_GATHER = 2 };

// One attention work item: a tile of queries of one unit.  It carries copies of the descriptor
// fields the attention kernels read, so that a work-group has one dependent table load in front of
// its first K/V copy instead of two (the small scale steps are pure latency chains).
struct alignas(16) AttnItem {
  int32_t desc;     // index into the UnitDesc table; < 0: padding entry, nothing to do
  int32_t q_tile;   // first query row = q_tile * (rows per tile)
  int32_t unit;     // UnitDesc::unit
  int32_t n_out;    // UnitDesc::n_out
  int64_t out_off;  // UnitDesc::out_off
  int64_t in_off;   // UnitDesc::in_off
  int32_t len_in;   // UnitDesc::len_in
  int32_t mode;     // UnitDesc::mode
  int32_t pad[2];
};
static_assert(sizeof(AttnItem) == 48, "AttnItem must stay 48 bytes");
inline AttnItem make_attn_item(const UnitDesc& d, int desc, int q_tile) {
  AttnItem it{};
  it.desc = desc; it.q_tile = q_tile; it.unit = d.unit; it.n_out = d.n_out; it.out_off = d.out_off; it.in_off = d.in_off;
  it.len_in = d.len_in; it.mode = d.mode;
  return it;
}
inline AttnItem attn_item_padding() { AttnItem it{}; it.desc = -1; return it; }

struct CachePtrs {
  void* k;
  void* v;
  int32_t* pos;
};

// Attention that performs the step's cache update itself: keys and values are read in place, row by row through the
// unit's list of kept rows, while further work-groups of the same launch move those rows to where the next step
// expects them.  An entry of a list is a row of the virtual concatenation [cached rows | rows of the current scale];
// lists ascend, so all but one 32-row block of a unit come from one of the two homes.
constexpr int kMoveItemRows = 128;   // rows per moving work-group
struct alignas(8) MoveItem {
  int32_t desc;   // index into the UnitDesc table
  int32_t row0;   // first of the rows it moves
};
// A whole compressing step of short units in one launch (launch_step_units): every work-group scores and selects for its unit, holds the rows
// that the unit keeps in LDS, moves a share of them and attends for its queries.
struct WholeStep {
  int32_t n_units;
  int32_t max_t, max_rows;  // longest compressing unit with its new rows (at most kWholeStepKeys), most rows a unit attends over
  int32_t queries;          // per work-group: 16, 32, 64, 128 or 256
  int32_t n_obs;
  const int32_t* q_rows;
  int* fault;
  bool moved;               // rows have been moved already: attention over the cache
  int32_t region;           // LDS in front of the list; set by the launcher
};
constexpr int kWholeStepKeys = 1024;
// LDS of such a work-group: the tiles of the scores, the rows or the partial results, whichever is most; the list of kept rows; the rest.
inline size_t whole_step_region(int head_dim, int max_rows) {
  const size_t held = (size_t)(max_rows + 31) / 32 * 32 * head_dim * 4, least = head_dim == 64 ? 65536 : 131072;
  return held > least ? held : least;
}
inline size_t whole_step_lds(int head_dim, int max_rows) {
  return whole_step_region(head_dim, max_rows) + (size_t)(max_rows + 31) / 32 * 32 * 4 + 18432;
}
// Queries per work-group of such a launch, 0 where launches of their own are the better form.  n_comp: compressing units, max_t: longest of them with
// its new rows, max_rows: most rows a unit attends over.  An XCD (32 compute units) takes every eighth unit.
//
// Figures: us a compressing step, launches of their own / this; units of queries, keys, kept rows, all units alike unless said otherwise.
//
// Work-groups of one unit repeat its scores and selection, so a unit gets several only while each of them finds a compute unit of its XCD to itself.
// (queries per work-group) head_dim 64: 4 of 462, 534, 236 13.6 / 12.7 (16), 60 of 64, 166, 102 10.5 / 9.2 (16, 32), 16 of 273, 345, 178 12.5 / 10.6 (32), 43 of
// 134, 776, 81 16.4 / 14.2 (32), 63 of 172, 753, 364 20.8 / 17.7 (64), 42 of 599, 618, 287 19.7 / 17.6 (128); 128: 3 of 310, 318, 175 13.6 / 11.9 (16), 32 of 100,
// 250, 100 13.9 / 11.2 (16), 59 of 142, 573, 256 23.1 / 20.4 (64).  A second round on an XCD costs what the first did: 3 of 567, 581, 95 (head_dim 128)
// 14.6 / 27.5 (16: 36 work-groups on one XCD), 14.6 (32: 18); 27 of 277, 606, 71 (64) 14.5 / 22.8 (32: 36), 13.4 (64: 20).
// With few queries or short lists one work-group for all of a unit's queries, which repeats and merges nothing, is as good as two or three: 90 of 84, 90, 37
// (128) 12.0 (64), 10.3 (256), 142 of 125, 168, 92 (64) 11.0, 9.9; but 37 of 208, 492, 235 (128) 17.2, 20.5, 60 of 137, 403, 377 (64) 14.9, 17.6, 59 of 142, 573, 256 (128)
// 20.4, 23.0.  For few units of many queries launches of their own are as fast, as attention alone fills the chip: in 64s 12 of 658, 688, 186 (128) 19.0 / 20.3,
// 20 of 561, 600, 85 (128) 17.1 / 17.9, 27 of 277, 606, 71 (64) 14.5 / 13.4, over units of lengths of their own up to 40 units on average 1.02 of them at head_dim 128, 0.99 at
// 64 (up to 300 queries 0.97), of more units 0.97; in 128s at head_dim 64 1.02 and 0.95.  Scores of few long units spread over more compute units in launches of
// their own: 3 of 428, 647, 110 (128) 14.3 / 16.3, 4 of 446, 643, 256 (128) 15.7 / 17.4, 8 of 474, 613, 244 (128) 15.9 / 16.3, 2 of 412, 527, 256 (128) 14.8 / 15.6, 17 of
// 17, 655, 256 (128) 15.7 / 17.2, 44 of 12, 891, 256 (128) 18.3 / 19.1, 6 of 392, 642, 158 (64) 13.1 / 13.6, 16 of 700, 1000 (64) 15.8 / 17.1.
//
// Beyond 256 units: one work-group a unit, in rounds.  A compute unit holds two of them at head_dim 64 up to 512 keys and 256 kept rows, otherwise one (LDS,
// registers).  A round that is nearly empty costs as much here as in launches of their own, which wait for the same chains, so most steps gain whatever
// the last round holds: 128, 264, 400, 512, 520 and 768 units of 256, 480, 144 42.7 / 39.3, 55.0 / 43.0, 65.4 / 49.6, 78.4 / 65.4, 99.9 / 79.4, of 256, 1000, 256 77.7 / 62.7,
// 94.4 / 73.0, 98.2 / 84.3, 123 / 97, 151 / 120; 64, 264, 400, 520 and 960 of 140, 512, 256 25.7 / 21.8, 34.2 / 26.2, 43.1 / 37.2, 77.5 / 58.3, of 256, 562, 358 39.7 / 38.4, 47.9 / 43.2,
// 63.8 / 60.1, 112 / 98.  Not so:
// - 128, up to 256 keys, where attention of its own fills its tiles (up to 128 queries) or is short (few rows), unless few units score: 264, 400, 512, 520 and 768 of 100,
//   250, 100 24.1 / 26.7, 28.1 / 28.8, 30.1 / 30.9, 35.0 / 42.1, 43.7 / 46.4, 520 of 200, 250, 60 38.0 / 42.7; 859 of 119, 143, 61 of which half compress 36.3 / 46.0; but 662 of 155, 248,
//   195 of which 71 compress 62.3 / 45.3, 916 of 159, 204, 154 84.5 / 70.7, 298 of 121, 245, 218 of which 94 compress 28.0 / 23.4;
// - 64, one work-group a compute unit though there are few keys: 264, 400, 520 and 960 of 256, 500, 300 29.2 / 34.5, 35.9 / 35.3, 48.0 / 51.5, 86.2 / 82.6; 1051 of 114, 318, 296 of
//   which a quarter compress 34.9 / 47.8;
// - 64, short units of few queries where most compress and the last round is at most half full: 520 of 100, 150, 45 18.6 / 19.8, 600 of 100, 200, 60 18.7 / 19.9, 1092 of
//   39, 163, 96 29.1 / 31.0 (768 of 100, 200, 60 20.0 / 19.7, 597 of 86, 120, 94 of which half compress 22.6 / 15.1);
// - few queries, whose launches are short: 640 of 25, 60 (64) 14.6 / 16.1, 512 of 36, 90 (128) 18.3 / 20.6.
inline int whole_step_queries(int head_dim, int n_units, int n_comp, int N_k, int max_t, int max_rows, int lds_bytes) {
  if (max_t > kWholeStepKeys || whole_step_lds(head_dim, max_rows) > (size_t)lds_bytes) return 0;
  const int longest = head_dim == 64 ? (n_units > 8 ? 640 + 8 * n_units : 640) : n_units > 8 ? 640 + 8 * std::max(n_units - 32, 0) : 512;
  if (max_t > longest) return 0;
  const int per_xcd = (n_units + 7) / 8;
  const auto groups = [&](int queries) { return (int64_t)per_xcd * ((N_k + queries - 1) / queries); };   // of the fullest XCD
  if (groups(16) <= 28) return 16;
  if (groups(32) <= 32) return 32;
  if (N_k > 144 || (N_k > 64 && max_rows > (head_dim == 64 ? 256 : 192))) {
    if (groups(64) <= 32) return n_units > 40 || (head_dim == 64 && N_k <= 300) ? 64 : 0;
    if (groups(128) <= 32) return n_units > 40 || head_dim == 128 ? 128 : 0;
  }
  if (groups(256) <= 32) return 256;
  if (N_k > 256 || N_k <= (head_dim == 64 ? 32 : 96)) return 0;
  if (head_dim == 128) return max_t > 256 || (N_k > 128 && max_rows > 96) || n_comp <= 128 ? 256 : 0;
  if (max_t <= 512 && max_rows > 256) return 0;
  if (max_t <= 256 && N_k <= 112 && n_comp > 512 && (per_xcd - 1) % 64 < 32) return 0;
  return 256;
}
struct GatherArgs {
  const int32_t* kept;     // [unit id, kept_stride] lists of the compressing units
  int64_t kept_stride;
  const int32_t* seam;     // [unit id] how many entries of that list are cached rows
  const int32_t* iota;     // 0, 1, 2, ...: the list of a unit that keeps everything
  const MoveItem* moves;
  int32_t n_moves;         // moving work-groups, the last ones of the launch
  int32_t pos_new;         // position of the current scale's first row
  const void* k_new;
  const void* v_new;
  CachePtrs cache;         // written by the moving work-groups
  bool eight;              // bf16: eight waves a work-group (attn_split_in_eight)
};

// fp32 score: keys per work-group of a launch over n_list units of up to max_t_in keys (see kernels_score.hip for the line
// between the two), and how many work-groups a launch over at most max_units units of at most max_len keys has (sizes the
// workspace).
constexpr int kF32SmallGroups = 640;
inline int64_t score_f32_groups(int n_list, int max_t_in, int chunk) { return (int64_t)n_list * ((max_t_in + chunk - 1) / chunk); }
inline int score_f32_chunk(int n_list, int max_t_in) { return score_f32_groups(n_list, max_t_in, 64) <= kF32SmallGroups ? 64 : 256; }
inline int64_t score_f32_max_groups(int max_units, int max_len) {
  const int64_t small = score_f32_groups(max_units, max_len, 64), large = score_f32_groups(max_units, max_len, 256);
  return small <= kF32SmallGroups ? small : large > kF32SmallGroups ? large : kF32SmallGroups;
}
constexpr int kMaxObs = 32;        // observation queries (one MFMA column block)

// ---- kernel launchers (each validates nothing: the API layer has done so) ----

// Append / gather K, V (and pos) rows.  `descs` has n_desc entries; every entry
// with mode != MOVE_NONE is processed.  max_rows = max over entries of the rows
// it moves.
void launch_move(hipStream_t s, int elem_bytes, int head_dim, const UnitDesc* descs, int n_desc,
                 int max_rows, CachePtrs in, CachePtrs out, const void* k_new, const void* v_new,
                 int N_k, int pos_new, const int32_t* kept_idx, int64_t idx_stride);

// Subset-attention importance, bf16: one launch over `items`, a DEVICE array with
// one entry per chunk of item_keys keys (one of kScoreItemKeys) of every scored unit, each unit
// padded with empty chunks to a multiple of 4 entries (one work-group takes 4
// consecutive entries, which must belong to one unit).  All items of a unit
// must be in the same launch and n_items must not exceed
// score_fused_capacity(head_dim, item_keys) (the waves the device holds at once: the kernel waits
// inside a launch for a unit's items).  slots is a workspace of slot_groups * 32
// 64-bit words per `pos` (slot_groups >= the work-groups of any unit), every word
// all-ones on entry and left all-ones; counters 2 uint32 per `pos`, zero on entry
// and left zero; q_rows DEVICE int32[32]; fault (host-visible int[2]): [0] is set
// if a wait gave up after spin_limit polls, [1] if a logit exceeded the range of
// the parked format.
struct alignas(16) ScoreItem {
  int64_t in_off;    // first row of the unit's cached keys
  int32_t unit;      // u = b*H + h (rows of q/k_new start at u*N_k)
  int32_t len_in;    // cached keys
  int32_t t_in;      // cached + new keys
  int32_t chunk;     // this item covers keys [chunk*keys, (chunk+1)*keys)
  int32_t pos;       // workspace slot of the unit
  int32_t n_groups;  // work-groups (sets of 4 items) of the unit
};
static_assert(sizeof(ScoreItem) == 32, "ScoreItem must stay 32 bytes");
constexpr int kScoreItemKeys[] = {32, 64, 96, 128, 192, 256}, kScoreSizes = 6;   // keys a wave takes
int score_max_groups();   // work-groups per unit the fused kernel's exchange supports
int score_fused_capacity(int head_dim, int item_keys);
// two_pass: two launches (row sums, then importance) that read K twice but never wait inside
// a launch, so n_items may then exceed the resident capacity and other kernels may share the
// device.  abort_flag: DEVICE word, zero in normal operation; a fused launch that gave up its
// wait sets it and later fused launches return at once until the host clears it.
// skip_publish: -1, or (test hook) the work-group of the launch that withholds its sums.
void launch_score_fused(hipStream_t s, int head_dim, int item_keys, bool two_pass, const ScoreItem* items, int n_items,
                        const void* q, const int32_t* q_rows, int n_obs, int N_k, float scale, const void* k_cache,
                        const void* k_new, unsigned long long* slots, int slot_groups, unsigned* counters,
                        float* importance, int64_t imp_stride, int* fault, int spin_limit, const unsigned* abort_flag,
                        int skip_publish);
// The same importance (bf16, two-pass form) with all scratch in a fixed device array of the
// library instead of context memory; no allocation, no host-to-device copy.  At most
// kStaticUnitsMax units per call; the plan travels by value as a kernel argument.
constexpr int kStaticUnitsMax = 64;
struct StaticScorePlan {
  int64_t in_off[kStaticUnitsMax];   // first cached row of each planned unit
  int32_t len_in[kStaticUnitsMax];   // cached rows
  int32_t unit[kStaticUnitsMax];     // u = b*H + h
  int32_t q_rows[kMaxObs];
  int32_t n_units;
  int32_t n_new;                     // rows of k_new that follow the cached ones (0 or N_k)
  int32_t item_keys;                 // keys per wave item, one of kScoreItemKeys
};
int score_static_units_max();
size_t score_static_scratch_bytes();
int score_static_item_count(const StaticScorePlan& plan);
hipError_t score_static_setup(int device);   // once per device: finds the device address of the array
hipError_t launch_score_static(hipStream_t s, int device, int head_dim, const StaticScorePlan& plan, const void* q, int n_obs,
                               int N_k, float scale, const void* k_cache, const void* k_new, float* importance,
                               int64_t imp_stride, int* fault);
// Launches over the n_units units whose descriptors stand at descs.
// fp32: two passes over (chunk of keys, unit); stats is a workspace of 64 doubles per work-group (score_f32_groups).
void launch_score_f32(hipStream_t s, int head_dim, const UnitDesc* descs, int n_units,
                      int max_t_in, const void* q, const int32_t* q_rows, int n_obs, int N_k, float scale,
                      const void* k_cache, const void* k_new, double* stats, float* importance,
                      int64_t imp_stride);

// fp32: score and selection of short units in one launch.  logits: workspace of kF32GroupLogits doubles per work-group of 64 keys
// (score_f32_groups(n_units, max_t_in, 64)); stats as launch_score_f32; counters: 2 uint32 per unit of the launch, zero on entry and
// left zero.
constexpr int kF32GroupLogits = 64 * kMaxObs;
// Where: units of up to 512 keys (one a thread); longer ones, whose work-groups leave room for one on a compute
// unit, as far as all of the launch's are resident at once and the last work-group's walk over the unit is shorter than the launches that it
// saves.  Measured, us a compressing step, three launches / one: head_dim 64, 16 units of 130, 256, 384, 512, 576, 768 keys 19.5 / 16.0,
// 22.0 / 19.2, 24.2 / 22.3, 26.2 / 25.5, 27.5 / 27.1, 30.6 / 31.9; 64 of 512 34.7 / 34.0; 32 of 576 (288 work-groups) 33.8 / 35.0, of 1024
// 41.2 / 55.7; head_dim 128, 16 units of 130, 512, 768, 900, 1024 26.9 / 20.4, 39.4 / 35.6, 47.3 / 45.2, 50.4 / 49.6, 53.7 / 53.6.
constexpr int kF32SmallKeys = 896;    // longest unit of such a launch
inline bool use_score_select_f32(int head_dim, int n_units, int max_t_in) {
  const int64_t groups = score_f32_groups(n_units, max_t_in, 64);
  return max_t_in <= 512 ? groups <= kF32SmallGroups : max_t_in <= (head_dim == 64 ? 576 : kF32SmallKeys) && groups <= 256;
}
inline int64_t score_select_f32_max_groups(int max_units, int max_len) {
  const int64_t n = score_f32_groups(max_units, max_len < kF32SmallKeys ? max_len : kF32SmallKeys, 64);
  return n < kF32SmallGroups ? n : kF32SmallGroups;
}
void launch_score_select_f32(hipStream_t s, int head_dim, const UnitDesc* descs, int n_units, int max_t_in, const void* q,
                             const int32_t* q_rows, int n_obs, int N_k, float scale, const void* k_cache, const void* k_new,
                             double* logits, double* stats, unsigned* counters, int32_t* kept_idx, int64_t idx_stride, int32_t* seam);

// bf16: score and selection of short units in one launch, one work-group per unit, no importance in memory.
bool use_score_select(int head_dim, int n_units, int max_t_in);
// Beyond kScoreSelectHalf keys a unit takes a compute unit for itself (16 waves), up to there two share one.  n_short of n_units units are that
// short: do they get a launch of their own?  Where that spares a round of work-groups over the 256 compute units; a round takes 17 to 19 us
// whichever form it is of.  480 units of 358 keys and 480 of 562: 64.6 -> 18.5 + 38.7 us (kernel trace; a batch of 32 256^2 images 282.1 -> 276.8,
// at half of the cache 295 -> 290).  Launches of their own for units of at most 256 keys, four of which share a compute unit, lose: 300 units of
// 213 and 300 of 281 keys in a schedule of 136.8 us 143.4.
constexpr int kScoreSelectHalf = 512;
// n_append work-groups that append rows ride in the launch of the longer units, or in the only one, where they fill the compute units that its
// last round leaves idle: the round has to be spared with them as well.  264 units of 401 keys, 256 of 824 and 200, 504, 1000 that append (three
// rounds, four and six either way), one launch / two, us a step: 40 rows 61.4 / 59.0, 69.0 / 67.1, 76.2 / 78.5; 124 rows 67.5 / 65.6, 77.3 / 77.5,
// 100.7 / 99.5; 300 rows 85 / 88, 118.5 / 121.6, 170.7 / 174.4.
inline bool split_score_select(int n_units, int n_short, int n_append) {
  auto rounds = [](int n, int at_once) { return (n + at_once - 1) / at_once; };
  auto spared = [&](int more) { return rounds(n_units + more, 256) - rounds(n_short, 512) - rounds(n_units - n_short + more, 256); };
  return n_short > 0 && n_short < n_units && spared(0) > 0 && spared(n_append) > 0;
}
void launch_score_select(hipStream_t s, int head_dim, const UnitDesc* descs, int n_units, int max_t_in,
                         const void* q, const int32_t* q_rows, int n_obs, int N_k, float scale, const void* k_cache,
                         const void* k_new, int32_t* kept_idx, int64_t idx_stride, int32_t* seam, int* fault);

// The same, and the rows of the step moved to where the next step expects them: the kept ones of the n_units compressing units,
// all new ones of the n_append others (launch_move's work).
void launch_score_select_move(hipStream_t s, int head_dim, const UnitDesc* descs, int n_units, const UnitDesc* append_descs, int n_append,
                              int max_t_in, const void* q, const int32_t* q_rows, int n_obs, int N_k, float scale, CachePtrs cache,
                              const void* k_new, const void* v_new, int pos_new, int32_t* kept_idx, int64_t idx_stride, int* fault);

// Budgeted selection; one work-group per unit.  seam[unit id] (or NULL) gets the number of
// kept rows below len_in; every unit must then have new rows.
void launch_select(hipStream_t s, const UnitDesc* descs, int n_units,
                   int max_t_in, const float* importance, int64_t imp_stride, int32_t* kept_idx,
                   int64_t idx_stride, int32_t* seam);

// bf16 attention of N_k queries per unit over rows [out_off, out_off + n_out), work items of 128 queries.
// bf16_kernel: which kernel serves the 128-query work items: the deeper software pipeline, the plain one-block
// pipeline (kept for A/B timing and as a second implementation the tests run over the same shapes), or the deeper one
// with the two halves of a unit's keys side by side in a work-group (head_dim 128; every unit needs more than 32 rows).
constexpr int kAttnTileRows = 128;
enum : int { kAttnPlain = 0, kAttnPipe = 1, kAttnHalves = 2 };
void launch_attn(hipStream_t s, int head_dim, const UnitDesc* descs, const AttnItem* items, int n_items, const void* q,
                 const void* k_cache, const void* v_cache, int N_k, float scale, void* out, int bf16_kernel);
// float32 attention; work items of q_tile_rows = attn_f32_q_tile_rows(units, N_k) queries (16 or 32); fuse != 0
// and its arguments as append in launch_attn_split.
constexpr int kAttnF32SmallItems = 384;   // launches with at most this many 16-query items take those
int attn_f32_q_tile_rows(int n_units, int N_k);
void launch_attn_f32(hipStream_t s, int head_dim, const AttnItem* items, int n_items, int q_tile_rows, const void* q,
                     const void* k_cache, const void* v_cache, const void* k_new, const void* v_new, void* k_app, void* v_app,
                     int32_t* pos_app, int pos_new, int fuse, int N_k, float scale, void* out);
// Over the rows the units keep, read in place through g; g.n_moves further work-groups update the cache.
void launch_attn_f32_gather(hipStream_t s, int head_dim, const UnitDesc* descs, const AttnItem* items, int n_items, int q_tile_rows,
                            const GatherArgs& g, const void* q, const void* k_cache, const void* v_cache, int N_k, float scale,
                            void* out);
// Streamed form of the 128-query bf16 kernel: work-group i serves segs[seg_begin[i] .. seg_begin[i+1]).
// part_o: n_slots * 128 * head_dim floats, part_ml: n_slots * 256 floats, part_count: one zeroed
// counter per cut work item (left zero).  Launches that share these arrays must not overlap.
int attn_stream_slots(int head_dim);   // work-groups the current device holds at once
void launch_attn_stream(hipStream_t s, int head_dim, const UnitDesc* descs, const AttnSeg* segs, const int32_t* seg_begin,
                        int n_groups, const void* q, const void* k_cache, const void* v_cache, int N_k, float scale,
                        void* out, float* part_o, float* part_ml, unsigned* part_count);
// bf16 attention for steps with few queries: work item = (unit, tile of
// attn_split_q_tile_rows() queries), keys split over the waves of a work-group.
// append == false: attends over rows [out_off, out_off + n_out) of k_cache / v_cache.
// append: attends over [rows in_off .. +len_in of the cache | the unit's N_k rows
// of k_new / v_new] (n_out = len_in + N_k) and also writes those rows (and their
// positions pos_new + row, if pos_app != nullptr) behind the cached ones in
// k_app / v_app / pos_app, i.e. it performs the append of the step as well.
// eight, GatherArgs::eight: eight waves a work-group instead of four.
// launch_attn_split_gather: over the rows the units keep (n_out of each), read in place through g; g.n_moves further
// work-groups update the cache.
// Eight waves instead of four halve the blocks that a wave walks one after the other.  At head_dim 128 they leave room for one
// work-group on a compute unit, and below twenty blocks the larger merge costs what the shorter walk gains.  Measured, us a launch,
// four / eight waves, 128 work items of 22, 47, 125 blocks: head_dim 64 7.9 / 7.1, 11.9 / 9.9, 25.4 / 19.4; 128 10.7 / 10.4, 16.6 / 14.6,
// 34.8 / 28.1; 256 items of 13 and 22: 64 6.7 / 6.7, 8.2 / 7.6; 128 9.4 / 9.9, 11.6 / 11.5; 480 items of 22: 10.4 / 11.0; 16.3 / 21.9.
// The work-groups beside them that move a step's rows have the same LDS, so at head_dim 128 they also take a compute unit each, and where
// attention leaves few of those they become a round of their own (a few per unit: units stand for them).  Whole compressing
// steps, four / eight waves, items + units: 192 + 32, 700, 1500, 3000 keys 26.9 / 24.9, 37.1 / 34.7, 56.6 / 48.9 us; 224 + 16 26.7 / 24.9, 35.1 / 31.5,
// 52.9 / 45.8; 224 + 32 27.1 / 27.6, 37.5 / 36.8, 57.2 / 54.0; 192 + 64 30.1 / 30.5, 44.0 / 43.9, 75.0 / 71.4; 256 + 16 26.7 / 27.5, 34.8 / 33.9, 53.6 / 51.3;
// 256 + 32 27.3 / 28.8, 38.3 / 40.2, 58.2 / 59.6; 192 + 96 34.5 / 36.0, 56.4 / 58.0, 110.8 / 113.0; 256 + 64 30.6 / 34.1, 43.3 / 48.9, 73.6 / 80.2
// (moves in a launch in front, eight waves: 700 and 1500 keys of 256 + 32 29.7, 40.7; 3000 of 256 + 64 81.6).
// hack_attn alone would take eight waves on to 256 items (256 + 32: 10.9 / 10.7, 16.3 / 14.7, 26.9 / 24.0), but the number of waves
// decides how the keys are summed, and a step gives the bits of hack_attn over the rows that it kept (unless one launch does all of it: WholeStep).
inline bool attn_split_in_eight(int head_dim, int n_items, int n_units, int max_keys) {
  if (max_keys <= 20 * 32 || n_items > 256) return false;
  const int busy = n_items + n_units;
  return head_dim == 64 || busy <= 240 || (busy <= 272 && max_keys > 32 * 32);
}
int attn_split_q_tile_rows();
void launch_attn_split_gather(hipStream_t s, int head_dim, const UnitDesc* descs, const AttnItem* items, int n_items,
                              const GatherArgs& g, const void* q, const void* k_cache, const void* v_cache, int N_k,
                              float scale, void* out);
void launch_attn_split(hipStream_t s, int head_dim, const UnitDesc* descs, const AttnItem* items, int n_items,
                       const void* q, const void* k_cache, const void* v_cache, const void* k_new, const void* v_new,
                       void* k_app, void* v_app, int32_t* pos_app, int pos_new, bool append, bool eight, int N_k, float scale,
                       void* out);
// A whole step (see WholeStep); kept: the lists of the compressing units are left there too, [unit id, kept_stride].
void launch_step_units(hipStream_t s, int head_dim, const UnitDesc* descs, WholeStep st, const void* q, const CachePtrs& cache, const void* k_new,
                       const void* v_new, int pos_new, int N_k, float scale, void* out, int32_t* kept, int64_t kept_stride);
// Attention variance of the listed units (bf16): sigma[desc.unit] = sum over the
// unit's n_out keys of the population variance, across its N_k queries, of the
// softmax probabilities.  stats: workspace of 2 floats per (unit, query).
void launch_head_variance(hipStream_t s, int head_dim, const UnitDesc* descs, int n_desc, int max_len, const void* q,
                          const void* k_cache, int N_k, float scale, float* stats, double* sigma);
// Final-step merge of the listed units (bf16): every row of the unit's uncompressed cache
// [rows in_off .. +len_in of k_in / v_in | its N_k rows of k_new / v_new] that kept_idx does not
// list is folded into its nearest kept row (cosine similarity of keys) by similarity-weighted
// averaging; the kept rows, which the gather has already written to rows [out_off, out_off + n_out)
// of k_out / v_out, are updated in place.  list[n_list] indexes descs.  nearest / weight /
// inv_norm: workspaces of ws_stride entries per unit id (>= the unit's T_in).
void launch_merge(hipStream_t s, int head_dim, const UnitDesc* descs, const int32_t* list, int n_list, int max_t_in,
                  int max_out, const void* k_in, const void* v_in, const void* k_new, const void* v_new, int N_k,
                  const int32_t* kept_idx, int64_t idx_stride, void* k_out, void* v_out, int32_t* nearest, float* weight,
                  float* inv_norm, int64_t ws_stride);
}  // namespace hack
