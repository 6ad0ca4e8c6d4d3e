// Host side of the C ABI declared in include/hack.h: argument validation, the
// host planner that turns (head class, budget, N_init, N_k) into per-unit launch
// tables, the launch-table cache, the managed double-slab cache of hack_step,
// and the kernel launches.  No device memory is ever read from the host.
#include <algorithm>
#include <cmath>
#include <climits>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <new>
#include <string>
#include <unordered_map>
#include <vector>

#include "../../include/hack.h"
#include "hack_internal.h"
#include "table_cache.h"

using namespace hack;

// ---------------------------------------------------------------------------
// context
// ---------------------------------------------------------------------------
namespace {

constexpr size_t kTableChunkBytes = 32u << 20;   // launch tables: one chunk (device memory + pinned mirror)
constexpr size_t kTableLimitBytes = 1u << 30;    // ... and all chunks of a context together
constexpr int kIotaRows = 32768;                 // rows a unit that keeps everything may have where its list is read
// Polls a score wave spends waiting for the other items of its unit before it gives up.  A poll, an atomic round trip and the shortest sleep,
// takes 0.16 us (launches that give up after 4096 and 16384 polls: 695 and 2662 us), so the wait lasts 96 ms; real ones last a few
// microseconds, longer only where other work keeps the unit's other work-groups from running.
constexpr int kScoreSpinLimit = 600000;

// Launch-table storage in device memory with a pinned host mirror.
struct HipTableBackend {
  bool alloc(size_t bytes, uint8_t** dev, uint8_t** host) {
    if (hipMalloc((void**)dev, bytes) != hipSuccess) return false;
    if (hipHostMalloc((void**)host, bytes, hipHostMallocDefault) != hipSuccess) {
      (void)hipFree(*dev);
      return false;
    }
    return true;
  }
  void release(uint8_t* dev, uint8_t* host) {
    (void)hipFree(dev);
    (void)hipHostFree(host);
  }
  bool upload(uint8_t* dev, const uint8_t* host, size_t bytes, void* stream) {
    return hipMemcpyAsync(dev, host, bytes, hipMemcpyHostToDevice, static_cast<hipStream_t>(stream)) == hipSuccess;
  }
  bool may_alloc(void* stream) {
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    (void)hipStreamIsCapturing(static_cast<hipStream_t>(stream), &cs);
    return cs == hipStreamCaptureStatusNone;
  }
};

}  // namespace

struct hack_ctx {
  hack_config cfg;
  int elem_bytes = 2;
  // workspace
  float* importance = nullptr;   // [max_units, ws_stride]
  int32_t* kept = nullptr;       // [max_units, ws_stride]
  int32_t* seam = nullptr;       // [max_units] kept rows of the step's selection that come from the cache
  int32_t* iota = nullptr;       // [kIotaRows] 0, 1, 2, ...
  double* f32_logits = nullptr;  // fp32 path: [score_select_f32_max_groups, kF32GroupLogits] logits of short units
  double* stats = nullptr;       // fp32 path: [score_f32_max_groups, 32, 2] softmax partials
  unsigned long long* rowstat = nullptr;  // bf16 path: [max_units, score_groups, 32] row-sum exchange slots, all-ones between launches
  unsigned long long* rowstat_side = nullptr;  // the same for the side branch of hack_step (two-pass form: its slots are not re-armed)
  int score_groups = 0;          // work-groups a unit of max_cache_len keys is scored by
  int spin_limit = 0;            // polls after which a score work-group gives up its wait for the unit's other work-groups
  unsigned* abort_flag = nullptr; // bf16 path: device word behind the counters; set by a fused score launch that gave up
  size_t n_slots = 0;            // 64-bit words in rowstat
  int score_mode = HACK_SCORE_FUSED;   // hack_score_mode: fused single launch / two launches without in-kernel waits
  int skip_publish = -1;         // test hook: work-group of a fused score launch that withholds its sums
  unsigned* counters = nullptr;  // [max_units, 2], zero between launches; bf16 path: reader counters, fp32 path: tickets of short units
  float* hv_stats = nullptr;     // head variance: [max_units, max_queries, 2] softmax statistics of every query
  int32_t* merge_nn = nullptr;   // final-step merge (bf16): [max_units, ws_stride] nearest kept row of every cache row
  float* merge_w = nullptr;      //   ... its weight
  float* merge_inv = nullptr;    //   ... inverse key norms of the kept rows
  int* fault = nullptr;          // pinned, device-visible int[2]: [0] a score wave's bounded wait gave up (fatal),
                                 // [1] a logit exceeded the range the bf16 score kernel supports
  int cus = 1;                   // compute units of the device
  int score_capacity[kScoreSizes] = {};   // bf16 path: score items one fused launch may hold (resident waves), by item size (kScoreItemKeys)
  int split_max_items = -1;      // launches with at most this many 32-query attention items use the key-split kernel (HACK_ATTN_SPLIT_ITEMS); -1 (default): see use_split_attention
  int attn_kernel = -1;          // bf16 kernel of the 128-query items (kAttnPlain ...); -1 (default): the deeper pipeline, keys in halves where use_key_halves says so
  // streamed form of that kernel: the launch is cut into equal runs of key blocks, one per resident work-group
  int attn_stream = -1;          // HACK_ATTN_STREAM; -1 (default): cut single work items where the pair model gains, 0: never, 1: equal runs
                                 // for every launch of the 128-query kernel, 2: A/B aid, 4: every cut the model likes (see use_stream_attention)
  int attn_slots = 0;            // work-groups of the streamed kernel the device holds at once
  float* part_o = nullptr;       // [2 * attn_slots, 128, head_dim] unnormalised partial outputs
  float* part_ml = nullptr;      // [2 * attn_slots, 2, 128] their references and normalisers
  unsigned* part_count = nullptr; // [attn_slots] ticket counters, zero between launches
  // hack_step overlap: the compression chain of one group of units runs beside the attention of the other group
  int lds_bytes = 0;             // of a work-group, as the device has it
  bool step_overlap = false;     // off by default (measured slower on MI355X, see step_impl); HACK_STEP_OVERLAP=1 switches it on
  hipStream_t aux_stream = nullptr;
  hipEvent_t ev_fork = nullptr, ev_join = nullptr;
  int64_t ws_stride = 0;
  // launch-table cache: tables keep their device address for the life of the context
  TableCache<HipTableBackend>* tables = nullptr;
  std::string err;
};

// What launching one group of a step's units needs once the launch tables are on the device (sizes, offsets into
// the uploaded table, launch shapes); built by upload_group.
struct StepGroup {
  int n_desc = 0, n_comp = 0, n_merge = 0, n_items = 0, n_stream = 0;   // units, compressing / merging ones, attention work items, streamed work-groups
  int max_t = 0, max_rows = 0, max_keys = 0, merge_t = 0, merge_out = 0;
  bool streamed = false;                  // attention in the streamed form (then n_items is 0)
  bool gathered = false;                  // attention reads the kept rows in place and updates the cache beside it (n_moves work-groups)
  int n_moves = 0;
  int attn_kernel = 0;                    // of the 128-query work items
  int item_keys = 0;
  bool two_pass = false;
  bool small = false;                     // score and selection in one launch
  int whole = 0;                          // queries per work-group of a launch that does the whole step (use_whole_step), 0: none
  int n_short = 0;                        // of the compressing units, the first ones: those of a launch of their own (split_score_select)
  std::vector<int> launches;              // score launch groups
  unsigned long long* slots = nullptr;    // row-sum exchange area of the group's score launches
  const uint8_t* dev = nullptr;
  size_t table = 0;                       // its number in the table store
  size_t o_desc = 0, o_merge = 0, o_rows = 0, o_items = 0, o_sit = 0, o_segs = 0, o_segb = 0, o_moves = 0;
  const UnitDesc* ddev() const { return reinterpret_cast<const UnitDesc*>(dev + o_desc); }
};

// A state of a managed cache (lengths, rows) together with the step that led to it and its launch plan.  The states
// form a tree below the empty cache: a schedule that is repeated (every image, every replay of the same budgets)
// walks the same path again, and a step whose arguments equal those of a child of the current state needs no planning:
// comparing budgets and head classes is all that is left.  (Building descriptors and work lists and hashing the table
// for every step took 230 us at 960 units, against 39 us of kernels.)
struct StepNode {
  // the step: plan inputs besides the parent's state
  int32_t N_k = 0, n_init = 0;
  bool final_merge = false, two_pass = false;
  std::vector<uint8_t> head_type;   // [H]
  std::vector<int32_t> budget;      // [units]
  // its plan
  int n_obs = 0, tile = 0, max_budget = 0;   // max_budget: rows the longest kept-index list needs
  bool split = false, fuse_append = false, two_groups = false;
  bool uploaded = false;            // both tables are on the device (false while only graphs hold their copies)
  StepGroup g[2];
  // the state after it
  std::vector<uint8_t> cur;         // which slab holds the unit's rows
  std::vector<int64_t> off;
  std::vector<int32_t> len;
  std::vector<std::unique_ptr<StepNode>> next;
};
constexpr int kMaxStepNodes = 512;   // per managed cache; beyond that the tree is dropped and grown again

struct hack_kvcache {
  hack_ctx* ctx;
  int32_t n_units;
  std::vector<int32_t> cap;
  std::vector<int64_t> slab[2];
  StepNode root;                    // the empty cache
  std::unique_ptr<StepNode> base;   // current state carried over when the tree was dropped
  const StepNode* at = nullptr;     // current state
  int n_nodes = 0;
  void* k;
  void* v;
  int32_t* pos;
  int64_t rows;
  int64_t tokens_seen;
};

namespace {

hack_status fail(hack_ctx* ctx, hack_status s, const char* fmt, ...) {
  if (ctx) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    try {
      ctx->err = buf;
    } catch (...) {   // no memory for the message: the status says enough
      ctx->err.clear();
    }
  }
  return s;
}

// Ends the body of an entry point that allocates host memory (`try { ... } HACK_NO_THROW(ctx)`): exceptions stop here.
#define HACK_NO_THROW(ctx) \
  catch (...) { return fail(ctx, HACK_EHIP, "out of host memory"); }

#define HIP_TRY(ctx, call)                                                              \
  do {                                                                                  \
    hipError_t e_ = (call);                                                             \
    if (e_ != hipSuccess)                                                               \
      return fail(ctx, HACK_EHIP, "%s failed: %s", #call, hipGetErrorString(e_));      \
  } while (0)

inline int64_t round_up(int64_t x, int64_t a) { return (x + a - 1) / a * a; }
inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// A launch table under construction: sections are appended 64-byte aligned.
struct Table {
  std::vector<uint8_t> bytes;
  template <typename T>
  size_t add(const T* data, size_t count) {
    const size_t off = (bytes.size() + 63) / 64 * 64;
    bytes.resize(off + std::max<size_t>(count, 1) * sizeof(T), 0);
    if (count) memcpy(bytes.data() + off, data, count * sizeof(T));
    return off;
  }
};

// Returns the device address of a table with these contents, uploading it on
// the given stream the first time it is seen (again, if that stream was being
// captured: see table_cache.h).  Tables are immutable and keep their address
// until the context is destroyed, so queued kernels and captured graphs may go
// on using them.
hack_status table_device(hack_ctx* ctx, const Table& t, hipStream_t stream, const uint8_t** dev, size_t* id = nullptr) {
  switch (ctx->tables->get(t.bytes.data(), t.bytes.size(), stream, dev, id)) {
    case TableStatus::kOk: return HACK_OK;
    case TableStatus::kTooLarge:
      return fail(ctx, HACK_ECAPACITY, "launch table of %zu bytes exceeds the %zu-byte table chunk", t.bytes.size(), kTableChunkBytes);
    case TableStatus::kFullDuringCapture:
      return fail(ctx, HACK_ECAPACITY, "launch-table storage is full and cannot grow while the stream is being captured: "
                                       "run the schedule once outside the capture first");
    case TableStatus::kLimit:
      return fail(ctx, HACK_ECAPACITY, "launch tables of this context exceed %zu bytes", kTableLimitBytes);
    case TableStatus::kAllocFailed: return fail(ctx, HACK_EHIP, "allocating launch-table storage failed");
    case TableStatus::kUploadFailed: return fail(ctx, HACK_EHIP, "uploading a launch table failed");
  }
  return HACK_EHIP;
}

// Sec. 4.4 policies as index ranges (see hack_select in hack.h).
void plan_select(int type, int T, int b, int n_init, int n_recent, UnitDesc* d) {
  if (b >= T) {  // identity
    d->keep_a = T; d->sel_lo = T; d->sel_hi = T; d->sel_m = 0; d->keep_b = T;
    return;
  }
  if (type == HACK_CONTEXTUAL) {
    d->keep_a = 0; d->sel_lo = 0; d->sel_hi = T; d->sel_m = b; d->keep_b = T;
    return;
  }
  const int n_rec = std::min(n_recent, T);
  const int n0 = std::max(0, std::min(n_init, T - n_rec));
  const int M = b - n0 - n_rec;
  if (M >= 0) {
    d->keep_a = n0; d->sel_lo = n0; d->sel_hi = T - n_rec; d->sel_m = M; d->keep_b = T - n_rec;
  } else {  // budget below init + recent: init rows, then the best of the recent scale
    const int ka = std::min(n0, b);
    d->keep_a = ka; d->sel_lo = T - n_rec; d->sel_hi = T; d->sel_m = b - ka; d->keep_b = T;
  }
}

// Brings the exchange workspace of the fused score kernel back to its idle state
// (every slot empty, counters and abort word zero).  Synchronises the device.
hipError_t rearm_score_workspace(hack_ctx* ctx) {
  hipError_t e = hipDeviceSynchronize();
  if (e == hipSuccess && ctx->rowstat) e = hipMemset(ctx->rowstat, 0xFF, ctx->n_slots * sizeof(unsigned long long));
  if (e == hipSuccess && ctx->counters) e = hipMemset(ctx->counters, 0, ((size_t)ctx->cfg.max_units * 2 + 64) * sizeof(unsigned));
  if (e == hipSuccess) e = hipDeviceSynchronize();
  return e;
}

// Conditions that kernels of earlier calls found on the device.
hack_status device_report(hack_ctx* ctx) {
  volatile int* f = ctx->fault;
  if (f && f[0]) {
    // A fused score launch gave up its wait (the device did not keep the launch resident as a
    // whole, e.g. because other work held compute units).  Later fused launches have refused to
    // run since.  Recover: drain, re-arm the workspace, and from now on score in two launches
    // that do not wait for each other inside a kernel.
    if (rearm_score_workspace(ctx) != hipSuccess)
      return fail(ctx, HACK_EHIP, "a score launch gave up its wait and the workspace could not be re-armed");
    f[0] = 0;
    ctx->score_mode = HACK_SCORE_TWO_PASS;
    return fail(ctx, HACK_EHIP, "a score launch gave up waiting for a unit's other work-groups: importance (and whatever "
                                "was derived from it) of the calls since the last successful check is incomplete and those "
                                "calls must be issued again; the context has been re-armed and now scores in two passes "
                                "without in-kernel waits");
  }
  if (f && f[1]) {
    f[1] = 0;
    return fail(ctx, HACK_EUNSUPPORTED, "an earlier bf16 score launch met a logit beyond +-354 (scale * q.k); such logits "
                                        "are clamped, so its importance may differ from the definition");
  }
  return HACK_OK;
}

hack_status check_common(hack_ctx* ctx, int32_t B, int32_t N_k, bool need_nk) {
  if (!ctx) return HACK_EINVAL;
  const hack_status dev = device_report(ctx);
  if (dev != HACK_OK) return dev;
  if (B < 1) return fail(ctx, HACK_EINVAL, "B must be >= 1 (got %d)", B);
  if ((int64_t)B * ctx->cfg.heads > ctx->cfg.max_units)
    return fail(ctx, HACK_ECAPACITY, "B*H = %lld exceeds max_units %d", (long long)B * ctx->cfg.heads, ctx->cfg.max_units);
  if (need_nk) {
    if (N_k < 1) return fail(ctx, HACK_EINVAL, "N_k must be >= 1 (got %d)", N_k);
    if (N_k > ctx->cfg.max_queries) return fail(ctx, HACK_ECAPACITY, "N_k = %d exceeds max_queries %d", N_k, ctx->cfg.max_queries);
  }
  return HACK_OK;
}

hack_status check_cache(hack_ctx* ctx, const hack_cache* c, int n_units, const char* name, bool need_v) {
  if (!c) return fail(ctx, HACK_EINVAL, "%s is NULL", name);
  if (!c->k || (need_v && !c->v) || !c->off || !c->len) return fail(ctx, HACK_EINVAL, "%s has a NULL member", name);
  if (!aligned16(c->k) || (c->v && !aligned16(c->v))) return fail(ctx, HACK_EINVAL, "%s k/v must be 16-byte aligned", name);
  if (c->rows < 0) return fail(ctx, HACK_EINVAL, "%s rows < 0", name);
  for (int u = 0; u < n_units; ++u) {
    if (c->len[u] < 0 || c->off[u] < 0 || (c->off[u] & 7) || c->off[u] + c->len[u] > c->rows)
      return fail(ctx, HACK_EINVAL, "%s unit %d: off %lld len %d outside [0, %lld) or off not a multiple of 8", name, u,
                  (long long)c->off[u], c->len[u], (long long)c->rows);
  }
  return HACK_OK;
}

bool scale_ok(float s) { return std::isfinite(s) && s > 0.f; }

// Attention work items: units dealt to the 8 XCDs in order of decreasing length
// (work-group ids are dispatched round-robin over XCDs, so id%8 picks the XCD);
// within an XCD all tiles of a unit are adjacent, so its K/V stay in that XCD's L2.
void build_attn_items(const std::vector<UnitDesc>& descs, int N_k, int tile_rows, std::vector<AttnItem>* items) {
  const int n = (int)descs.size();
  std::vector<int> order(n);
  for (int i = 0; i < n; ++i) order[i] = i;
  // equal lengths: in the order of the units, wherever their descriptors stand
  std::sort(order.begin(), order.end(), [&](int a, int b) {
    return descs[a].n_out != descs[b].n_out ? descs[a].n_out > descs[b].n_out : descs[a].unit < descs[b].unit;
  });
  const int tiles = (N_k + tile_rows - 1) / tile_rows;
  constexpr int X = 8;
  std::vector<AttnItem> per[X];
  int64_t load[X] = {0};
  for (int r = 0; r < n; ++r) {
    int x = 0;
    for (int i = 1; i < X; ++i) if (load[i] < load[x]) x = i;   // least-loaded XCD
    load[x] += (int64_t)descs[order[r]].n_out * tiles;
    for (int t = 0; t < tiles; ++t) per[x].push_back(make_attn_item(descs[order[r]], order[r], t));
  }
  size_t longest = 0;
  for (int x = 0; x < X; ++x) longest = std::max(longest, per[x].size());
  items->assign(longest * X, attn_item_padding());
  for (int x = 0; x < X; ++x)
    for (size_t i = 0; i < per[x].size(); ++i) (*items)[i * X + x] = per[x][i];
}

// Steps with few queries (the early scales) go to the key-split kernel (bf16
// only): its 32-query work items fill the chip where 128-query tiles would not,
// and a step that does not compress then needs no separate append launch.  It is
// used while all of its work items are resident at once or nearly so; beyond
// that the 128-query kernel, which shares every K/V block among four times as
// many queries, is faster.  Whole steps on their own, split / 128 queries, us.  head_dim 128, compressing to 300 and 1943 rows, appending to as
// many: 512 queries, 512 items 29.5 / 31.9, 61.9 / 60.6; 22.5 / 29.4, 40.9 / 40.4; 576, 576 33.8 / 31.9, 76.6 / 66.1; 29.5 / 29.2, 57.8 / 47.6.
// head_dim 64: up to 2048 items, but tiles of 128 queries win earlier where they are nearly full and all start together.  Compressing to 102
// and 1200 rows, appending to as many: 960 queries, 1800 items 32.4 / 29.8, 64.5 / 56.6; 40.0 / 36.9, 64.9 / 54.8; 900, 1450 27.5 / 27.4, 59.3 / 54.3;
// 33.7 / 33.6, 56.2 / 51.0; 512, 1920 30.6 / 29.9, 67.7 / 61.8; 29.7 / 29.8, 56.0 / 46.4; 256, 1920 25.6 / 23.4, 86.6 / 82.9; 24.3 / 26.1, 51.6 / 42.1;
// 256, 1600 24.1 / 22.4, 76.6 / 78.6; 22.6 / 25.8, 45.0 / 41.5; 256, 1440 23.2 / 22.2, 73.1 / 76.9; 21.5 / 24.6, 41.4 / 40.8; 256, 1280 22.6 / 21.9,
// 60.4 / 65.3; 20.4 / 23.6, 37.6 / 40.2.  In two rounds of them or part empty they lose: 576, 1980 31.1 / 31.5, 67.0 / 68.4; 32.0 / 34.9, 57.5 / 58.2;
// 224, 1960 29.1 / 28.7, 94.6 / 97.9; 23.8 / 30.4, 51.9 / 51.0; 140, 2000 28.4 / 30.3, 128.5 / 142.3; 21.7 / 29.2, 49.6 / 60.0.
// (All with 32x32x16 products in the split kernel.  With its present ones, head_dim 128, 32 units, 512 queries, compressing to 300 and 1943 rows, appending
// to 2000 25.4 / 26.1, 52.8 / 58.8; 30.0 / 36.5; 576 31.2 / 26.0, 72.1 / 59.6; to 1500 36.4 / 31.5: the line stands.  head_dim 64, 256 queries, compressing to 1200,
// appending to 1500, 1920 items 75.8 / 82.8; 52.1 / 38.1; 1600 62.6 / 75.0; 50.2 / 36.0; 1440 67.8 / 70.2; 39.8 / 34.4: a compressing step would gain by the split kernel
// what an appending one and more would lose, and one line serves both.  Compressing steps of short units, to 102 rows, mostly leave it: 24.8 / 19.9, in one
// launch 16.2.)
bool use_split_attention(const hack_ctx* ctx, int n_units, int N_k) {
  if (ctx->cfg.dtype != HACK_BF16) return false;
  const int tile = attn_split_q_tile_rows();
  const int64_t items = (int64_t)n_units * ((N_k + tile - 1) / tile);
  if (ctx->split_max_items >= 0) return items <= ctx->split_max_items;
  if (ctx->cfg.head_dim != 64) return items <= 512;
  const int64_t large = (int64_t)n_units * ((N_k + kAttnTileRows - 1) / kAttnTileRows);   // items of 128 queries
  if (N_k > kAttnTileRows && items > (N_k > 512 ? 1400 : 1500) && large <= 512 && 5 * items >= 18 * large) return false;
  return items <= 2048;
}

// Launches of 128-query work items that leave a compute unit one of them take the form that walks the two halves of the keys
// side by side: one work-group alone feeds a compute unit's matrix cores at half of their rate.  Measured, us a launch, whole
// keys / halves (head_dim 128): 256 items of 28, 41, 79 blocks 23.3 / 23.0, 30.5 / 29.0, 51.5 / 47.2; 160 items of 25, 41, 47, 157
// 19.9 / 19.7, 27.7 / 26.2, 30.6 / 29.0, 84.7 / 71.1; of 17 blocks 15.6 / 16.2.  A compute unit holds one such work-group: beyond one per
// compute unit of an XCD it loses (416 items 102 / 110).
// Where few items are long, whole items with the long ones cut over the idle compute units (plan_attn_cuts) are the better form: 144 to 256
// items of 16 to 64 units, a quarter of them of 160 blocks and the rest of 16: 66 to 70 us in halves, 41 to 46 so; half of 80, the rest of 24: 40 to 43
// and 37 to 40; three quarters of 160, the rest of 16: 71 to 78 and 58 to 82.  The rule puts a pair of blocks at a microsecond in halves, and otherwise a
// compute unit at 1.7 blocks in one and 8 for the launch besides.  These rates were fitted to a stage that took longer (a pair now takes 0.78); with the
// present one, over 480 such launches, it picks a form that is 0.2 % slower than the better one on average, 10 % at most (always halves: 13 and 77 %,
// never: 2 and 15 %).
constexpr int kHalvesMinBlocks = 28;
// items: left empty, or the launch's whole work items.
bool use_key_halves(const hack_ctx* ctx, const std::vector<UnitDesc>& descs, int N_k, std::vector<AttnItem>* items) {
  if (ctx->cfg.dtype != HACK_BF16 || ctx->cfg.head_dim != 128 || (ctx->attn_kernel != -1 && ctx->attn_kernel != kAttnHalves) || ctx->attn_stream > 0) return false;
  const bool forced = ctx->attn_kernel == kAttnHalves;
  int longest = 0;
  for (const UnitDesc& d : descs) {
    if (d.n_out <= kAttnKeyBlock) return false;   // either half needs a block
    longest = std::max(longest, d.n_out);
  }
  const int64_t n = (int64_t)descs.size() * ((N_k + kAttnTileRows - 1) / kAttnTileRows);
  if (!forced && (n > ctx->attn_slots / 2 || longest <= (kHalvesMinBlocks - 1) * kAttnKeyBlock)) return false;
  build_attn_items(descs, N_k, kAttnTileRows, items);   // padded to as many for every XCD
  if (forced) return true;
  if ((int)items->size() > ctx->attn_slots / 2) return false;
  int64_t blocks[kAttnXcds] = {0};   // of each XCD
  for (size_t i = 0; i < items->size(); ++i) blocks[i % kAttnXcds] += ((*items)[i].n_out + kAttnKeyBlock - 1) / kAttnKeyBlock;
  // longest / 2 <= blocks / (1.7 compute units) + 8
  const int64_t most = *std::max_element(blocks, blocks + kAttnXcds), cus = ctx->attn_slots / 2 / kAttnXcds;
  return 17 * cus * ((longest + kAttnKeyBlock - 1) / kAttnKeyBlock - 16) <= 20 * most;
}

// Queries per attention work item of a launch.
int attn_tile_rows(const hack_ctx* ctx, int n_units, int N_k) {
  if (ctx->cfg.dtype == HACK_F32) return attn_f32_q_tile_rows(n_units, N_k);
  return use_split_attention(ctx, n_units, N_k) ? attn_split_q_tile_rows() : kAttnTileRows;
}

// The 128-query bf16 kernel in its streamed form: the work items of the launch are cut into one run of
// key blocks per resident work-group (plan_attn_stream), so that every work-group holds the same number of
// blocks whatever the number and the lengths of the work items are; work items that a cut falls into are
// put together from partial results.  OFF by default (HACK_ATTN_STREAM=1 when the context is created
// switches it on for every launch of the 128-query kernel): on MI355X it measured no faster than one work
// item per work-group on any step of the benchmark workloads (1024^2 schedules, scale steps 9-13,
// us per launch, plain / streamed: 16 heads x batch 2: 30 / 37, 48 / 59, 100 / 100, 116 / 135, 186 / 220;
// 32 heads x batch 2: 46 / 53, 65 / 90, 141 / 172, 214 / 254, 356 / 428).  In-kernel time stamps, taken with an earlier
// stage of 32x32x16 instructions, show why: of the two work-groups that share a compute unit the older one is served first and ran the
// steady loop at 0.73-0.76 us per key block, the younger one at 0.97-1.0 (0.55 alone), so equal shares finish
// up to 30 % apart and the launch lasts as long as the slowest; the hardware's own dispatch of whole work
// items absorbs that difference.  On top came about 3 us per extra segment (pipeline fill), 3-4 us per
// partial result written and 3-4 us per part added up.
// `shared` says that another attention launch of the context may run at the same time (the partial-result
// arrays are the context's), which rules the streamed form out.
// What the library does by default (HACK_ATTN_STREAM unset) is narrower: launches whose work items all start
// at once (no more items than resident work-groups) keep whole work items, and plan_attn_cuts halves the few
// whose compute unit would finish last under the measured pair model, if that shortens the modelled launch by
// kCutMinGain.  On the 1024^2 benchmark workloads this fires at scale step 11 with 16 heads x batch 2 (416 work
// items on 256 compute units: the long items that would share a compute unit with another long one are
// halved; 99.8 -> 83.8 us) and at step 9 with 32 heads x batch 2 (46.4 -> 37.9 us).  Launches with more work items than resident work-groups are
// left alone (there the model is 10-15 % off), unless all items are of one length and a few of them make up a last round
// (plan_attn_tail: the whole cache of a 1024^2 image, scale step 12, 250 -> 204 us).  HACK_ATTN_STREAM=0 switches it off, =4 applies every cut
// the model likes (tests).
// The model's rates, us per key block alone / first / second of a pair, are those of the earlier stage; equal pairs take 0.89 a block by them.  The
// present stage takes 0.53 alone and 0.87 in pairs (slopes of 256 and 512 equal items of 50 to 300 blocks).  0.5 / 0.7 / 0.92, 0.5 / 0.78 / 0.85 and
// 8, 10 or 20 blocks for the fixed cost of a piece changed no schedule by more than 0.3 %.
constexpr AttnPairModel kPairModel128{0.55, 0.75, 1.0, 4.0, 14.0};   // and fixed costs in blocks: a whole item, a piece of a cut one
constexpr double kCutMinGain = 0.05;
constexpr int kCutMinBlocks = 8;
constexpr int kStreamOverheadBlocks = 4;   // start and end of a segment, in key blocks of the steady loop
constexpr int kStreamMinBlocks = 4;        // shortest segment a work item is cut into
// items: the launch's whole work items if they are known, else empty; filled where the decision needed them.
bool use_stream_attention(const hack_ctx* ctx, const std::vector<UnitDesc>& descs, int N_k, bool shared, std::vector<AttnItem>* items,
                          AttnStreamPlan* plan) {
  if (ctx->cfg.dtype != HACK_BF16 || ctx->attn_kernel == 0 || ctx->attn_stream == 0 || ctx->attn_slots <= 0 || shared) return false;
  if (descs.empty()) return false;
  const int tile = kAttnTileRows;
  std::vector<int32_t> n_keys(descs.size());
  for (size_t i = 0; i < descs.size(); ++i) n_keys[i] = descs[i].n_out;
  if (ctx->attn_stream == 2) {
    // A/B aid: the streamed kernel on uncut work items, one per work-group, in the order of the plain launch
    if (items->empty()) build_attn_items(descs, N_k, tile, items);
    plan->segs.clear();
    plan->seg_begin.assign(1, 0);
    for (const AttnItem& it : *items) {
      if (it.desc >= 0) plan->segs.push_back(AttnSeg{it.desc, it.q_tile, 0, 0x3fffffff, -1, 0, 0, 0});
      plan->seg_begin.push_back((int32_t)plan->segs.size());
    }
    plan->n_groups = (int)items->size();
    plan->n_parts = plan->n_counters = 0;
    return plan->n_groups > 0;
  }
  if (ctx->attn_stream < 0 || ctx->attn_stream == 4) {
    // whole work items, a few of them cut in two where the pair model says the launch gets shorter (plan_attn_cuts)
    int cus = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, ctx->cfg.device) != hipSuccess || cus < kAttnXcds) return false;
    const bool forced = ctx->attn_stream == 4;
    // the model's constants were measured for head_dim 128, two work-groups per compute unit
    if (!forced && (ctx->cfg.head_dim != 128 || ctx->attn_slots != 2 * cus)) return false;
    if (items->empty()) build_attn_items(descs, N_k, tile, items);
    std::vector<AttnLaneItem> lanes[kAttnXcds];
    for (size_t i = 0; i < items->size(); ++i) {
      const AttnItem& it = (*items)[i];
      if (it.desc >= 0) lanes[i % kAttnXcds].push_back(AttnLaneItem{it.desc, it.q_tile, (it.n_out + kAttnKeyBlock - 1) / kAttnKeyBlock});
    }
    double before = 0.0, after = 0.0;
    if (!(!forced && plan_attn_tail(lanes, cus / kAttnXcds, plan)) &&
        !plan_attn_cuts(lanes, cus / kAttnXcds, kCutMinBlocks, kPairModel128, forced ? 1e-9 : kCutMinGain, plan, &before, &after)) return false;
    return plan->n_groups > 0 && plan->n_parts <= 2 * ctx->attn_slots && plan->n_counters <= ctx->attn_slots;
  }
  plan_attn_stream(n_keys.data(), (int)descs.size(), (N_k + tile - 1) / tile, ctx->attn_slots, kStreamOverheadBlocks,
                   kStreamMinBlocks, plan);
  return plan->n_groups > 0 && plan->n_parts <= 2 * ctx->attn_slots && plan->n_counters <= ctx->attn_slots;
}

// One score work item per chunk of each of the first n units, longest units first so the
// tail of a launch is made of short units.  All items of a unit go into the same
// launch group and no group exceeds `capacity` items; group_begin gets the first
// item of every group plus the total as its last entry.
void build_score_items(const std::vector<UnitDesc>& descs, int n, int item_keys, int capacity,
                       std::vector<ScoreItem>* items, std::vector<int>* group_begin) {
  items->clear();
  group_begin->assign(1, 0);
  std::vector<int> order(n);
  for (int i = 0; i < n; ++i) order[i] = i;
  auto t_in = [&](int pos) { return descs[pos].len_in + descs[pos].n_new; };
  std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return t_in(a) > t_in(b); });
  auto groups = [&](int pos) { return ((t_in(pos) + item_keys - 1) / item_keys + 3) / 4; };   // 4 items per work-group, same unit
  size_t n_items = 0;
  for (int pos : order) n_items += 4 * groups(pos);
  items->reserve(n_items);
  for (int pos : order) {
    const UnitDesc& d = descs[pos];
    const int wgs = groups(pos);
    if ((int)items->size() - group_begin->back() + 4 * wgs > capacity) group_begin->push_back((int)items->size());
    for (int c = 0; c < 4 * wgs; ++c)
      items->push_back(ScoreItem{d.in_off, d.unit, d.len_in, t_in(pos), c, pos, wgs});
  }
  group_begin->push_back((int)items->size());
}

// bf16: keys per score item (wave) for units of these many keys.
// Smaller items spread a launch over more compute units and shorten every wave's serial tile work, so the
// smallest size is taken whose items all fit one launch (the fused kernel's work-groups wait for each other
// inside a launch, so a launch holds at most what the device keeps resident) and whose work-groups per unit the
// exchange area supports; if no size fits one launch, the size that needs the fewest launches.  A wave's tiles take some 1.7 us each, one after
// the other, hence sizes between the powers of two.  Without / with those of 96 and 192 keys, us a launch, head_dim 128: 32 units of 3543 or 5485
// keys 16.8 / 15.2, of 4247 or 6189 17.2 / 15.9, 64 of 3883 or 7039 33.8 / 29.5; in two passes 26.0 / 23.0, 26.7 / 24.5, 48.0 / 43.5; 200 units of
// 1200 or 1500, head_dim 64, 23.8 / 19.6.
// At head_dim 64 a compute unit holds two work-groups of 128-key and 256-key items, three of 96-key and 192-key ones, four of 64-key ones, so items
// of 192 keys spare a launch, or fit one, by putting a third work-group of many tiles on a compute unit; that takes as long as the launch spared.
// They are taken instead of 256 where they spare a launch or put no more work-groups on a compute unit in the last one, and of no other
// size; nor do single-tile items in two launches stand in for them.  Time of 192 over the other, graph replays, fused / two passes, launches and work-groups a
// compute unit in the last one: 256 for 192, one launch, 2 for 2 0.82 / 0.82, 3 for 2 up to 1.10 / 1.11; two for three 0.70 to 0.80 / 0.80 to 0.86; two, 3 for 1 1.17 /
// 1.15; three, 2 for 1 1.06 / 1.01; one launch against two of 64 0.96 to 1.02 / 1.12 to 1.17, two against three 1.09 to 1.14 / 1.18 to 1.24; one against
// two of 96 0.96 / 1.07, two against three 1.10 to 1.30 / 1.12 to 1.31; two launches of 32 over two of 64 1.12 to 1.20 / 1.08 to 1.11.
// The choice does not depend on the score mode, so both modes (and the fixed-scratch entry point, which applies the same
// rule) group the keys alike and give the same bits.
int choose_score_item_keys(const hack_ctx* ctx, std::vector<int> t_in) {
  // lengths in the order build_score_items fills launches in, each with the number of its units (most units share a few lengths: six sizes over
  // 609 units of two cost a call of hack_score 10 us one unit at a time)
  std::sort(t_in.begin(), t_in.end(), [](int a, int b) { return a > b; });
  std::vector<std::pair<int, long>> lengths;
  for (int t : t_in) {
    if (lengths.empty() || lengths.back().first != t) lengths.push_back({t, 0});
    ++lengths.back().second;
  }
  struct Size { int keys; long launches, last; };   // last: work-groups of the last launch
  auto choose = [&](bool others) {
    Size best{256, 0, 0};
    for (int i = 0; i < kScoreSizes; ++i) {
      const int keys = kScoreItemKeys[i], cap = ctx->score_capacity[i] / 4;
      if (cap <= 0 || (others && (keys == 192 || keys == 32))) continue;
      Size x{keys, 1, 0};
      bool fits = true;
      for (const auto& run : lengths) {
        const long wgs = ((run.first + keys - 1) / keys + 3) / 4;
        if (wgs > score_max_groups() || wgs > cap) { fits = false; break; }
        long left = run.second;
        while (left > (cap - x.last) / wgs) {
          left -= (cap - x.last) / wgs;
          ++x.launches;
          x.last = 0;
        }
        x.last += left * wgs;
      }
      if (!fits) continue;
      if (x.launches <= 1) return x;
      if (best.launches == 0 || x.launches < best.launches) best = x;
    }
    return best;
  };
  Size x = choose(false);
  if (x.keys == 192 && ctx->cfg.head_dim == 64) {
    const Size y = choose(true);
    auto per_cu = [&](long groups) { return (groups + ctx->cus - 1) / ctx->cus; };
    if (y.keys != 256 || (x.launches == y.launches && per_cu(x.last) > per_cu(y.last))) x = y;
  }
  return x.keys;
}

// Builds the item list of the first n units for the size chosen: launch groups for the fused form, one group for the two-pass
// form (no in-kernel wait: one launch pair holds any number of items).
int plan_score_items(const hack_ctx* ctx, const std::vector<UnitDesc>& descs, int n, bool two_pass, std::vector<ScoreItem>* items,
                     std::vector<int>* group_begin) {
  std::vector<int> t_in;
  for (int i = 0; i < n; ++i) t_in.push_back(descs[i].len_in + descs[i].n_new);
  const int keys = choose_score_item_keys(ctx, std::move(t_in));
  int idx = 0;
  while (kScoreItemKeys[idx] != keys) ++idx;
  build_score_items(descs, n, keys, two_pass ? INT32_MAX : ctx->score_capacity[idx], items, group_begin);
  return keys;
}

// Scores units whose descriptors are on the device already.
void run_score(hack_ctx* ctx, hipStream_t s, bool two_pass, unsigned long long* slots, const UnitDesc* ddev, int n_units, int max_t,
               const ScoreItem* items_dev, int item_keys, const std::vector<int>& group_begin, const void* q,
               const int32_t* rows_dev, int n_obs, int N_k, float scale, const void* k_cache, const void* k_new,
               float* importance, int64_t imp_stride) {
  if (ctx->cfg.dtype == HACK_F32) {
    launch_score_f32(s, ctx->cfg.head_dim, ddev, n_units, max_t, q, rows_dev, n_obs, N_k, scale, k_cache, k_new,
                     ctx->stats, importance, imp_stride);
    return;
  }
  for (size_t g = 0; g + 1 < group_begin.size(); ++g)
    launch_score_fused(s, ctx->cfg.head_dim, item_keys, two_pass, items_dev + group_begin[g],
                       group_begin[g + 1] - group_begin[g], q, rows_dev, n_obs, N_k, scale, k_cache, k_new, slots,
                       ctx->score_groups, ctx->counters, importance, imp_stride, ctx->fault, ctx->spin_limit, ctx->abort_flag,
                       ctx->skip_publish);
}

void fill_q_rows(const int32_t* q_idx, int n_obs, int N_k, int32_t* rows) {
  for (int i = 0; i < kMaxObs; ++i) rows[i] = 0;
  for (int i = 0; i < n_obs; ++i) rows[i] = q_idx ? q_idx[i] : (int32_t)(((int64_t)i * N_k) / n_obs);
}

}  // namespace

// ---------------------------------------------------------------------------
// life cycle
// ---------------------------------------------------------------------------
extern "C" const char* hack_strerror(hack_status s) {
  switch (s) {
    case HACK_OK: return "ok";
    case HACK_EINVAL: return "invalid argument";
    case HACK_ECAPACITY: return "capacity exceeded";
    case HACK_EUNSUPPORTED: return "unsupported";
    case HACK_EHIP: return "HIP runtime error";
  }
  return "unknown status";
}

extern "C" const char* hack_last_error(const hack_ctx* ctx) { return ctx ? ctx->err.c_str() : "NULL context"; }

extern "C" hack_status hack_check(hack_ctx* ctx) {
  if (!ctx) return HACK_EINVAL;
  return device_report(ctx);
}

extern "C" hack_status hack_set_score_mode(hack_ctx* ctx, int32_t mode) {
  if (!ctx) return HACK_EINVAL;
  if (mode != HACK_SCORE_FUSED && mode != HACK_SCORE_TWO_PASS) return fail(ctx, HACK_EINVAL, "unknown score mode %d", mode);
  if (mode == ctx->score_mode) return HACK_OK;
  // the two forms leave the exchange slots in different states: start the other one from a clean workspace
  if (rearm_score_workspace(ctx) != hipSuccess) return fail(ctx, HACK_EHIP, "re-arming the score workspace failed");
  ctx->score_mode = mode;
  return HACK_OK;
}

extern "C" int32_t hack_get_score_mode(const hack_ctx* ctx) { return ctx ? ctx->score_mode : (int32_t)HACK_EINVAL; }

extern "C" hack_status hack_create(hack_ctx** out, const hack_config* cfg) {
  if (!out || !cfg) return HACK_EINVAL;
  *out = nullptr;
  if (cfg->head_dim != 64 && cfg->head_dim != 128) return HACK_EINVAL;
  if (cfg->dtype != HACK_BF16 && cfg->dtype != HACK_F32) return HACK_EINVAL;
  if (cfg->heads < 1 || cfg->max_units < cfg->heads || cfg->max_cache_len < 1 || cfg->max_queries < 1) return HACK_EINVAL;
  if (cfg->n_obs < 1 || cfg->n_obs > kMaxObs) return HACK_EINVAL;
  if (cfg->max_cache_len > 32768) return HACK_EUNSUPPORTED;  // selection: 1024 threads of 32 keys in registers
  hack_ctx* ctx = new (std::nothrow) hack_ctx();
  if (!ctx) return HACK_EHIP;
  ctx->cfg = *cfg;
  ctx->elem_bytes = cfg->dtype == HACK_F32 ? 4 : 2;
  ctx->ws_stride = round_up(cfg->max_cache_len, 64);
  ctx->spin_limit = kScoreSpinLimit;
  // test hook: a tiny limit makes the score kernel's bounded wait give up (every work-group still exits normally)
  if (const char* v = std::getenv("HACK_SCORE_SPIN_LIMIT")) ctx->spin_limit = std::max(0, std::atoi(v));
  // test hook: this work-group of every fused score launch does not publish its row sums, so the work-groups of its
  // unit run into the (tiny) spin limit deterministically
  if (const char* v = std::getenv("HACK_SCORE_TEST_SKIP_PUBLISH")) ctx->skip_publish = std::atoi(v);
  if (const char* v = std::getenv("HACK_SCORE_MODE")) ctx->score_mode = std::atoi(v) == 1 ? HACK_SCORE_TWO_PASS : HACK_SCORE_FUSED;
  if (const char* v = std::getenv("HACK_ATTN_SPLIT_ITEMS")) ctx->split_max_items = std::max(std::atoi(v), 0);   // tuning / test override
  if (const char* v = std::getenv("HACK_STEP_OVERLAP")) ctx->step_overlap = std::atoi(v) != 0;
  if (const char* v = std::getenv("HACK_ATTN_PIPE")) ctx->attn_kernel = std::min(std::max(std::atoi(v), 0), 2);   // A/B and test override
  if (const char* v = std::getenv("HACK_ATTN_STREAM")) ctx->attn_stream = std::atoi(v);       // A/B and test override
  hipError_t e = hipSetDevice(cfg->device);
  const size_t n_ws = (size_t)cfg->max_units * ctx->ws_stride;
  if (e == hipSuccess) e = hipMalloc((void**)&ctx->importance, n_ws * sizeof(float));
  if (e == hipSuccess) e = hipMalloc((void**)&ctx->kept, n_ws * sizeof(int32_t));
  if (e == hipSuccess) e = hipMalloc((void**)&ctx->seam, (size_t)cfg->max_units * sizeof(int32_t));
  if (e == hipSuccess) e = hipMalloc((void**)&ctx->iota, kIotaRows * sizeof(int32_t));
  if (e == hipSuccess) {
    std::unique_ptr<int32_t[]> rows(new (std::nothrow) int32_t[kIotaRows]);
    for (int i = 0; rows && i < kIotaRows; ++i) rows[i] = i;
    e = rows ? hipMemcpy(ctx->iota, rows.get(), kIotaRows * sizeof(int32_t), hipMemcpyHostToDevice) : hipErrorOutOfMemory;
  }
  if (e == hipSuccess && cfg->dtype == HACK_F32)
    e = hipMalloc((void**)&ctx->f32_logits, (size_t)score_select_f32_max_groups(cfg->max_units, cfg->max_cache_len) * kF32GroupLogits * sizeof(double));
  if (e == hipSuccess && cfg->dtype == HACK_F32)
    e = hipMalloc((void**)&ctx->stats, (size_t)score_f32_max_groups(cfg->max_units, cfg->max_cache_len) * kMaxObs * 2 * sizeof(double));
  ctx->score_groups = score_max_groups();   // exchange slots per unit: enough for every item size
  const size_t n_slots = (size_t)cfg->max_units * ctx->score_groups * kMaxObs;
  ctx->n_slots = n_slots;
  if (e == hipSuccess) e = hipMalloc((void**)&ctx->rowstat, n_slots * sizeof(unsigned long long));
  if (e == hipSuccess && cfg->dtype == HACK_BF16) e = hipMalloc((void**)&ctx->rowstat_side, n_slots * sizeof(unsigned long long));
  const size_t n_counters = (size_t)cfg->max_units * 2 + 64;   // per-unit reader counters, then the abort word
  if (e == hipSuccess) e = hipMalloc((void**)&ctx->counters, n_counters * sizeof(unsigned));
  if (e == hipSuccess) e = hipMemset(ctx->counters, 0, n_counters * sizeof(unsigned));
  if (e == hipSuccess) ctx->abort_flag = ctx->counters + (size_t)cfg->max_units * 2;
  if (e == hipSuccess && cfg->dtype == HACK_BF16)
    e = hipMalloc((void**)&ctx->hv_stats, (size_t)cfg->max_units * cfg->max_queries * 2 * sizeof(float));
  if (e == hipSuccess && cfg->dtype == HACK_BF16) e = hipMalloc((void**)&ctx->merge_nn, n_ws * sizeof(int32_t));
  if (e == hipSuccess && cfg->dtype == HACK_BF16) e = hipMalloc((void**)&ctx->merge_w, n_ws * sizeof(float));
  if (e == hipSuccess && cfg->dtype == HACK_BF16) e = hipMalloc((void**)&ctx->merge_inv, n_ws * sizeof(float));
  if (e == hipSuccess && cfg->dtype == HACK_BF16) {
    ctx->attn_slots = attn_stream_slots(cfg->head_dim);
    if (hipDeviceGetAttribute(&ctx->lds_bytes, hipDeviceAttributeMaxSharedMemoryPerBlock, cfg->device) != hipSuccess) ctx->lds_bytes = 0;
    const size_t n_part = 2 * (size_t)std::max(ctx->attn_slots, 1);
    e = hipMalloc((void**)&ctx->part_o, n_part * 128 * cfg->head_dim * sizeof(float));
    if (e == hipSuccess) e = hipMalloc((void**)&ctx->part_ml, n_part * 256 * sizeof(float));
    if (e == hipSuccess) e = hipMalloc((void**)&ctx->part_count, (n_part / 2) * sizeof(unsigned));
    if (e == hipSuccess) e = hipMemset(ctx->part_count, 0, (n_part / 2) * sizeof(unsigned));
  }
  if (e == hipSuccess) e = hipHostMalloc((void**)&ctx->fault, 2 * sizeof(int), hipHostMallocDefault);
  if (e == hipSuccess) ctx->fault[0] = ctx->fault[1] = 0;
  if (e == hipSuccess) e = hipMemset(ctx->rowstat, 0xFF, n_slots * sizeof(unsigned long long));   // every slot empty
  if (e == hipSuccess) e = hipDeviceSynchronize();
  if (e == hipSuccess) {
    try {
      ctx->tables = new TableCache<HipTableBackend>(HipTableBackend{}, kTableChunkBytes, kTableLimitBytes);
      if (!ctx->tables->reserve_first_chunk()) e = hipErrorOutOfMemory;
    } catch (...) {
      e = hipErrorOutOfMemory;
    }
  }
  if (e == hipSuccess) e = hipStreamCreateWithFlags(&ctx->aux_stream, hipStreamNonBlocking);   // default priority
  if (e == hipSuccess) e = hipEventCreateWithFlags(&ctx->ev_fork, hipEventDisableTiming);
  if (e == hipSuccess) e = hipEventCreateWithFlags(&ctx->ev_join, hipEventDisableTiming);
  if (e == hipSuccess) e = score_static_setup(cfg->device);   // device address of the library's fixed scratch array
  if (e == hipSuccess && cfg->dtype == HACK_BF16) {
    // a unit's score items wait for each other inside one launch, so a launch may
    // hold at most as many items as the device keeps resident at once
    for (int i = 0; i < kScoreSizes; ++i) ctx->score_capacity[i] = score_fused_capacity(cfg->head_dim, kScoreItemKeys[i]);
    if (hipDeviceGetAttribute(&ctx->cus, hipDeviceAttributeMultiprocessorCount, cfg->device) != hipSuccess || ctx->cus < 1) ctx->cus = 1;
    // the largest unit must fit one launch with the largest items
    const int per_unit = (cfg->max_cache_len + 255) / 256 + 3;
    if (ctx->score_capacity[kScoreSizes - 1] < per_unit || (per_unit + 3) / 4 > score_max_groups()) e = hipErrorInvalidConfiguration;
  }
  if (e != hipSuccess) {
    hack_destroy(ctx);
    return HACK_EHIP;
  }
  *out = ctx;
  return HACK_OK;
}

extern "C" void hack_destroy(hack_ctx* ctx) {
  if (!ctx) return;
  if (ctx->importance) (void)hipFree(ctx->importance);
  if (ctx->kept) (void)hipFree(ctx->kept);
  if (ctx->seam) (void)hipFree(ctx->seam);
  if (ctx->iota) (void)hipFree(ctx->iota);
  if (ctx->f32_logits) (void)hipFree(ctx->f32_logits);
  if (ctx->stats) (void)hipFree(ctx->stats);
  if (ctx->rowstat) (void)hipFree(ctx->rowstat);
  if (ctx->rowstat_side) (void)hipFree(ctx->rowstat_side);
  if (ctx->counters) (void)hipFree(ctx->counters);
  if (ctx->fault) (void)hipHostFree(ctx->fault);
  if (ctx->hv_stats) (void)hipFree(ctx->hv_stats);
  if (ctx->merge_nn) (void)hipFree(ctx->merge_nn);
  if (ctx->merge_w) (void)hipFree(ctx->merge_w);
  if (ctx->merge_inv) (void)hipFree(ctx->merge_inv);
  if (ctx->part_o) (void)hipFree(ctx->part_o);
  if (ctx->part_ml) (void)hipFree(ctx->part_ml);
  if (ctx->part_count) (void)hipFree(ctx->part_count);
  if (ctx->ev_fork) (void)hipEventDestroy(ctx->ev_fork);
  if (ctx->ev_join) (void)hipEventDestroy(ctx->ev_join);
  if (ctx->aux_stream) (void)hipStreamDestroy(ctx->aux_stream);
  delete ctx->tables;
  delete ctx;
}

// ---------------------------------------------------------------------------
// a1: score
// ---------------------------------------------------------------------------
extern "C" hack_status hack_score(hack_ctx* ctx, int32_t B, int32_t N_k, const void* q, const int32_t* q_idx,
                                  int32_t n_obs, float scale, const hack_cache* in, const void* k_new,
                                  const uint8_t* active, float* importance, int64_t imp_stride,
                                  hack_stream stream) try {
  hack_status st = check_common(ctx, B, N_k, true);
  if (st != HACK_OK) return st;
  const int U = B * ctx->cfg.heads;
  if (!q || !importance) return fail(ctx, HACK_EINVAL, "q and importance must not be NULL");
  if (!aligned16(q) || (k_new && !aligned16(k_new))) return fail(ctx, HACK_EINVAL, "q/k_new must be 16-byte aligned");
  if (n_obs < 1 || n_obs > ctx->cfg.n_obs || n_obs > N_k)
    return fail(ctx, HACK_EINVAL, "n_obs = %d outside [1, min(%d, N_k = %d)]", n_obs, ctx->cfg.n_obs, N_k);
  if (!scale_ok(scale)) return fail(ctx, HACK_EINVAL, "scale must be finite and > 0");
  if (q_idx)
    for (int i = 0; i < n_obs; ++i)
      if (q_idx[i] < 0 || q_idx[i] >= N_k) return fail(ctx, HACK_EINVAL, "q_idx[%d] = %d outside [0, %d)", i, q_idx[i], N_k);
  if ((st = check_cache(ctx, in, U, "in", false)) != HACK_OK) return st;
  const int n_new = k_new ? N_k : 0;
  std::vector<UnitDesc> descs;
  int max_t = 0;
  for (int u = 0; u < U; ++u) {
    if (active && !active[u]) continue;
    const int64_t T = (int64_t)in->len[u] + n_new;
    if (T < 1) return fail(ctx, HACK_EINVAL, "unit %d has no keys to score", u);
    if (T > ctx->cfg.max_cache_len) return fail(ctx, HACK_ECAPACITY, "unit %d: T_in = %lld exceeds max_cache_len %d", u, (long long)T, ctx->cfg.max_cache_len);
    if (T > imp_stride) return fail(ctx, HACK_ECAPACITY, "imp_stride %lld < T_in %lld of unit %d", (long long)imp_stride, (long long)T, u);
    UnitDesc d{};
    d.in_off = in->off[u]; d.out_off = in->off[u]; d.len_in = in->len[u]; d.n_new = n_new; d.n_out = (int)T; d.unit = u;
    descs.push_back(d);
    max_t = std::max(max_t, (int)T);
  }
  if (descs.empty()) return HACK_OK;
  int32_t rows[kMaxObs];
  fill_q_rows(q_idx, n_obs, N_k, rows);
  std::vector<ScoreItem> sitems;
  std::vector<int> groups;
  int item_keys = 0;
  const bool two_pass = ctx->score_mode == HACK_SCORE_TWO_PASS;
  if (ctx->cfg.dtype == HACK_BF16) item_keys = plan_score_items(ctx, descs, (int)descs.size(), two_pass, &sitems, &groups);
  Table t;
  const size_t o_desc = t.add(descs.data(), descs.size());
  const size_t o_rows = t.add(rows, kMaxObs);
  const size_t o_sit = t.add(sitems.data(), sitems.size());
  const uint8_t* dev;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if ((st = table_device(ctx, t, s, &dev)) != HACK_OK) return st;
  run_score(ctx, s, two_pass, ctx->rowstat, (const UnitDesc*)(dev + o_desc), (int)descs.size(), max_t,
            (const ScoreItem*)(dev + o_sit), item_keys, groups, q, (const int32_t*)(dev + o_rows), n_obs, N_k, scale, in->k, k_new,
            importance, imp_stride);
  HIP_TRY(ctx, hipGetLastError());
  return HACK_OK;
} HACK_NO_THROW(ctx)

extern "C" int32_t hack_score_item_keys(const hack_ctx* ctx, int32_t n, const int32_t* t_in) try {
  if (!ctx || n < 1 || !t_in) return HACK_EINVAL;
  if (ctx->cfg.dtype != HACK_BF16) return 0;
  for (int i = 0; i < n; ++i)
    if (t_in[i] < 1 || t_in[i] > ctx->cfg.max_cache_len) return HACK_EINVAL;
  return choose_score_item_keys(ctx, std::vector<int>(t_in, t_in + n));
} catch (...) { return HACK_EHIP; }

// The same call for callers that cannot allocate (see hack.h): scratch in the library's fixed device array.
extern "C" hack_status hack_score_static(hack_ctx* ctx, int32_t B, int32_t N_k, const void* q, const int32_t* q_idx,
                                         int32_t n_obs, float scale, const hack_cache* in, const void* k_new,
                                         const uint8_t* active, float* importance, int64_t imp_stride,
                                         hack_stream stream) try {
  hack_status st = check_common(ctx, B, N_k, true);
  if (st != HACK_OK) return st;
  if (ctx->cfg.dtype != HACK_BF16) return fail(ctx, HACK_EUNSUPPORTED, "hack_score_static is implemented for bf16 contexts");
  const int U = B * ctx->cfg.heads;
  if (!q || !importance) return fail(ctx, HACK_EINVAL, "q and importance must not be NULL");
  if (!aligned16(q) || (k_new && !aligned16(k_new))) return fail(ctx, HACK_EINVAL, "q/k_new must be 16-byte aligned");
  if (n_obs < 1 || n_obs > ctx->cfg.n_obs || n_obs > N_k)
    return fail(ctx, HACK_EINVAL, "n_obs = %d outside [1, min(%d, N_k = %d)]", n_obs, ctx->cfg.n_obs, N_k);
  if (!scale_ok(scale)) return fail(ctx, HACK_EINVAL, "scale must be finite and > 0");
  if (q_idx)
    for (int i = 0; i < n_obs; ++i)
      if (q_idx[i] < 0 || q_idx[i] >= N_k) return fail(ctx, HACK_EINVAL, "q_idx[%d] = %d outside [0, %d)", i, q_idx[i], N_k);
  if ((st = check_cache(ctx, in, U, "in", false)) != HACK_OK) return st;
  StaticScorePlan plan{};
  plan.n_new = k_new ? N_k : 0;
  for (int u = 0; u < U; ++u) {
    if (active && !active[u]) continue;
    const int64_t T = (int64_t)in->len[u] + plan.n_new;
    if (T < 1) return fail(ctx, HACK_EINVAL, "unit %d has no keys to score", u);
    if (T > ctx->cfg.max_cache_len) return fail(ctx, HACK_ECAPACITY, "unit %d: T_in = %lld exceeds max_cache_len %d", u, (long long)T, ctx->cfg.max_cache_len);
    if (T > imp_stride) return fail(ctx, HACK_ECAPACITY, "imp_stride %lld < T_in %lld of unit %d", (long long)imp_stride, (long long)T, u);
    if (plan.n_units == kStaticUnitsMax)
      return fail(ctx, HACK_ECAPACITY, "hack_score_static scores at most %d units per call", kStaticUnitsMax);
    plan.in_off[plan.n_units] = in->off[u];
    plan.len_in[plan.n_units] = in->len[u];
    plan.unit[plan.n_units] = u;
    ++plan.n_units;
  }
  if (plan.n_units == 0) return HACK_OK;
  {   // the item size hack_score would take for these units: same grouping of the keys, same bits
    std::vector<int> t_in;
    for (int i = 0; i < plan.n_units; ++i) t_in.push_back(plan.len_in[i] + plan.n_new);
    plan.item_keys = choose_score_item_keys(ctx, std::move(t_in));
  }
  fill_q_rows(q_idx, n_obs, N_k, plan.q_rows);
  HIP_TRY(ctx, launch_score_static(static_cast<hipStream_t>(stream), ctx->cfg.device, ctx->cfg.head_dim, plan, q, n_obs, N_k, scale,
                                   in->k, k_new, importance, imp_stride, ctx->fault));
  return HACK_OK;
} HACK_NO_THROW(ctx)

// ---------------------------------------------------------------------------
// a2: select
// ---------------------------------------------------------------------------
extern "C" hack_status hack_select(hack_ctx* ctx, int32_t B, const float* importance, int64_t imp_stride,
                                   const int32_t* t_in, const uint8_t* head_type, const int32_t* budget,
                                   int32_t n_init, int32_t n_recent, int32_t* kept_idx, int64_t idx_stride,
                                   int32_t* len_out, hack_stream stream) try {
  hack_status st = check_common(ctx, B, 0, false);
  if (st != HACK_OK) return st;
  const int U = B * ctx->cfg.heads, H = ctx->cfg.heads;
  if (!importance || !t_in || !head_type || !budget || !kept_idx) return fail(ctx, HACK_EINVAL, "NULL argument");
  if (n_init < 0 || n_recent < 0) return fail(ctx, HACK_EINVAL, "n_init and n_recent must be >= 0");
  for (int h = 0; h < H; ++h)
    if (head_type[h] > 1) return fail(ctx, HACK_EINVAL, "head_type[%d] = %d is not a head class", h, head_type[h]);
  std::vector<UnitDesc> descs(U);
  int max_t = 0;
  for (int u = 0; u < U; ++u) {
    const int T = t_in[u];
    if (T < 1) return fail(ctx, HACK_EINVAL, "t_in[%d] = %d", u, T);
    if (T > ctx->cfg.max_cache_len) return fail(ctx, HACK_ECAPACITY, "t_in[%d] = %d exceeds max_cache_len %d", u, T, ctx->cfg.max_cache_len);
    if (budget[u] < 1) return fail(ctx, HACK_EINVAL, "budget[%d] = %d", u, budget[u]);
    if (head_type[u % H] == HACK_STRUCTURAL && n_recent > T) return fail(ctx, HACK_EINVAL, "n_recent %d > t_in[%d] = %d", n_recent, u, T);
    const int b = std::min(budget[u], T);
    if (T > imp_stride || b > idx_stride) return fail(ctx, HACK_ECAPACITY, "strides too small for unit %d", u);
    UnitDesc d{};
    d.len_in = T; d.n_new = 0; d.n_out = b; d.unit = u;
    plan_select(head_type[u % H], T, b, n_init, n_recent, &d);
    descs[u] = d;
    max_t = std::max(max_t, T);
    if (len_out) len_out[u] = b;
  }
  Table t;
  const size_t o_desc = t.add(descs.data(), descs.size());
  const uint8_t* dev;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if ((st = table_device(ctx, t, s, &dev)) != HACK_OK) return st;
  launch_select(s, (const UnitDesc*)(dev + o_desc), U, max_t, importance, imp_stride,
                kept_idx, idx_stride, nullptr);
  HIP_TRY(ctx, hipGetLastError());
  return HACK_OK;
} HACK_NO_THROW(ctx)

// ---------------------------------------------------------------------------
// a3: compact
// ---------------------------------------------------------------------------
extern "C" hack_status hack_compact(hack_ctx* ctx, int32_t B, int32_t N_k, const hack_cache* in, const void* k_new,
                                    const void* v_new, int32_t pos_new, const int32_t* kept_idx, int64_t idx_stride,
                                    const hack_cache* out, hack_stream stream) try {
  const bool has_new = (k_new != nullptr);
  hack_status st = check_common(ctx, B, N_k, has_new);
  if (st != HACK_OK) return st;
  const int U = B * ctx->cfg.heads;
  if (!kept_idx) return fail(ctx, HACK_EINVAL, "kept_idx is NULL");
  if (has_new != (v_new != nullptr)) return fail(ctx, HACK_EINVAL, "k_new and v_new must both be given or both be NULL");
  if (has_new && (!aligned16(k_new) || !aligned16(v_new))) return fail(ctx, HACK_EINVAL, "k_new/v_new must be 16-byte aligned");
  if ((st = check_cache(ctx, in, U, "in", true)) != HACK_OK) return st;
  if ((st = check_cache(ctx, out, U, "out", true)) != HACK_OK) return st;
  const int n_new = has_new ? N_k : 0;
  std::vector<UnitDesc> descs;
  int max_rows = 0;
  std::vector<std::pair<int64_t, int64_t>> in_iv;
  for (int u = 0; u < U; ++u) {
    const int n = out->len[u];
    if (n == 0) continue;
    if (n > idx_stride) return fail(ctx, HACK_ECAPACITY, "idx_stride %lld < out->len[%d] = %d", (long long)idx_stride, u, n);
    if ((int64_t)n > (int64_t)in->len[u] + n_new) return fail(ctx, HACK_EINVAL, "unit %d keeps %d rows of %lld", u, n, (long long)in->len[u] + n_new);
    UnitDesc d{};
    d.in_off = in->off[u]; d.out_off = out->off[u]; d.len_in = in->len[u]; d.n_new = n_new; d.n_out = n;
    d.mode = MOVE_GATHER; d.unit = u;
    descs.push_back(d);
    max_rows = std::max(max_rows, n);
    if (in->len[u] > 0) in_iv.emplace_back(in->off[u], in->off[u] + in->len[u]);
  }
  if (descs.empty()) return HACK_OK;
  if (out->k == in->k || out->v == in->v || out->k == in->v || out->v == in->k) {
    std::sort(in_iv.begin(), in_iv.end());
    for (const UnitDesc& d : descs) {
      const int64_t a = d.out_off, b = d.out_off + d.n_out;
      auto it = std::lower_bound(in_iv.begin(), in_iv.end(), std::make_pair(b, (int64_t)INT64_MIN));
      // intervals starting before b: the one with the largest end among them may overlap
      for (auto p = in_iv.begin(); p != it; ++p)
        if (p->second > a) return fail(ctx, HACK_EINVAL, "output rows of unit %d overlap input rows that are read", d.unit);
    }
  }
  Table t;
  const size_t o_desc = t.add(descs.data(), descs.size());
  const uint8_t* dev;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if ((st = table_device(ctx, t, s, &dev)) != HACK_OK) return st;
  CachePtrs pin{in->k, in->v, in->pos}, pout{out->k, out->v, out->pos};
  launch_move(s, ctx->elem_bytes, ctx->cfg.head_dim, (const UnitDesc*)(dev + o_desc), (int)descs.size(), max_rows, pin,
              pout, k_new, v_new, N_k, pos_new, kept_idx, idx_stride);
  HIP_TRY(ctx, hipGetLastError());
  return HACK_OK;
} HACK_NO_THROW(ctx)

// ---------------------------------------------------------------------------
// final-step merge of contextual heads
// ---------------------------------------------------------------------------
extern "C" hack_status hack_merge(hack_ctx* ctx, int32_t B, int32_t N_k, const hack_cache* in, const void* k_new,
                                  const void* v_new, const int32_t* kept_idx, int64_t idx_stride, const uint8_t* active,
                                  const hack_cache* out, hack_stream stream) try {
  const bool has_new = (k_new != nullptr);
  hack_status st = check_common(ctx, B, N_k, has_new);
  if (st != HACK_OK) return st;
  if (ctx->cfg.dtype != HACK_BF16) return fail(ctx, HACK_EUNSUPPORTED, "the final-step merge is implemented for bf16 contexts");
  const int U = B * ctx->cfg.heads;
  if (!kept_idx) return fail(ctx, HACK_EINVAL, "kept_idx is NULL");
  if (has_new != (v_new != nullptr)) return fail(ctx, HACK_EINVAL, "k_new and v_new must both be given or both be NULL");
  if (has_new && (!aligned16(k_new) || !aligned16(v_new))) return fail(ctx, HACK_EINVAL, "k_new/v_new must be 16-byte aligned");
  if ((st = check_cache(ctx, in, U, "in", true)) != HACK_OK) return st;
  if ((st = check_cache(ctx, out, U, "out", true)) != HACK_OK) return st;
  const int n_new = has_new ? N_k : 0;
  std::vector<UnitDesc> descs;
  std::vector<int32_t> list;
  int max_t = 0, max_out = 0;
  for (int u = 0; u < U; ++u) {
    if (active && !active[u]) continue;
    const int64_t T = (int64_t)in->len[u] + n_new;
    const int n = out->len[u];
    if (n < 1) return fail(ctx, HACK_EINVAL, "unit %d keeps no row", u);
    if (n > T) return fail(ctx, HACK_EINVAL, "unit %d keeps %d rows of %lld", u, n, (long long)T);
    if (T > ctx->cfg.max_cache_len) return fail(ctx, HACK_ECAPACITY, "unit %d: T_in = %lld exceeds max_cache_len %d", u, (long long)T, ctx->cfg.max_cache_len);
    if (n > idx_stride) return fail(ctx, HACK_ECAPACITY, "idx_stride %lld < out->len[%d] = %d", (long long)idx_stride, u, n);
    if (n == T) continue;   // nothing evicted
    // the kept rows are rewritten in place while the evicted ones are still read from `in`
    if ((out->k == in->k || out->v == in->v) && in->len[u] > 0 && out->off[u] < in->off[u] + in->len[u] &&
        in->off[u] < out->off[u] + n)
      return fail(ctx, HACK_EINVAL, "output rows of unit %d overlap its input rows", u);
    UnitDesc d{};
    d.in_off = in->off[u]; d.out_off = out->off[u]; d.len_in = in->len[u]; d.n_new = n_new; d.n_out = n; d.unit = u;
    list.push_back((int32_t)descs.size());
    descs.push_back(d);
    max_t = std::max(max_t, (int)T);
    max_out = std::max(max_out, n);
  }
  if (descs.empty()) return HACK_OK;
  Table t;
  const size_t o_desc = t.add(descs.data(), descs.size());
  const size_t o_list = t.add(list.data(), list.size());
  const uint8_t* dev;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if ((st = table_device(ctx, t, s, &dev)) != HACK_OK) return st;
  launch_merge(s, ctx->cfg.head_dim, (const UnitDesc*)(dev + o_desc), (const int32_t*)(dev + o_list), (int)list.size(), max_t,
               max_out, in->k, in->v, k_new, v_new, N_k, kept_idx, idx_stride, out->k, out->v, ctx->merge_nn, ctx->merge_w,
               ctx->merge_inv, ctx->ws_stride);
  HIP_TRY(ctx, hipGetLastError());
  return HACK_OK;
} HACK_NO_THROW(ctx)

// ---------------------------------------------------------------------------
// a4: attention
// ---------------------------------------------------------------------------
extern "C" hack_status hack_attn(hack_ctx* ctx, int32_t B, int32_t N_k, const void* q, const hack_cache* kv,
                                 float scale, void* out, hack_stream stream) try {
  hack_status st = check_common(ctx, B, N_k, true);
  if (st != HACK_OK) return st;
  const int U = B * ctx->cfg.heads;
  if (!q || !out) return fail(ctx, HACK_EINVAL, "q and out must not be NULL");
  if (!aligned16(q) || !aligned16(out)) return fail(ctx, HACK_EINVAL, "q/out must be 16-byte aligned");
  if (!scale_ok(scale)) return fail(ctx, HACK_EINVAL, "scale must be finite and > 0");
  if ((st = check_cache(ctx, kv, U, "kv", true)) != HACK_OK) return st;
  std::vector<UnitDesc> descs(U);
  int max_keys = 0;
  for (int u = 0; u < U; ++u) {
    if (kv->len[u] < 1) return fail(ctx, HACK_EINVAL, "unit %d has an empty cache", u);
    UnitDesc d{};
    d.in_off = kv->off[u]; d.out_off = kv->off[u]; d.len_in = kv->len[u]; d.n_out = kv->len[u]; d.unit = u;
    descs[u] = d;
    max_keys = std::max(max_keys, d.n_out);
  }
  const bool split = use_split_attention(ctx, U, N_k);
  const int tile = attn_tile_rows(ctx, U, N_k);
  std::vector<AttnItem> items;
  AttnStreamPlan plan;
  const bool halves = !split && use_key_halves(ctx, descs, N_k, &items);
  const bool streamed = !split && !halves && use_stream_attention(ctx, descs, N_k, false, &items, &plan);
  if (streamed) items.clear();
  else if (items.empty()) build_attn_items(descs, N_k, tile, &items);
  Table t;
  const size_t o_desc = t.add(descs.data(), descs.size());
  const size_t o_items = t.add(items.data(), items.size());
  const size_t o_segs = t.add(plan.segs.data(), plan.segs.size());
  const size_t o_segb = t.add(plan.seg_begin.data(), plan.seg_begin.size());
  const uint8_t* dev;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if ((st = table_device(ctx, t, s, &dev)) != HACK_OK) return st;
  if (streamed)
    launch_attn_stream(s, ctx->cfg.head_dim, (const UnitDesc*)(dev + o_desc), (const AttnSeg*)(dev + o_segs),
                       (const int32_t*)(dev + o_segb), plan.n_groups, q, kv->k, kv->v, N_k, scale, out, ctx->part_o,
                       ctx->part_ml, ctx->part_count);
  else if (split)
    launch_attn_split(s, ctx->cfg.head_dim, (const UnitDesc*)(dev + o_desc), (const AttnItem*)(dev + o_items),
                      (int)items.size(), q, kv->k, kv->v, nullptr, nullptr, nullptr, nullptr, nullptr, 0, false,
                      attn_split_in_eight(ctx->cfg.head_dim, (int)items.size(), U, max_keys), N_k, scale, out);
  else if (ctx->cfg.dtype == HACK_F32)
    launch_attn_f32(s, ctx->cfg.head_dim, (const AttnItem*)(dev + o_items), (int)items.size(), tile, q, kv->k, kv->v, nullptr,
                    nullptr, nullptr, nullptr, nullptr, 0, 0, N_k, scale, out);
  else
    launch_attn(s, ctx->cfg.head_dim, (const UnitDesc*)(dev + o_desc), (const AttnItem*)(dev + o_items), (int)items.size(), q,
                kv->k, kv->v, N_k, scale, out, halves ? kAttnHalves : ctx->attn_kernel == kAttnPlain ? kAttnPlain : kAttnPipe);
  HIP_TRY(ctx, hipGetLastError());
  return HACK_OK;
} HACK_NO_THROW(ctx)

extern "C" int32_t hack_attn_variant(const hack_ctx* ctx, int32_t B, int32_t N_k) {
  if (!ctx || B < 1 || N_k < 1) return (int32_t)HACK_EINVAL;
  return use_split_attention(ctx, B * ctx->cfg.heads, N_k) ? 1 : 0;
}

// ---------------------------------------------------------------------------
// offline head classification: attention variance
// ---------------------------------------------------------------------------
extern "C" hack_status hack_head_variance(hack_ctx* ctx, int32_t B, int32_t N_k, const void* q, const hack_cache* kv,
                                          float scale, double* sigma, hack_stream stream) try {
  hack_status st = check_common(ctx, B, N_k, true);
  if (st != HACK_OK) return st;
  if (ctx->cfg.dtype != HACK_BF16) return fail(ctx, HACK_EUNSUPPORTED, "head variance is implemented for bf16 contexts");
  const int U = B * ctx->cfg.heads;
  if (!q || !sigma) return fail(ctx, HACK_EINVAL, "q and sigma must not be NULL");
  if (!aligned16(q) || ((uintptr_t)sigma & 7)) return fail(ctx, HACK_EINVAL, "q must be 16-byte and sigma 8-byte aligned");
  if (!scale_ok(scale)) return fail(ctx, HACK_EINVAL, "scale must be finite and > 0");
  if ((st = check_cache(ctx, kv, U, "kv", false)) != HACK_OK) return st;
  std::vector<UnitDesc> descs(U);
  int max_len = 0;
  for (int u = 0; u < U; ++u) {
    if (kv->len[u] < 1) return fail(ctx, HACK_EINVAL, "unit %d has an empty cache", u);
    UnitDesc d{};
    d.in_off = kv->off[u]; d.out_off = kv->off[u]; d.len_in = kv->len[u]; d.n_out = kv->len[u]; d.unit = u;
    descs[u] = d;
    max_len = std::max(max_len, (int)kv->len[u]);
  }
  Table t;
  const size_t o_desc = t.add(descs.data(), descs.size());
  const uint8_t* dev;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if ((st = table_device(ctx, t, s, &dev)) != HACK_OK) return st;
  launch_head_variance(s, ctx->cfg.head_dim, (const UnitDesc*)(dev + o_desc), U, max_len, q, kv->k, N_k, scale,
                       ctx->hv_stats, sigma);
  HIP_TRY(ctx, hipGetLastError());
  return HACK_OK;
} HACK_NO_THROW(ctx)

// ---------------------------------------------------------------------------
// a5: managed cache + fused step
// ---------------------------------------------------------------------------
extern "C" hack_status hack_kvcache_rows_required(int32_t n_units, const int32_t* cap, int64_t* rows) {
  if (n_units < 1 || !cap || !rows) return HACK_EINVAL;
  int64_t r = 0;
  for (int u = 0; u < n_units; ++u) {
    if (cap[u] < 1) return HACK_EINVAL;
    r += 2 * round_up(cap[u], 8);
  }
  *rows = r;
  return HACK_OK;
}

extern "C" hack_status hack_kvcache_create(hack_ctx* ctx, int32_t n_units, const int32_t* cap, void* k_mem,
                                           void* v_mem, int32_t* pos_mem, int64_t mem_rows, hack_kvcache** out) try {
  if (!ctx) return HACK_EINVAL;
  if (!out || !cap || !k_mem || !v_mem) return fail(ctx, HACK_EINVAL, "NULL argument");
  *out = nullptr;
  if (n_units < 1 || n_units > ctx->cfg.max_units || n_units % ctx->cfg.heads)
    return fail(ctx, HACK_EINVAL, "n_units = %d must be a multiple of H within max_units", n_units);
  if (!aligned16(k_mem) || !aligned16(v_mem)) return fail(ctx, HACK_EINVAL, "k_mem/v_mem must be 16-byte aligned");
  int64_t need;
  if (hack_kvcache_rows_required(n_units, cap, &need) != HACK_OK) return fail(ctx, HACK_EINVAL, "cap entries must be >= 1");
  if (need > mem_rows) return fail(ctx, HACK_ECAPACITY, "cache needs %lld rows, %lld given", (long long)need, (long long)mem_rows);
  std::unique_ptr<hack_kvcache> c(new hack_kvcache());
  c->ctx = ctx; c->n_units = n_units; c->k = k_mem; c->v = v_mem; c->pos = pos_mem; c->rows = mem_rows; c->tokens_seen = 0;
  c->cap.assign(cap, cap + n_units);
  c->slab[0].resize(n_units); c->slab[1].resize(n_units);
  c->root.cur.assign(n_units, 0); c->root.len.assign(n_units, 0); c->root.off.resize(n_units);
  c->at = &c->root;
  int64_t r = 0;
  for (int u = 0; u < n_units; ++u) {
    c->slab[0][u] = r; r += round_up(cap[u], 8);
    c->slab[1][u] = r; r += round_up(cap[u], 8);
    c->root.off[u] = c->slab[0][u];
  }
  *out = c.release();
  return HACK_OK;
} HACK_NO_THROW(ctx)

extern "C" void hack_kvcache_destroy(hack_kvcache* c) { delete c; }

extern "C" hack_status hack_kvcache_reset(hack_kvcache* c) {
  if (!c) return HACK_EINVAL;
  c->at = &c->root;
  c->tokens_seen = 0;
  return HACK_OK;
}

extern "C" hack_status hack_kvcache_view(const hack_kvcache* c, hack_cache* view) {
  if (!c || !view) return HACK_EINVAL;
  view->k = c->k; view->v = c->v; view->pos = c->pos; view->rows = c->rows;
  view->off = c->at->off.data(); view->len = c->at->len.data();
  return HACK_OK;
}

extern "C" int32_t hack_kvcache_step_form(const hack_kvcache* c) { return c ? c->at->g[0].whole : 0; }

namespace {

// The units of a step that are launched together on one stream, before their tables are uploaded.
struct GroupUnits {
  std::vector<UnitDesc> descs;            // copies of the group's unit descriptors: the compressing units' stand in front, so that
                                          // launches over either kind find theirs together (through an index list, one more memory round trip
                                          // each, a 256^2 schedule took 117.3 us instead of 116.7 in float32, 93.3 instead of 92.8 in bf16)
  int n_comp = 0;                         // units that compress
  std::vector<int32_t> merging;           // indices into descs: units that also merge
};

struct StepArgs {
  const void *q, *k_new, *v_new;
  void* out;
  float scale;
  int32_t* kept;
  int64_t kstride;
  CachePtrs cp;
  int32_t pos_new;
  // Attention may read k_new / v_new in place and update the cache while other work-groups of the launch already store
  // their outputs: not where `out` shares memory with them.  The rows are then moved by a launch in front of it.
  bool in_place;
  bool apart;      // ... nor with q: a launch that scores, too, reads rows of q that other work-groups of it attend for
};

bool overlap(const void* a, const void* b, size_t bytes) {
  const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
  return x < y + bytes && y < x + bytes;
}

void add_unit(GroupUnits* u, StepGroup* g, const UnitDesc& d, bool merges, int N_k) {
  const int idx = (int)u->descs.size();
  u->descs.push_back(d);
  g->max_keys = std::max(g->max_keys, d.n_out);
  if (d.mode == MOVE_GATHER) {
    ++u->n_comp;
    g->max_t = std::max(g->max_t, d.len_in + d.n_new);
    g->max_rows = std::max(g->max_rows, d.n_out);
    if (merges) {
      u->merging.push_back(idx);
      g->merge_t = std::max(g->merge_t, d.len_in + d.n_new);
      g->merge_out = std::max(g->merge_out, d.n_out);
    }
  } else {
    g->max_rows = std::max(g->max_rows, N_k);
  }
}

// Queries per work-group of a launch that does the whole step, 0 where the step takes launches of its own.
int use_whole_step(const hack_ctx* ctx, const GroupUnits& u, const StepNode& n, const StepGroup& g) {
  // (a kernel that the environment asks for serves every step)
  if (ctx->cfg.dtype != HACK_BF16 || ctx->split_max_items >= 0 || ctx->attn_kernel != -1 || ctx->attn_stream != -1) return 0;
  if (u.n_comp == 0 || !u.merging.empty()) return 0;
  return whole_step_queries(ctx->cfg.head_dim, (int)u.descs.size(), u.n_comp, n.N_k, g.max_t, g.max_keys, ctx->lds_bytes);
}

bool score_select_short(const UnitDesc& d) { return d.len_in + d.n_new <= kScoreSelectHalf; }

// shared: another group of the step may attend at the same time
hack_status upload_group(hack_ctx* ctx, const GroupUnits& u, const StepNode& n, bool shared, const int32_t* rows, hipStream_t s,
                         StepGroup* g) {
  AttnStreamPlan plan;
  std::vector<AttnItem> items;
  std::vector<ScoreItem> sitems;
  // (a launch that does the whole step needs no work items, and no moves: outputs over its inputs have the rows moved by the launch that scores)
  g->whole = shared ? 0 : use_whole_step(ctx, u, n, *g);
  if (!g->whole) {
    g->attn_kernel = ctx->attn_kernel == kAttnPlain ? kAttnPlain : kAttnPipe;
    if (!n.split && !shared && use_key_halves(ctx, u.descs, n.N_k, &items)) g->attn_kernel = kAttnHalves;
    g->streamed = !n.split && g->attn_kernel != kAttnHalves && use_stream_attention(ctx, u.descs, n.N_k, shared, &items, &plan);
    if (g->streamed) items.clear();
    else if (items.empty()) build_attn_items(u.descs, n.N_k, n.tile, &items);
  }
  g->small = ctx->cfg.dtype == HACK_BF16 ? use_score_select(ctx->cfg.head_dim, u.n_comp, g->max_t)
                                         : use_score_select_f32(ctx->cfg.head_dim, u.n_comp, g->max_t);
  if (ctx->cfg.dtype == HACK_BF16 && u.n_comp > 0 && !g->small)
    g->item_keys = plan_score_items(ctx, u.descs, u.n_comp, g->two_pass, &sitems, &g->launches);
  // The key-split and the float32 kernel read the rows in place unless they change on the way (merge) or a unit's cache is longer than
  // the list of a unit that keeps everything.
  std::vector<MoveItem> moves;
  g->gathered = !g->whole && (n.split || ctx->cfg.dtype == HACK_F32) && !n.fuse_append && u.merging.empty();
  for (const UnitDesc& d : u.descs) g->gathered = g->gathered && (d.mode == MOVE_GATHER || d.n_out <= kIotaRows);
  if (g->gathered)
    for (size_t i = 0; i < u.descs.size(); ++i)
      for (int r = 0; r < (u.descs[i].mode == MOVE_GATHER ? u.descs[i].n_out : u.descs[i].n_new); r += kMoveItemRows)
        moves.push_back(MoveItem{(int32_t)i, r});
  if (ctx->cfg.dtype == HACK_BF16 && g->small && g->max_t > kScoreSelectHalf) {
    while (g->n_short < u.n_comp && score_select_short(u.descs[g->n_short])) ++g->n_short;
    if (!split_score_select(u.n_comp, g->n_short, g->gathered ? 0 : (int)u.descs.size() - u.n_comp)) g->n_short = 0;
  }
  g->n_moves = (int)moves.size();
  g->n_desc = (int)u.descs.size();
  g->n_comp = u.n_comp;
  g->n_merge = (int)u.merging.size();
  g->n_items = (int)items.size();
  g->n_stream = plan.n_groups;
  Table t;
  g->o_desc = t.add(u.descs.data(), u.descs.size());
  g->o_merge = t.add(u.merging.data(), u.merging.size());
  g->o_rows = t.add(rows, kMaxObs);
  g->o_items = t.add(items.data(), items.size());
  g->o_sit = t.add(sitems.data(), sitems.size());
  g->o_segs = t.add(plan.segs.data(), plan.segs.size());
  g->o_segb = t.add(plan.seg_begin.data(), plan.seg_begin.size());
  g->o_moves = t.add(moves.data(), moves.size());
  return table_device(ctx, t, s, &g->dev, &g->table);
}

// score -> select -> append / gather (-> merge) of a group's units
void launch_chain(hack_ctx* ctx, const StepNode& n, const StepGroup& g, const StepArgs& a, hipStream_t s) {
  if (g.whole && a.apart) return;
  bool moves = g.whole || !a.in_place || (!n.fuse_append && !g.gathered);   // rows move in front of the attention launch
  if (g.n_comp > 0 && g.small && ctx->cfg.dtype == HACK_F32) {
    launch_score_select_f32(s, ctx->cfg.head_dim, g.ddev(), g.n_comp, g.max_t, a.q, reinterpret_cast<const int32_t*>(g.dev + g.o_rows),
                            n.n_obs, n.N_k, a.scale, a.cp.k, a.k_new, ctx->f32_logits, ctx->stats, ctx->counters, a.kept, a.kstride, ctx->seam);
  } else if (g.n_comp > 0 && g.small && moves) {
    auto go = [&](int first, int n_units, int n_append, int max_t) {
      launch_score_select_move(s, ctx->cfg.head_dim, g.ddev() + first, n_units, g.ddev() + g.n_comp, n_append, max_t, a.q,
                               reinterpret_cast<const int32_t*>(g.dev + g.o_rows), n.n_obs, n.N_k, a.scale, a.cp, a.k_new, a.v_new, a.pos_new,
                               a.kept, a.kstride, ctx->fault);
    };
    if (g.n_short > 0) go(0, g.n_short, 0, kScoreSelectHalf);
    go(g.n_short, g.n_comp - g.n_short, g.n_desc - g.n_comp, g.max_t);
    moves = false;
  } else if (g.n_comp > 0 && g.small) {
    auto go = [&](int first, int n_units, int max_t) {
      launch_score_select(s, ctx->cfg.head_dim, g.ddev() + first, n_units, max_t, a.q,
                          reinterpret_cast<const int32_t*>(g.dev + g.o_rows), n.n_obs, n.N_k, a.scale, a.cp.k, a.k_new, a.kept, a.kstride,
                          ctx->seam, ctx->fault);
    };
    if (g.n_short > 0) go(0, g.n_short, kScoreSelectHalf);
    go(g.n_short, g.n_comp - g.n_short, g.max_t);
  } else if (g.n_comp > 0) {
    run_score(ctx, s, g.two_pass, g.slots, g.ddev(), g.n_comp, g.max_t,
              reinterpret_cast<const ScoreItem*>(g.dev + g.o_sit), g.item_keys, g.launches, a.q,
              reinterpret_cast<const int32_t*>(g.dev + g.o_rows), n.n_obs, n.N_k, a.scale, a.cp.k, a.k_new, ctx->importance,
              ctx->ws_stride);
    launch_select(s, g.ddev(), g.n_comp, g.max_t, ctx->importance, ctx->ws_stride, a.kept, a.kstride, ctx->seam);
  }
  if (moves)
    launch_move(s, ctx->elem_bytes, ctx->cfg.head_dim, g.ddev(), g.n_desc, g.max_rows, a.cp, a.cp, a.k_new, a.v_new, n.N_k,
                a.pos_new, a.kept, a.kstride);
  if (g.n_merge > 0)   // compression, the merge included, precedes the attention of the step
    launch_merge(s, ctx->cfg.head_dim, g.ddev(), reinterpret_cast<const int32_t*>(g.dev + g.o_merge), g.n_merge, g.merge_t,
                 g.merge_out, a.cp.k, a.cp.v, a.k_new, a.v_new, n.N_k, a.kept, a.kstride, a.cp.k, a.cp.v, ctx->merge_nn,
                 ctx->merge_w, ctx->merge_inv, ctx->ws_stride);
}

void launch_group_attention(hack_ctx* ctx, const StepNode& n, const StepGroup& g, const StepArgs& a, hipStream_t s) {
  const AttnItem* items = reinterpret_cast<const AttnItem*>(g.dev + g.o_items);
  const bool append = n.fuse_append && a.in_place;
  const bool eight = n.split && attn_split_in_eight(ctx->cfg.head_dim, g.n_items, g.n_desc, g.max_keys);
  if (g.whole) {
    const WholeStep st{g.n_desc, g.max_t, g.max_keys, g.whole, n.n_obs, reinterpret_cast<const int32_t*>(g.dev + g.o_rows), ctx->fault, !a.apart, 0};
    launch_step_units(s, ctx->cfg.head_dim, g.ddev(), st, a.q, a.cp, a.k_new, a.v_new, a.pos_new, n.N_k, a.scale, a.out, a.kept, a.kstride);
    return;
  }
  if (g.gathered && a.in_place) {
    const GatherArgs ga{a.kept, a.kstride, ctx->seam, ctx->iota, reinterpret_cast<const MoveItem*>(g.dev + g.o_moves), g.n_moves,
                        a.pos_new, a.k_new, a.v_new, a.cp, eight};
    if (ctx->cfg.dtype == HACK_F32)
      launch_attn_f32_gather(s, ctx->cfg.head_dim, g.ddev(), items, g.n_items, n.tile, ga, a.q, a.cp.k, a.cp.v, n.N_k, a.scale, a.out);
    else
      launch_attn_split_gather(s, ctx->cfg.head_dim, g.ddev(), items, g.n_items, ga, a.q, a.cp.k, a.cp.v, n.N_k, a.scale, a.out);
    return;
  }
  if (g.streamed)
    launch_attn_stream(s, ctx->cfg.head_dim, g.ddev(), reinterpret_cast<const AttnSeg*>(g.dev + g.o_segs),
                       reinterpret_cast<const int32_t*>(g.dev + g.o_segb), g.n_stream, a.q, a.cp.k, a.cp.v, n.N_k, a.scale, a.out,
                       ctx->part_o, ctx->part_ml, ctx->part_count);
  else if (n.split)
    launch_attn_split(s, ctx->cfg.head_dim, g.ddev(), items, g.n_items, a.q, a.cp.k, a.cp.v, a.k_new, a.v_new, a.cp.k, a.cp.v,
                      a.cp.pos, a.pos_new, append, eight, n.N_k, a.scale, a.out);
  else if (ctx->cfg.dtype == HACK_F32)
    launch_attn_f32(s, ctx->cfg.head_dim, items, g.n_items, n.tile, a.q, a.cp.k, a.cp.v, a.k_new, a.v_new, a.cp.k, a.cp.v, a.cp.pos,
                    a.pos_new, append ? 1 : 0, n.N_k, a.scale, a.out);
  else
    launch_attn(s, ctx->cfg.head_dim, g.ddev(), items, g.n_items, a.q, a.cp.k, a.cp.v, n.N_k, a.scale, a.out, g.attn_kernel);
}

// Sees to it that a known step's tables are on the device for the work that is issued on `s` next: a step that was
// planned while its stream was being captured has them only where that graph is replayed.
hack_status upload_step(hack_ctx* ctx, StepNode* n, hipStream_t s) {
  n->uploaded = true;
  for (int i = 0; i < (n->two_groups ? 2 : 1); ++i) {
    if (ctx->tables->upload(n->g[i].table, s) != TableStatus::kOk) {
      n->uploaded = false;
      return fail(ctx, HACK_EHIP, "uploading a launch table failed");
    }
    n->uploaded = n->uploaded && ctx->tables->uploaded(n->g[i].table);
  }
  return HACK_OK;
}

// The child of the cache's current state that these arguments lead to, if it is known.
StepNode* find_step(const hack_kvcache* c, int32_t N_k, const uint8_t* head_type, int H, const int32_t* budget, int U,
                          int32_t n_init, bool final_merge, bool two_pass) {
  for (const auto& p : c->at->next)
    if (p->N_k == N_k && p->n_init == n_init && p->final_merge == final_merge && p->two_pass == two_pass &&
        memcmp(p->head_type.data(), head_type, H) == 0 && memcmp(p->budget.data(), budget, (size_t)U * sizeof(int32_t)) == 0)
      return p.get();
  return nullptr;
}

// Validates and plans a step from the cache's current state, uploads its tables and adds it to the tree.
hack_status plan_step(hack_ctx* ctx, hack_kvcache* cache, int32_t B, int32_t N_k, const uint8_t* head_type, const int32_t* budget,
                      int32_t n_init, bool final_merge, hipStream_t s, StepNode** out) {
  const int U = B * ctx->cfg.heads, H = ctx->cfg.heads;
  for (int h = 0; h < H; ++h)
    if (head_type[h] > 1) return fail(ctx, HACK_EINVAL, "head_type[%d] = %d is not a head class", h, head_type[h]);
  std::unique_ptr<StepNode> n(new StepNode());
  const StepNode& from = *cache->at;
  std::vector<UnitDesc> descs[2];   // compressing units, the others
  for (auto& v : descs) v.reserve(U);
  int n_side = 0;
  n->cur = from.cur;
  n->off = from.off;
  n->len.resize(U);
  for (int u = 0; u < U; ++u) {
    const int L = from.len[u];
    const int64_t T = (int64_t)L + N_k;
    if (budget[u] < 1) return fail(ctx, HACK_EINVAL, "budget[%d] = %d", u, budget[u]);
    UnitDesc d{};
    d.unit = u; d.in_off = from.off[u]; d.len_in = L; d.n_new = N_k;
    if (budget[u] < T) {
      if (T > ctx->cfg.max_cache_len) return fail(ctx, HACK_ECAPACITY, "unit %d: T_in = %lld exceeds max_cache_len %d", u, (long long)T, ctx->cfg.max_cache_len);
      if (budget[u] > cache->cap[u]) return fail(ctx, HACK_ECAPACITY, "unit %d: budget %d exceeds its slab of %d rows", u, budget[u], cache->cap[u]);
      n->cur[u] ^= 1;
      n->off[u] = cache->slab[n->cur[u]][u];
      n->max_budget = std::max(n->max_budget, budget[u]);
      d.mode = MOVE_GATHER; d.n_out = budget[u];
      plan_select(head_type[u % H], (int)T, budget[u], n_init, N_k, &d);
      if (head_type[u % H] == HACK_CONTEXTUAL) ++n_side;
    } else {
      if (T > cache->cap[u]) return fail(ctx, HACK_ECAPACITY, "unit %d: %lld rows do not fit its slab of %d", u, (long long)T, cache->cap[u]);
      d.mode = MOVE_APPEND; d.n_out = (int)T;
    }
    d.out_off = n->off[u];
    n->len[u] = d.n_out;
    descs[d.mode == MOVE_GATHER ? 0 : 1].push_back(d);
  }
  n->N_k = N_k;
  n->n_init = n_init;
  n->final_merge = final_merge;
  n->two_pass = ctx->score_mode == HACK_SCORE_TWO_PASS;
  n->head_type.assign(head_type, head_type + H);
  n->budget.assign(budget, budget + U);
  n->n_obs = std::min(ctx->cfg.n_obs, N_k);
  n->split = use_split_attention(ctx, U, N_k);
  // no unit compresses: the key-split bf16 kernel and the float32 kernel append as well
  n->fuse_append = (n->split || ctx->cfg.dtype == HACK_F32) && descs[0].empty();
  n->tile = attn_tile_rows(ctx, U, N_k);
  int32_t rows[kMaxObs];
  fill_q_rows(nullptr, n->n_obs, N_k, rows);

  // group 0: the caller's stream; group 1 (optional): the compressing contextual units, beside group 0's attention
  n->two_groups = ctx->step_overlap && ctx->cfg.dtype == HACK_BF16 && n_side > 0 && n_side < U;
  GroupUnits units[2];
  n->g[0].two_pass = n->two_pass;
  n->g[0].slots = ctx->rowstat;
  n->g[1].two_pass = true;          // leaves its sums in the slots, hence an exchange area of its own
  n->g[1].slots = ctx->rowstat_side;
  for (GroupUnits& g : units) g.descs.reserve(U);
  if (ctx->cfg.dtype == HACK_BF16 && descs[0].size() > 512)   // where a launch may be over the short ones alone it finds them together
    std::stable_partition(descs[0].begin(), descs[0].end(), score_select_short);
  for (const UnitDesc& d : descs[0]) {
    const bool ctxl = head_type[d.unit % H] == HACK_CONTEXTUAL;
    const int i = n->two_groups && ctxl ? 1 : 0;
    add_unit(&units[i], &n->g[i], d, final_merge && ctxl, N_k);
  }
  for (const UnitDesc& d : descs[1]) add_unit(&units[0], &n->g[0], d, false, N_k);
  for (int i = 0; i < (n->two_groups ? 2 : 1); ++i) {
    const hack_status st = upload_group(ctx, units[i], *n, n->two_groups, rows, s, &n->g[i]);
    if (st != HACK_OK) return st;
  }
  n->uploaded = ctx->tables->uploaded(n->g[0].table) && (!n->two_groups || ctx->tables->uploaded(n->g[1].table));
  if (cache->n_nodes >= kMaxStepNodes) {
    // the tree is full (arguments that keep changing): keep the current state alone and start over
    std::unique_ptr<StepNode> base(new StepNode());
    base->cur = from.cur; base->off = from.off; base->len = from.len;
    const bool at_root = cache->at == &cache->root;
    cache->root.next.clear();
    cache->base = std::move(base);   // drops the earlier one and what grew below it
    cache->at = at_root ? &cache->root : cache->base.get();
    cache->n_nodes = 0;
  }
  *out = n.get();
  const_cast<StepNode*>(cache->at)->next.push_back(std::move(n));
  ++cache->n_nodes;
  return HACK_OK;
}

}  // namespace

// One scale step.  Units are independent, so a step may be issued as two groups: the compression chain
// (score -> select -> gather) is a sequence of short, latency-bound launches that leaves most of the device
// idle, while attention fills it.  With the overlap switched on (HACK_STEP_OVERLAP=1 when the context is
// created), when contextual units compress at this step and other units exist, the others go first on the
// caller's stream (their chain, then their attention, which is the longer one: structural budgets are the
// larger), and the contextual units' chain and attention run beside that attention on a stream of the context,
// forked and joined with events (capturable: a HIP graph gets two parallel branches).  The side chain scores
// in the two-pass form, whose work-groups never wait for each other and can therefore share the device with
// the attention launch.  What is computed per unit is the same; only the grouping of a unit's keys into work
// items (chosen per launch) may differ from a single-group step.
// The overlap is OFF by default: on MI355X it measured slower (1024^2 benchmark workload: 1005 against 841 us
// per layer).  The attention launch of the first group holds every wave slot of the device, so the side chain
// only advances as attention work-groups retire and ends with them; the second group's attention then runs
// on its own, and a lone attention launch takes one work item's full latency (60 to 120 key blocks at half a
// microsecond each) however few items it has.  Splitting a step therefore lengthens its critical path.
static hack_status step_impl(hack_ctx* ctx, hack_kvcache* cache, int32_t B, int32_t N_k, const void* q,
                             const void* k_new, const void* v_new, const uint8_t* head_type,
                             const int32_t* budget, int32_t n_init, float scale, void* out,
                             int32_t* kept_idx_opt, int64_t idx_stride, hack_stream stream, bool final_merge) try {
  hack_status st = check_common(ctx, B, N_k, true);
  if (st != HACK_OK) return st;
  if (final_merge && ctx->cfg.dtype != HACK_BF16)
    return fail(ctx, HACK_EUNSUPPORTED, "the final-step merge is implemented for bf16 contexts");
  const int U = B * ctx->cfg.heads, H = ctx->cfg.heads;
  if (!cache || cache->ctx != ctx || cache->n_units != U) return fail(ctx, HACK_EINVAL, "cache does not belong to this context / batch");
  if (!q || !k_new || !v_new || !head_type || !budget || !out) return fail(ctx, HACK_EINVAL, "NULL argument");
  if (!aligned16(q) || !aligned16(k_new) || !aligned16(v_new) || !aligned16(out)) return fail(ctx, HACK_EINVAL, "q/k_new/v_new/out must be 16-byte aligned");
  if (!scale_ok(scale)) return fail(ctx, HACK_EINVAL, "scale must be finite and > 0");
  if (n_init < 0) return fail(ctx, HACK_EINVAL, "n_init must be >= 0");
  if (cache->tokens_seen + N_k > INT32_MAX) return fail(ctx, HACK_ECAPACITY, "token ids overflow int32");

  StepArgs a{};
  a.kept = kept_idx_opt ? kept_idx_opt : ctx->kept;
  a.kstride = kept_idx_opt ? idx_stride : ctx->ws_stride;
  a.q = q; a.k_new = k_new; a.v_new = v_new; a.out = out; a.scale = scale;
  a.cp = CachePtrs{cache->k, cache->v, cache->pos};
  a.pos_new = (int32_t)cache->tokens_seen;
  const size_t new_bytes = (size_t)U * N_k * ctx->cfg.head_dim * ctx->elem_bytes;
  a.in_place = !overlap(out, k_new, new_bytes) && !overlap(out, v_new, new_bytes);
  a.apart = a.in_place && !overlap(out, q, new_bytes);

  hipStream_t s = static_cast<hipStream_t>(stream);
  StepNode* n = find_step(cache, N_k, head_type, H, budget, U, n_init, final_merge, ctx->score_mode == HACK_SCORE_TWO_PASS);
  if (n) {
    if (!n->uploaded && (st = upload_step(ctx, n, s)) != HACK_OK) return st;
  } else if ((st = plan_step(ctx, cache, B, N_k, head_type, budget, n_init, final_merge, s, &n)) != HACK_OK) {
    return st;
  }
  if (n->max_budget > a.kstride)
    return fail(ctx, HACK_ECAPACITY, "idx_stride %lld < largest budget %d of a compressing unit", (long long)a.kstride, n->max_budget);

  launch_chain(ctx, *n, n->g[0], a, s);
  if (n->two_groups) {
    HIP_TRY(ctx, hipEventRecord(ctx->ev_fork, s));
    HIP_TRY(ctx, hipStreamWaitEvent(ctx->aux_stream, ctx->ev_fork, 0));
  }
  launch_group_attention(ctx, *n, n->g[0], a, s);
  if (n->two_groups) {
    launch_chain(ctx, *n, n->g[1], a, ctx->aux_stream);
    launch_group_attention(ctx, *n, n->g[1], a, ctx->aux_stream);
    HIP_TRY(ctx, hipEventRecord(ctx->ev_join, ctx->aux_stream));
    HIP_TRY(ctx, hipStreamWaitEvent(s, ctx->ev_join, 0));
  }
  HIP_TRY(ctx, hipGetLastError());
  cache->at = n;
  cache->tokens_seen += N_k;
  return HACK_OK;
} HACK_NO_THROW(ctx)

extern "C" hack_status hack_step(hack_ctx* ctx, hack_kvcache* cache, int32_t B, int32_t N_k, const void* q,
                                 const void* k_new, const void* v_new, const uint8_t* head_type,
                                 const int32_t* budget, int32_t n_init, float scale, void* out,
                                 int32_t* kept_idx_opt, int64_t idx_stride, hack_stream stream) {
  return step_impl(ctx, cache, B, N_k, q, k_new, v_new, head_type, budget, n_init, scale, out, kept_idx_opt, idx_stride,
                   stream, false);
}

extern "C" hack_status hack_step_final(hack_ctx* ctx, hack_kvcache* cache, int32_t B, int32_t N_k, const void* q,
                                       const void* k_new, const void* v_new, const uint8_t* head_type,
                                       const int32_t* budget, int32_t n_init, float scale, void* out,
                                       int32_t* kept_idx_opt, int64_t idx_stride, hack_stream stream) {
  return step_impl(ctx, cache, B, N_k, q, k_new, v_new, head_type, budget, n_init, scale, out, kept_idx_opt, idx_stride,
                   stream, true);
}
