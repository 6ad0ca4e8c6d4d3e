// Host-side checks of csrc/hack_api.cpp over a stand-in for the HIP runtime (hip_host_stub.h); argv[1] names the check.
#include "hip_host_stub.h"

#include "../../paper_2504_09261_amd/csrc/hack_api.cpp"

#define CHECK(c)                                    \
  do {                                              \
    if (!(c)) {                                     \
      printf("FAILED line %d: %s\n", __LINE__, #c); \
      return 1;                                     \
    }                                               \
  } while (0)

namespace {

constexpr int kH = 4, kD = 64;
void* const kStream = reinterpret_cast<void*>(0x10);

struct Setup {
  hack_ctx* ctx = nullptr;
  hack_kvcache* cache = nullptr;
  std::vector<uint8_t> mem, k_mem, v_mem;
  void *q, *k, *v, *out;
  Setup(int dtype, int cap, int max_len, int max_queries) {
    hack_config cfg{0, kH, kD, dtype, kH, max_len, max_queries, 32};
    if (hack_create(&ctx, &cfg) != HACK_OK) abort();
    const size_t row = kD * 4, n = (size_t)kH * max_queries * row;
    mem.resize(4 * n + 64);
    uint8_t* p = reinterpret_cast<uint8_t*>((reinterpret_cast<uintptr_t>(mem.data()) + 63) / 64 * 64);
    q = p; k = p + n; v = p + 2 * n; out = p + 3 * n;
    std::vector<int32_t> caps(kH, cap);
    int64_t rows;
    hack_kvcache_rows_required(kH, caps.data(), &rows);
    k_mem.resize(rows * row + 64);
    v_mem.resize(rows * row + 64);
    auto up = [](std::vector<uint8_t>& m) { return reinterpret_cast<void*>((reinterpret_cast<uintptr_t>(m.data()) + 63) / 64 * 64); };
    if (hack_kvcache_create(ctx, kH, caps.data(), up(k_mem), up(v_mem), nullptr, rows, &cache) != HACK_OK) abort();
  }
  ~Setup() {
    hack_kvcache_destroy(cache);
    hack_destroy(ctx);
  }
  hack_status step(int n, int budget, bool final_merge = false, int n_init = 5, void* to = nullptr) {
    const int32_t b[kH] = {budget, budget, budget, budget};
    return step_each(n, b, final_merge, n_init, to);
  }
  hack_status step_each(int n, const int32_t (&budget)[kH], bool final_merge = false, int n_init = 5, void* to = nullptr) {
    const uint8_t types[kH] = {0, 1, 0, 1};
    auto fn = final_merge ? hack_step_final : hack_step;
    return fn(ctx, cache, 1, n, q, k, v, types, budget, n_init, 0.125f, to ? to : out, nullptr, 0, kStream);
  }
  // three steps, the last one compresses
  bool schedule() {
    hack_kvcache_reset(cache);
    return step(8, 1 << 30) == HACK_OK && step(40, 1 << 30) == HACK_OK && step(30, 50) == HACK_OK;
  }
};

// A table first seen while the stream is being captured is copied when the graph is replayed and not before: calls
// outside that graph must not rely on it.
int capture() {
  for (int dtype : {HACK_BF16, HACK_F32}) {
    {   // the graph is thrown away; the schedule then runs eagerly
      Setup s(dtype, 64, 128, 64);
      stub::Graph g;
      stub::begin_capture(&g, kStream);
      CHECK(s.schedule());
      stub::end_capture();
      CHECK(g.copies > 0 && stub::launches.empty());
      CHECK(s.schedule());
      CHECK(stub::bad_launches == 0 && !stub::launches.empty());
      // ... after which a capture needs no copies and repeated steps issue none
      const int before = stub::copies;
      CHECK(s.schedule() && stub::copies == before);
      stub::Graph g2;
      stub::begin_capture(&g2, kStream);
      CHECK(s.schedule());
      stub::end_capture();
      CHECK(g2.copies == 0);
      stub::replay(g2);
      CHECK(stub::bad_launches == 0);
    }
    {   // two graphs are captured one after the other; only the second one is replayed
      Setup s(dtype, 64, 128, 64);
      stub::Graph g1, g2;
      for (stub::Graph* g : {&g1, &g2}) {
        stub::begin_capture(g, kStream);
        CHECK(s.schedule());
        stub::end_capture();
      }
      stub::replay(g2);
      CHECK(stub::bad_launches == 0);
      stub::replay(g2);
      stub::replay(g1);
      CHECK(stub::bad_launches == 0);
    }
    {   // eager steps up to a state, a captured step from it, the same step eagerly before any replay
      Setup s(dtype, 64, 128, 64);
      CHECK(s.step(8, 1 << 30) == HACK_OK && s.step(40, 1 << 30) == HACK_OK);
      stub::Graph g;
      stub::begin_capture(&g, kStream);
      CHECK(s.step(30, 50) == HACK_OK);
      stub::end_capture();
      hack_kvcache_reset(s.cache);
      CHECK(s.step(8, 1 << 30) == HACK_OK && s.step(40, 1 << 30) == HACK_OK && s.step(30, 50) == HACK_OK);
      CHECK(stub::bad_launches == 0);
      stub::replay(g);
      CHECK(stub::bad_launches == 0);
    }
    {   // the single entry points share the store
      Setup s(dtype, 64, 128, 64);
      const int64_t off[kH] = {0, 128, 256, 384};
      const int32_t len[kH] = {60, 50, 40, 30};
      std::vector<uint8_t> rows(512 * kD * 4 + 64);
      void* p = reinterpret_cast<void*>((reinterpret_cast<uintptr_t>(rows.data()) + 63) / 64 * 64);
      const hack_cache kv{p, p, nullptr, 512, off, len};
      stub::Graph g;
      stub::begin_capture(&g, kStream);
      CHECK(hack_attn(s.ctx, 1, 20, s.q, &kv, 0.125f, s.out, kStream) == HACK_OK);
      stub::end_capture();
      CHECK(hack_attn(s.ctx, 1, 20, s.q, &kv, 0.125f, s.out, kStream) == HACK_OK);
      CHECK(stub::bad_launches == 0);
    }
    stub::launches.clear();
  }
  return 0;
}

// Outputs stored over the new keys or values: no launch may read those in place beside work-groups that store outputs.
int out_over_new_rows() {
  for (int dtype : {HACK_BF16, HACK_F32}) {
    Setup s(dtype, 64, 128, 64);
    for (int pass = 0; pass < 3; ++pass) {
      void* to = pass == 0 ? s.k : pass == 1 ? s.v : static_cast<void*>(static_cast<uint8_t*>(s.k) + 1024);
      hack_kvcache_reset(s.cache);
      for (int step = 0; step < 3; ++step) {
        const int n = step == 0 ? 8 : step == 1 ? 40 : 30;
        stub::launches.clear();
        CHECK(s.step(n, step == 2 ? 50 : 1 << 30, false, 5, to) == HACK_OK);
        const auto& l = stub::launches;
        CHECK(l.size() >= 2 && l[l.size() - 2] == "move" && l.back() == (dtype == HACK_F32 ? "attn_f32" : "attn_split"));
      }
    }
    // outputs of their own: the remembered steps keep their shorter form
    CHECK(s.schedule());
    CHECK(stub::launches.back() == (dtype == HACK_F32 ? "attn_f32_gather" : "attn_split_gather"));
    CHECK(stub::bad_launches == 0);
    stub::launches.clear();
  }
  return 0;
}

// Short units: which launches serve a step that compresses all, some or one of its units, with outputs of their own and over the new
// rows, eagerly and from a graph; the launch that moves rows gets every unit once, on the side that it belongs to.
int short_units() {
  typedef std::vector<std::string> Names;
  const int32_t all[kH] = {50, 50, 50, 50}, some[kH] = {50, 1 << 30, 1 << 30, 40}, one[kH] = {1 << 30, 1 << 30, 30, 1 << 30};
  for (int dtype : {HACK_BF16, HACK_F32})
    for (int over = 0; over < 2; ++over)
      for (int last = 0; last < (dtype == HACK_BF16 ? 2 : 1); ++last)
        for (const auto* budget : {&all, &some, &one}) {
          Setup s(dtype, 96, 128, 64);
          void* to = over ? s.v : s.out;
          auto run = [&] {
            hack_kvcache_reset(s.cache);
            if (s.step(8, 1 << 30) != HACK_OK || s.step(40, 1 << 30) != HACK_OK) return false;
            stub::launches.clear();
            stub::moving_launches.clear();
            return s.step_each(30, *budget, last == 1, 5, to) == HACK_OK;
          };
          const int n_comp = budget == &all ? 4 : budget == &some ? 2 : 1;
          const bool merges = last == 1, moved = over || merges, f32 = dtype == HACK_F32;   // unit 2, contextual, or units 0 and 2 merge
          Names want{f32 ? "score_select_f32" : "score_select"};
          if (moved) want.push_back("move");
          if (merges) want.push_back("merge");
          want.push_back(f32 ? (moved ? "attn_f32" : "attn_f32_gather") : moved ? "attn_split" : "attn_split_gather");
          auto as_wanted = [&] {
            if (stub::launches != want || stub::bad_launches) return false;
            if (f32 || !moved) return stub::moving_launches.empty();
            return stub::moving_launches.size() == 1 && stub::moving_launches[0].n_units == n_comp && stub::moving_launches[0].n_append == kH - n_comp;
          };
          CHECK(run() && as_wanted());
          hack_kvcache_reset(s.cache);
          CHECK(s.step(8, 1 << 30) == HACK_OK && s.step(40, 1 << 30) == HACK_OK);
          stub::Graph g;
          stub::begin_capture(&g, kStream);
          CHECK(s.step_each(30, *budget, last == 1, 5, to) == HACK_OK);
          stub::end_capture();
          for (int replay = 0; replay < 2; ++replay) {
            stub::launches.clear();
            stub::moving_launches.clear();
            stub::replay(g);
            CHECK(as_wanted());
          }
        }
  // the float32 workspace covers every launch of a context
  for (int units : {4, 12, 60, 132})
    for (int max_len : {1, 64, 65, 511, 512, 513, 700, 2048}) {
      hack_config cfg{0, kH, kD, HACK_F32, units, max_len, 16, 32};
      hack_ctx* ctx;
      CHECK(hack_create(&ctx, &cfg) == HACK_OK);
      const int64_t have = (int64_t)(stub::device_memory.at(ctx->f32_logits) / (kF32GroupLogits * sizeof(double)));
      const int64_t partials = (int64_t)(stub::device_memory.at(ctx->stats) / (kMaxObs * 2 * sizeof(double)));
      int64_t most = 0;
      for (int d : {64, 128})
        for (int n = 1; n <= units; ++n)
          for (int t = 1; t <= max_len; ++t)
            if (use_score_select_f32(d, n, t)) most = std::max(most, score_f32_groups(n, t, 64));
      CHECK(most <= have && most <= partials && have <= kF32SmallGroups);
      hack_destroy(ctx);
    }
  return 0;
}

// Units of up to 512 keys beside longer ones: two launches where that spares a round of work-groups over the device, those that
// append rows included where they ride along (128-query attention).
int short_units_apart() {
  struct Case { int n_short, n_long, n_append; bool rows_move, apart; };
  const Case cases[] = {
      {512, 256, 0, true, true}, {512, 257, 0, true, true}, {513, 256, 0, true, true}, {513, 255, 0, true, false},   // 2 + 1 rounds for 4; for 3
      {1, 768, 0, true, false}, {768, 1, 0, true, true}, {767, 1, 0, true, false}, {256, 257, 0, true, false}, {257, 256, 0, true, true},
      {769, 0, 0, true, false}, {0, 769, 0, true, false}, {504, 8, 0, true, false}, {504, 9, 0, true, true},
      {264, 256, 200, true, false}, {264, 256, 200, false, true}, {264, 256, 256, true, true}, {264, 256, 504, true, false},
      {264, 256, 504, false, true}, {512, 256, 512, true, true}, {512, 256, 1504, true, true}, {300, 300, 400, true, false},
      {300, 100, 150, true, false},   // only the appending ones make it three rounds
  };
  std::vector<uint8_t> mem(64);
  void* p = reinterpret_cast<void*>((reinterpret_cast<uintptr_t>(mem.data()) + 15) / 16 * 16);
  uint8_t* const fresh = static_cast<uint8_t*>(p);
  for (const Case& c : cases) {
    const int U = c.n_short + c.n_long + c.n_append, n0 = 600, n1 = 100;
    setenv("HACK_ATTN_SPLIT_ITEMS", c.rows_move ? "0" : "2000000000", 1);
    hack_config cfg{0, 1, kD, HACK_BF16, U, n0 + n1, n0, 32};
    hack_ctx* ctx;
    CHECK(hack_create(&ctx, &cfg) == HACK_OK);
    unsetenv("HACK_ATTN_SPLIT_ITEMS");
    std::vector<int32_t> first(U), last(U);
    for (int i = 0; i < U; ++i) {   // the three kinds in turn through the units
      const int u = (int)((int64_t)i * 7919 % U);
      first[u] = i < c.n_short ? 412 - i % 300 : i < c.n_short + c.n_long ? 413 + i % 80 : 30;   // rows; 100 come on top: 512 and fewer, 513 and more
      last[u] = i < c.n_short + c.n_long ? first[u] : 1 << 30;
    }
    const std::vector<int32_t> cap(U, n0);
    const uint8_t type = 0;
    int64_t rows;
    hack_kvcache* cache;
    CHECK(U % 7919 != 0 && hack_kvcache_rows_required(U, cap.data(), &rows) == HACK_OK);
    CHECK(hack_kvcache_create(ctx, U, cap.data(), p, p, nullptr, rows, &cache) == HACK_OK);
    auto step = [&](int n, const std::vector<int32_t>& b) {
      return hack_step(ctx, cache, U, n, fresh, fresh + 16, fresh + 32, &type, b.data(), 5, 0.1f, fresh + ((size_t)1 << 40), nullptr, 0, kStream);
    };
    CHECK(step(n0, first) == HACK_OK);
    stub::launches.clear();
    stub::moving_launches.clear();
    CHECK(step(n1, last) == HACK_OK);
    const int n_launches = (int)std::count(stub::launches.begin(), stub::launches.end(), "score_select");
    int n_units = 0, n_append = 0;
    for (const auto& l : stub::moving_launches) {
      n_units += l.n_units;
      n_append += l.n_append;
    }
    const bool each_once = c.rows_move ? n_units == c.n_short + c.n_long && n_append == c.n_append : stub::moving_launches.empty();
    hack_kvcache_destroy(cache);
    hack_destroy(ctx);
    if (n_launches != 1 + c.apart || !each_once || stub::bad_launches) {
      printf("%d short, %d long, %d appending: %d launches, %d and %d units\n", c.n_short, c.n_long, c.n_append, n_launches, n_units, n_append);
      return 1;
    }
  }
  return 0;
}

// Every allocation of a call fails once: the call returns an error, and the same call succeeds afterwards.
template <typename Call>
bool survives(Call call) {
  for (long k = 0;; ++k) {
    if (k > 5000) return false;
    stub::allocation_failed = false;
    stub::allocations_left = k;
    const hack_status st = call();
    stub::allocations_left = -1;
    if (!stub::allocation_failed) return st == HACK_OK && k > 0;
    // (an allocation that has a fallback, as the buffer of a stable sort, may fail without failing the call)
    if (st != HACK_OK && st != HACK_EHIP) return false;
  }
}

int no_exceptions() {
  for (int dtype : {HACK_BF16, HACK_F32}) {
    CHECK(survives([&] {
      hack_config cfg{0, kH, kD, dtype, kH, 128, 64, 32};
      hack_ctx* ctx;
      const hack_status st = hack_create(&ctx, &cfg);
      if (st == HACK_OK) hack_destroy(ctx);
      return st;
    }));
    CHECK(stub::device_memory.empty());
    const std::vector<int32_t> caps(kH, 200);
    {
      Setup s(dtype, 64, 128, 64);
      int64_t rows;
      hack_kvcache_rows_required(kH, caps.data(), &rows);
      CHECK(survives([&] {
        hack_kvcache* c;
        const hack_status st = hack_kvcache_create(s.ctx, kH, caps.data(), s.q, s.q, nullptr, rows, &c);
        if (st == HACK_OK) hack_kvcache_destroy(c);
        return st;
      }));
    }
    // steps: a fresh cache each time, so that every call plans; a failed step leaves the state alone
    for (int last = 0; last < 3; ++last) {
      if (last == 2 && dtype == HACK_F32) continue;
      CHECK(survives([&] {
        ++stub::quiet;
        Setup s(dtype, 64, 128, 64);
        s.step(8, 1 << 30);
        s.step(40, 1 << 30);
        --stub::quiet;
        const hack_status st = s.step(last == 0 ? 10 : 30, last == 0 ? 1 << 30 : 50, last == 2);
        const stub::Quiet checks;
        hack_cache view;
        hack_kvcache_view(s.cache, &view);
        for (int u = 0; u < kH; ++u)
          if (view.len[u] != (st != HACK_OK ? 48 : last == 0 ? 58 : 50)) return HACK_EINVAL;
        if (s.step(last == 0 ? 2 : 5, 50) != HACK_OK) return HACK_EINVAL;
        return st;
      }));
    }
    {
      Setup s(dtype, 64, 128, 64);
      const int64_t off[kH] = {0, 128, 256, 384}, off_out[kH] = {512, 640, 768, 896};
      const int32_t len[kH] = {60, 50, 40, 30}, len_out[kH] = {20, 20, 20, 20}, t_in[kH] = {80, 70, 60, 50};
      const uint8_t types[kH] = {0, 1, 0, 1};
      std::vector<uint8_t> rows(1024 * kD * 4 + 64);
      void* p = reinterpret_cast<void*>((reinterpret_cast<uintptr_t>(rows.data()) + 63) / 64 * 64);
      const hack_cache in{p, p, nullptr, 1024, off, len}, out{p, p, nullptr, 1024, off_out, len_out};
      int32_t* kept = static_cast<int32_t*>(p);
      float* imp = static_cast<float*>(p);
      double* sigma = static_cast<double*>(p);
      int n = 0;
      // other arguments each time, so that every call builds and uploads a table
      CHECK(survives([&] { return hack_score(s.ctx, 1, 20 + n++ % 40, s.q, nullptr, 16, 0.1f, &in, s.k, nullptr, imp, 128, kStream); }));
      CHECK(survives([&] { return hack_select(s.ctx, 1, imp, 128, t_in, types, len_out, n++ % 30, 20, kept, 128, nullptr, kStream); }));
      CHECK(survives([&] { return hack_compact(s.ctx, 1, 20 + n++ % 40, &in, s.k, s.v, 0, kept, 128, &out, kStream); }));
      CHECK(survives([&] { return hack_attn(s.ctx, 1, 20 + n++ % 40, s.q, &in, 0.1f, s.out, kStream); }));
      if (dtype == HACK_BF16) {
        CHECK(survives([&] { return hack_score_static(s.ctx, 1, 20, s.q, nullptr, 16, 0.1f, &in, s.k, nullptr, imp, 128, kStream); }));
        CHECK(survives([&] { return hack_merge(s.ctx, 1, 20 + n++ % 40, &in, s.k, s.v, kept, 128, nullptr, &out, kStream); }));
        CHECK(survives([&] { return hack_head_variance(s.ctx, 1, 20, s.q, n++ % 2 ? &in : &out, 0.1f, sigma, kStream); }));
      }
    }
    CHECK(stub::bad_launches == 0 && stub::device_memory.empty());
  }
  return 0;
}

// A step that is remembered is found again only with the same arguments: sink rows, score mode, plain or final.
int step_keys() {
  Setup s(HACK_BF16, 400, 1000, 300);
  auto last_step = [&](int n_init, bool final_merge, int mode) -> const StepNode* {
    if (hack_set_score_mode(s.ctx, mode) != HACK_OK) return nullptr;
    hack_kvcache_reset(s.cache);
    stub::launches.clear();
    if (s.step(300, 1 << 30) != HACK_OK || s.step(200, 250, final_merge, n_init) != HACK_OK) return nullptr;
    return s.cache->at;
  };
  auto launched = [](const char* name) { return std::find(stub::launches.begin(), stub::launches.end(), name) != stub::launches.end(); };
  std::vector<const StepNode*> nodes;
  for (int pass = 0; pass < 2; ++pass) {
    size_t i = 0;
    for (int mode : {HACK_SCORE_FUSED, HACK_SCORE_TWO_PASS})
      for (int n_init : {5, 9})
        for (bool final_merge : {false, true}) {
          const StepNode* n = last_step(n_init, final_merge, mode);
          CHECK(n != nullptr);
          CHECK(launched("merge") == final_merge && launched("score_two_pass") == (mode == HACK_SCORE_TWO_PASS) &&
                launched("score_fused") == (mode == HACK_SCORE_FUSED));
          if (pass == 0) {
            CHECK(std::find(nodes.begin(), nodes.end(), n) == nodes.end());
            nodes.push_back(n);
          } else {
            CHECK(nodes[i++] == n);
          }
        }
  }
  CHECK(stub::bad_launches == 0);
  return 0;
}

// The table of a step holds every unit's descriptor once: the compressing units first, either kind in the order of the units.
int step_tables() {
  for (int dtype : {HACK_BF16, HACK_F32})
    for (int long_units = 0; long_units < 2; ++long_units)   // score and selection in one launch, in launches of their own
      for (int compress = 0; compress < 16; ++compress) {    // bit u: unit u compresses
        Setup s(dtype, long_units ? 1100 : 96, 1200, 900);
        const int n[2] = {long_units ? 900 : 40, 30};
        int32_t budget[kH];
        for (int u = 0; u < kH; ++u) budget[u] = compress >> u & 1 ? n[0] - u : 1 << 30;
        CHECK(s.step(n[0], 1 << 30) == HACK_OK && s.step_each(n[1], budget) == HACK_OK);
        const StepGroup& g = s.cache->at->g[0];
        const int n_comp = __builtin_popcount(compress);
        CHECK(g.n_desc == kH && g.n_comp == n_comp);
        const UnitDesc* d = g.ddev();
        int at = 0;
        for (const int kind : {MOVE_GATHER, MOVE_APPEND})
          for (int u = 0; u < kH; ++u)
            if ((compress >> u & 1) == (kind == MOVE_GATHER)) {
              CHECK(d[at].unit == u && d[at].mode == kind);
              ++at;
            }
        int copies = 0;
        for (size_t o = 0; o + sizeof(UnitDesc) <= stub::copied; o += 16)   // of the step's table
          for (int u = 0; u < kH; ++u) copies += memcmp(g.dev + o, &d[u], sizeof(UnitDesc)) == 0;
        CHECK(copies == kH);
      }
  CHECK(stub::bad_launches == 0);
  return 0;
}

// Which launches the key-split attention kernel serves, and that a limit given in the environment is taken as it is.
int attn_rule() {
  const auto variants = [](int head_dim, const char* limit, std::vector<std::pair<int, int>> shapes) {   // (units, queries)
    if (limit) setenv("HACK_ATTN_SPLIT_ITEMS", limit, 1);
    hack_config cfg{0, 1, head_dim, HACK_BF16, 4096, 64, 4096, 32};
    hack_ctx* ctx = nullptr;
    std::string got;
    if (hack_create(&ctx, &cfg) != HACK_OK) return got;
    for (const auto& x : shapes) got += (char)('0' + hack_attn_variant(ctx, x.first, x.second));
    hack_destroy(ctx);
    unsetenv("HACK_ATTN_SPLIT_ITEMS");
    return got;
  };
  // head_dim 64: 2048 items of 32 queries, fewer where tiles of 128 queries are well filled and start together; head_dim 128: 512
  CHECK(variants(64, nullptr, {{2048, 32}, {2049, 32}, {512, 128}, {513, 128}}) == "1010");
  CHECK(variants(64, nullptr, {{187, 256}, {188, 256}, {256, 256}, {257, 256}, {48, 900}, {49, 900}, {77, 576}, {78, 576}, {60, 1024}}) == "100010100");
  CHECK(variants(64, nullptr, {{300, 160}, {409, 130}, {410, 130}, {400, 140}, {341, 192}, {342, 192}, {280, 224}, {156, 400}}) == "11011011");   // half-empty tiles
  CHECK(variants(64, nullptr, {{102, 576}, {103, 576}, {113, 576}, {114, 576}}) == "0110");   // 510 and 515 of 128 queries
  CHECK(variants(128, nullptr, {{512, 32}, {513, 32}, {128, 128}, {129, 128}, {102, 129}, {103, 129}}) == "101010");
  for (const char* limit : {"2047", "2048", "2049"}) {
    const int n = atoi(limit);
    CHECK(variants(64, limit, {{n, 32}, {n + 1, 32}, {n / 5, 129}, {n / 5 + 1, 129}, {60, 1024}}) == "10101");
  }
  CHECK(variants(64, "0", {{1, 1}, {1, 129}}) == "00" && variants(64, "-1", {{1, 1}}) == "0" && variants(64, "1", {{1, 32}, {1, 33}, {1, 129}}) == "100");
  CHECK(variants(128, "512", {{512, 32}, {513, 32}, {102, 129}, {103, 129}}) == "1010");
  return 0;
}

// Steps of short units that one launch does: every unit once, in the routes that outputs over an input take (scores, selection and moves in
// front of it; nothing may read queries or new rows that another work-group stores over), eagerly and from a graph; merging, appending and forced
// steps take the launches that they took, and so do steps beyond the sizes.
int whole_steps() {
  typedef std::vector<std::string> Names;
  stub::lds_bytes = 163840;
  const int32_t all[kH] = {50, 50, 50, 50}, some[kH] = {50, 1 << 30, 1 << 30, 40}, none[kH] = {1 << 30, 1 << 30, 1 << 30, 1 << 30};
  for (const auto* budget : {&all, &some, &none})
    for (int over = 0; over < 4; ++over)
      for (int last = 0; last < 2; ++last) {
        Setup s(HACK_BF16, 96, 128, 64);
        void* to = over == 0 ? s.out : over == 1 ? s.q : over == 2 ? s.k : s.v;
        Names want;
        if (budget == &none) want = over < 2 ? Names{"attn_split_append"} : Names{"move", "attn_split"};
        else if (last) want = {"score_select", "move", "merge", "attn_split"};
        else if (over == 0) want = {"step_whole"};
        else want = {"score_select", "move", "attend_whole"};
        auto before = [&] {
          hack_kvcache_reset(s.cache);
          return s.step(8, 1 << 30) == HACK_OK && s.step(40, 1 << 30) == HACK_OK;
        };
        auto as_wanted = [&] {
          if (stub::launches != want || stub::bad_launches) return false;
          if (budget == &none || last) return stub::whole_launches.empty();
          if (stub::whole_launches.size() != 1) return false;
          const stub::WholeLaunch& l = stub::whole_launches[0];
          std::vector<int> seen(kH, 0);
          int max_t = 0, max_rows = 0;
          for (const UnitDesc& d : l.descs) {
            ++seen[d.unit];
            max_rows = std::max(max_rows, d.n_out);
            if (d.mode == MOVE_GATHER) max_t = std::max(max_t, d.len_in + d.n_new);
            if (d.n_out != std::min((*budget)[d.unit], 78) || d.n_new != 30) return false;
          }
          return seen == std::vector<int>(kH, 1) && l.step.max_t == max_t && l.step.max_rows == max_rows && l.step.n_obs == 30 && l.step.moved == (over != 0);
        };
        CHECK(before());
        for (int pass = 0; pass < 2; ++pass) {   // planned, remembered
          CHECK(before());
          stub::launches.clear();
          stub::whole_launches.clear();
          CHECK(s.step_each(30, *budget, last == 1, 5, to) == HACK_OK && as_wanted());
          const StepGroup& group = s.cache->at->g[0];
          CHECK(hack_kvcache_step_form(s.cache) == (stub::whole_launches.empty() ? 0 : 16));
          CHECK((group.whole == 0) == (group.n_items > 0) && (group.whole == 0 || group.n_moves == 0));   // nothing planned that no launch reads
        }
        CHECK(before() && hack_kvcache_step_form(s.cache) == 0);
        stub::Graph g;
        stub::begin_capture(&g, kStream);
        CHECK(s.step_each(30, *budget, last == 1, 5, to) == HACK_OK);
        stub::end_capture();
        for (int replay = 0; replay < 2; ++replay) {
          stub::launches.clear();
          stub::whole_launches.clear();
          stub::replay(g);
          CHECK(as_wanted());
        }
      }
  for (const char* name : {"HACK_ATTN_SPLIT_ITEMS", "HACK_ATTN_PIPE", "HACK_ATTN_STREAM", "HACK_STEP_OVERLAP"}) {   // a form that is asked for
    setenv(name, "1", 1);
    Setup s(HACK_BF16, 96, 128, 64);
    unsetenv(name);
    stub::launches.clear();
    CHECK(s.schedule());
    CHECK(std::find(stub::launches.begin(), stub::launches.end(), "step_whole") == stub::launches.end());
  }
  // queries per work-group: several work-groups a unit while each finds one of the 32 compute units of its XCD, which takes every eighth unit; one
  // work-group a unit beyond; nothing beyond the LDS
  const auto q = [](int d, int units, int n, int t, int rows, int comp = 1 << 20) {
    return whole_step_queries(d, units, std::min(comp, units), n, t, rows, 163840);
  };
  CHECK(q(64, 56, 64, 166, 100) == 16 && q(64, 57, 64, 166, 100) == 32 && q(64, 128, 64, 166, 100) == 32 && q(64, 129, 64, 166, 100) == 256);
  CHECK(q(64, 60, 144, 250, 100) == 256 && q(64, 60, 145, 250, 100) == 64 && q(64, 120, 256, 500, 300) == 128 && q(64, 256, 256, 500, 300) == 256);
  CHECK(q(64, 60, 144, 400, 256) == 256 && q(64, 60, 144, 400, 257) == 64 && q(128, 60, 144, 400, 192) == 256 && q(128, 60, 144, 400, 193) == 64);
  // few units hold many work-groups on few XCDs
  CHECK(q(128, 3, 448, 500, 95) == 16 && q(128, 3, 449, 500, 95) == 32 && q(128, 8, 512, 512, 95) == 32 && q(128, 9, 256, 512, 95) == 32 && q(128, 9, 512, 600, 95) == 32);
  CHECK(q(128, 9, 513, 600, 95) == 0 && q(64, 27, 256, 500, 71) == 32 && q(64, 27, 300, 500, 71) == 64 && q(64, 27, 301, 500, 71) == 0 && q(64, 40, 320, 500, 71) == 0 && q(64, 41, 320, 500, 71) == 64);
  CHECK(q(128, 32, 600, 640, 71) == 128 && q(64, 32, 600, 640, 71) == 0 && q(64, 48, 600, 640, 71) == 128);
  // more than 256 units: one work-group each, where the launch's own sizes do not make it the slower one
  CHECK(q(64, 960, 256, 562, 306) == 256 && q(64, 960, 257, 562, 306) == 0 && q(64, 960, 33, 80, 40) == 256 && q(64, 960, 32, 80, 40) == 0);
  CHECK(q(128, 512, 97, 257, 140) == 256 && q(128, 512, 96, 257, 140) == 0 && q(128, 256, 36, 90, 60) == 256);
  CHECK(q(128, 264, 128, 256, 256) == 0 && q(128, 264, 129, 256, 97) == 256 && q(128, 264, 129, 256, 96) == 0 && q(128, 264, 128, 256, 256, 128) == 256 && q(128, 264, 128, 256, 256, 129) == 0);
  CHECK(q(64, 264, 256, 512, 256) == 256 && q(64, 264, 256, 512, 257) == 0 && q(64, 264, 256, 513, 257) == 256);
  CHECK(q(64, 512, 100, 250, 150) == 256 && q(64, 513, 100, 250, 150) == 0 && q(64, 768, 100, 250, 150) == 0 && q(64, 769, 100, 250, 150) == 256);
  CHECK(q(64, 520, 113, 250, 150) == 256 && q(64, 520, 100, 257, 150) == 256 && q(64, 1025, 100, 250, 150) == 0 && q(64, 600, 100, 250, 150, 513) == 0 && q(64, 600, 100, 250, 150, 512) == 256);
  CHECK(q(64, 60, 100, 1024, 300) > 0 && q(64, 60, 100, 1025, 300) == 0 && q(64, 16, 100, 768, 300) == 16 && q(64, 16, 100, 769, 300) == 0);
  CHECK(q(64, 8, 100, 640, 300) == 16 && q(64, 8, 100, 641, 300) == 0 && q(128, 8, 100, 512, 200) == 16 && q(128, 8, 100, 513, 200) == 0);
  CHECK(q(128, 32, 100, 640, 200) == 16 && q(128, 32, 100, 641, 200) == 0 && q(128, 64, 100, 896, 200) == 32 && q(128, 64, 100, 897, 200) == 0);
  CHECK(q(64, 60, 100, 600, 544) > 0 && q(64, 60, 100, 600, 560) == 0 && q(128, 60, 100, 300, 256) > 0 && q(128, 60, 100, 300, 288) == 0);
  CHECK(whole_step_queries(64, 60, 60, 100, 300, 100, 65536) == 0);
  stub::lds_bytes = 256;
  return 0;
}

// Waves of a key-split work-group: a step that compresses to n_keys rows and hack_attn over as many take the same number (the bits depend
// on it), eight where that is the faster one for both.
int split_waves() {
  struct Case { int head_dim, units, queries, keys, waves; };
  const Case cases[] = {
      {64, 32, 32, 640, 4}, {64, 32, 32, 641, 8}, {64, 64, 128, 700, 8}, {64, 72, 128, 700, 4}, {64, 256, 32, 2000, 8},
      {128, 16, 64, 640, 4}, {128, 16, 64, 641, 8}, {128, 32, 160, 700, 8}, {128, 32, 192, 700, 8}, {128, 16, 448, 700, 8},
      // compute units left for the work-groups that move a step's rows
      {128, 32, 224, 1024, 4}, {128, 32, 224, 1025, 8}, {128, 16, 512, 700, 4}, {128, 16, 512, 1500, 8}, {128, 64, 96, 700, 4},
      {128, 64, 96, 1500, 8}, {128, 32, 256, 700, 4}, {128, 32, 256, 1500, 4}, {128, 64, 128, 3000, 4}, {128, 96, 64, 1500, 4}, {128, 128, 64, 3000, 4},
  };
  std::vector<uint8_t> mem(64 << 20);
  void* p = reinterpret_cast<void*>((reinterpret_cast<uintptr_t>(mem.data()) + 63) / 64 * 64);
  uint8_t* const fresh = static_cast<uint8_t*>(p);
  for (const Case& c : cases) {
    hack_config cfg{0, c.units, c.head_dim, HACK_BF16, c.units, c.keys + c.queries, std::max(c.keys, c.queries), 32};
    hack_ctx* ctx;
    CHECK(hack_create(&ctx, &cfg) == HACK_OK);
    const std::vector<int32_t> cap(c.units, c.keys), all(c.units, 1 << 30);
    const std::vector<uint8_t> types(c.units, 0);
    int64_t rows;
    hack_kvcache* cache;
    CHECK(hack_kvcache_rows_required(c.units, cap.data(), &rows) == HACK_OK);
    CHECK(hack_kvcache_create(ctx, c.units, cap.data(), p, p, nullptr, rows, &cache) == HACK_OK);
    auto step = [&](int n, const std::vector<int32_t>& b) {
      return hack_step(ctx, cache, 1, n, fresh, fresh, fresh, types.data(), b.data(), 5, 0.1f, fresh + (48 << 20), nullptr, 0, kStream);
    };
    CHECK(step(c.keys, all) == HACK_OK);
    stub::waves.clear();
    stub::launches.clear();
    CHECK(step(c.queries, cap) == HACK_OK);
    CHECK(stub::launches.back() == "attn_split_gather");
    hack_cache view;
    CHECK(hack_kvcache_view(cache, &view) == HACK_OK);
    CHECK(hack_attn(ctx, 1, c.queries, fresh, &view, 0.1f, fresh, kStream) == HACK_OK);
    if (stub::waves != std::vector<int>{c.waves, c.waves}) {
      printf("head_dim %d, %d units, %d queries, %d keys: %d and %d waves\n", c.head_dim, c.units, c.queries, c.keys, stub::waves[0], stub::waves[1]);
      return 1;
    }
    hack_kvcache_destroy(cache);
    hack_destroy(ctx);
  }
  return 0;
}

// 128-query launches of at most one work item per compute unit: the two halves of the keys side by side where most items are long,
// whole items (the long ones cut) where few are.
int key_halves() {
  struct Case { int units, tiles, n_long, long_blocks, short_blocks; bool halves; };
  const Case cases[] = {
      {32, 8, 32, 79, 79, true}, {32, 8, 20, 79, 61, true}, {32, 5, 32, 41, 41, true}, {16, 16, 16, 28, 28, true}, {16, 16, 16, 27, 27, false},
      {8, 32, 2, 160, 16, true},      // one unit an XCD: the long ones' XCDs hold nothing else
      {16, 15, 8, 160, 16, false}, {32, 8, 8, 80, 24, false}, {32, 6, 8, 160, 80, false}, {64, 4, 16, 160, 80, false}, {32, 5, 16, 80, 24, false},
      {33, 8, 33, 79, 79, false},     // 264 items
      {32, 8, 31, 79, 1, false},      // a unit of one block has no second half
  };
  std::vector<uint8_t> mem(64);
  void* p = reinterpret_cast<void*>((reinterpret_cast<uintptr_t>(mem.data()) + 15) / 16 * 16);
  for (const Case& c : cases) {
    hack_config cfg{0, c.units, 128, HACK_BF16, c.units, 8192, 4096, 32};
    hack_ctx* ctx;
    CHECK(hack_create(&ctx, &cfg) == HACK_OK);
    std::vector<int64_t> off(c.units);
    std::vector<int32_t> len(c.units, 32 * c.short_blocks);
    for (int i = 0; i < c.n_long; ++i) len[i * c.units / c.n_long] = 32 * c.long_blocks;
    for (int u = 0; u < c.units; ++u) off[u] = 8192 * u;
    const hack_cache kv{p, p, nullptr, 8192 * c.units, off.data(), len.data()};
    stub::launches.clear();
    CHECK(hack_attn(ctx, 1, 128 * c.tiles, p, &kv, 0.1f, p, kStream) == HACK_OK);
    const bool halves = stub::launches.back() == "attn_halves";
    hack_destroy(ctx);
    if (halves != c.halves) {
      printf("%d units of %d tiles, %d of %d blocks and the rest of %d: %s\n", c.units, c.tiles, c.n_long, c.long_blocks, c.short_blocks, stub::launches.back().c_str());
      return 1;
    }
  }
  return 0;
}

// The float32 score workspace covers every launch the context accepts (chunk of 64 keys for small ones, 256 beyond) and
// is no larger than those need.
int f32_workspace() {
  for (int units : {4, 16, 60, 64, 132}) {
    for (int max_len : {1, 64, 65, 680, 2048, 10521, 32768}) {
      hack_config cfg{0, kH, kD, HACK_F32, units, max_len, 16, 32};
      hack_ctx* ctx;
      CHECK(hack_create(&ctx, &cfg) == HACK_OK);
      const int64_t have = (int64_t)(stub::device_memory.at(ctx->stats) / (kMaxObs * 2 * sizeof(double)));   // (unit, chunk) pairs
      int64_t most = 0;
      for (int n = 1; n <= units; ++n)
        for (int t = 1; t <= max_len; t += t < max_len && t + 61 > max_len ? max_len - t : 61)
          most = std::max(most, (int64_t)n * ((t + score_f32_chunk(n, t) - 1) / score_f32_chunk(n, t)));
      CHECK(most <= have);
      CHECK(have <= std::max<int64_t>(640, (int64_t)units * ((max_len + 255) / 256)));
      hack_destroy(ctx);
    }
  }
  return 0;
}

}  // namespace

// Keys per score item: the smallest that fit one launch, otherwise those that need the fewest; at head_dim 64 items of 192 keys only in place of 256,
// where they spare a launch or put no more work-groups on a compute unit in the last one.
int score_items() {
  hack_ctx* ctx[2] = {};
  for (int i = 0; i < 2; ++i) {
    hack_config cfg{0, 1, 64 << i, HACK_BF16, 1024, 8192, 64, 32};
    CHECK(hack_create(&ctx[i], &cfg) == HACK_OK);
  }
  const auto keys = [&](int d, int n, int t, int n2 = 0, int t2 = 1) {   // n units of t keys, n2 of t2
    std::vector<int32_t> ts(n, t);
    ts.insert(ts.begin(), n2, t2);
    return hack_score_item_keys(ctx[d == 128], n + n2, ts.data());
  };
  // head_dim 128: 512 work-groups a launch
  CHECK(keys(128, 512, 128) == 32 && keys(128, 512, 129) == 64 && keys(128, 128, 1024) == 64 && keys(128, 128, 1025) == 96 && keys(128, 128, 1536) == 96);
  CHECK(keys(128, 128, 1537) == 128 && keys(128, 128, 2048) == 128 && keys(128, 128, 2049) == 192 && keys(128, 128, 3072) == 192 && keys(128, 128, 3073) == 256);
  CHECK(keys(128, 128, 4097) == 192 && keys(128, 513, 128) == 32 && keys(128, 513, 384) == 96 && keys(128, 400, 384, 112, 384) == 96);
  // head_dim 64: 1280, 1024, 768, 512, 768 and 512
  CHECK(keys(64, 256, 640) == 32 && keys(64, 256, 641) == 64 && keys(64, 256, 1024) == 64 && keys(64, 256, 1025) == 96 && keys(64, 256, 1152) == 96);
  CHECK(keys(64, 128, 3072) == 192 && keys(64, 128, 3073) == 256 && keys(64, 129, 3072) == 256);      // 512, 640, 516 work-groups; 256: 384, 512, 387
  CHECK(keys(64, 109, 4999) == 192);                                                                 // one launch for two
  CHECK(keys(64, 100, 5776) == 192 && keys(64, 103, 6923) == 256 && keys(64, 130, 7182) == 192);      // 32 and 90, 270 and 210 in the last; two launches for three
  CHECK(keys(64, 643, 781) == 256 && keys(64, 100, 7700) == 192);                                    // 3 for 1, 2 for 2 on a compute unit
  CHECK(keys(64, 521, 484) == 64 && keys(64, 259, 1188) == 64 && keys(64, 562, 1040) == 64);          // not for 32 and 64
  CHECK(keys(64, 100, 5147) == 96 && keys(64, 613, 1040) == 96);                                     // nor for 96
  CHECK(keys(64, 16, 8192) == 32 && keys(64, 16, 8192, 1000, 32) == 32);
  // units of a few lengths, in any order: launches counted one unit at a time, as build_score_items fills them
  unsigned seed = 1;
  const auto rnd = [&](int n) { return (int)((seed = seed * 1664525u + 1013904223u) >> 8) % n; };
  for (int rep = 0; rep < 400; ++rep) {
    std::vector<int32_t> ts(1 + rnd(700));
    int32_t some[5];
    for (int32_t& t : some) t = 1 + rnd(rep % 2 ? 8192 : 900);
    for (int32_t& t : ts) t = rep % 3 ? some[rnd(5)] : 1 + rnd(1200);
    const int32_t got = hack_score_item_keys(ctx[1], (int)ts.size(), ts.data());
    std::sort(ts.begin(), ts.end(), [](int a, int b) { return a > b; });
    int want = 0, fewest = 1 << 30;
    for (int k : {32, 64, 96, 128, 192, 256}) {
      int launches = 1, in_launch = 0;
      for (int t : ts) {
        const int groups = ((t + k - 1) / k + 3) / 4;
        if (in_launch + groups > 512) ++launches, in_launch = 0;
        in_launch += groups;
      }
      if (launches < fewest) want = k, fewest = launches;
      if (launches == 1) break;
    }
    CHECK(got == want);
  }
  // the order of the units does not matter; what is refused
  const int32_t a[] = {700, 300, 8000}, b[] = {8000, 700, 300}, bad[] = {5, 0}, large[] = {8193};
  CHECK(hack_score_item_keys(ctx[0], 3, a) == hack_score_item_keys(ctx[0], 3, b));
  CHECK(hack_score_item_keys(ctx[0], 2, bad) == HACK_EINVAL && hack_score_item_keys(ctx[0], 1, large) == HACK_EINVAL);
  CHECK(hack_score_item_keys(ctx[0], 0, a) == HACK_EINVAL && hack_score_item_keys(ctx[0], 1, nullptr) == HACK_EINVAL);
  for (hack_ctx* c : ctx) hack_destroy(c);
  return 0;
}

int main(int argc, char** argv) {
  const std::string which = argc > 1 ? argv[1] : "";
  int rc = 2;
  if (which == "capture") rc = capture();
  if (which == "out_over_new_rows") rc = out_over_new_rows();
  if (which == "short_units") rc = short_units();
  if (which == "short_units_apart") rc = short_units_apart();
  if (which == "no_exceptions") rc = no_exceptions();
  if (which == "step_keys") rc = step_keys();
  if (which == "step_tables") rc = step_tables();
  if (which == "split_waves") rc = split_waves();
  if (which == "key_halves") rc = key_halves();
  if (which == "attn_rule") rc = attn_rule();
  if (which == "f32_workspace") rc = f32_workspace();
  if (which == "whole_steps") rc = whole_steps();
  if (which == "score_items") rc = score_items();
  if (rc == 0) printf("ok\n");
  return rc;
}
