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
    const uint8_t types[kH] = {0, 1, 0, 1};
    std::vector<int32_t> b(kH, budget);
    auto fn = final_merge ? hack_step_final : hack_step;
    return fn(ctx, cache, 1, n, q, k, v, types, b.data(), n_init, 0.125f, to ? to : out, nullptr, 0, kStream);
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

}  // namespace

int main(int argc, char** argv) {
  const std::string which = argc > 1 ? argv[1] : "";
  int rc = 2;
  if (which == "capture") rc = capture();
  if (which == "out_over_new_rows") rc = out_over_new_rows();
  if (rc == 0) printf("ok\n");
  return rc;
}
