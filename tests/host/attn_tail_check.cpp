// Host check of plan_attn_tail: every block of every work item served once, by parts that are numbered consistently; only last
// rounds of equal items are cut, into no more pieces than the XCD has compute units.  No GPU involved.
#include <cstdio>
#include <map>
#include <vector>

#include "../../paper_2504_09261_amd/csrc/attn_plan.h"

using namespace hack;

#define CHECK(c)                                                                    \
  do {                                                                              \
    if (!(c)) { std::printf("FAILED line %d: %s\n", __LINE__, #c); return 1; }      \
  } while (0)

static int check(const int (&sizes)[kAttnXcds], int blocks, int shorter, int cus, bool expect) {
  std::vector<AttnLaneItem> lanes[kAttnXcds];
  int desc = 0, most = 0;
  for (int x = 0; x < kAttnXcds; ++x, ++desc)
    for (int i = 0; i < sizes[x]; ++i) lanes[x].push_back(AttnLaneItem{desc, i, x == kAttnXcds - 1 ? blocks - shorter : blocks});
  for (int n : sizes) most = std::max(most, n);
  AttnStreamPlan p;
  CHECK(plan_attn_tail(lanes, cus, &p) == expect);
  if (!expect) return 0;
  CHECK(p.n_groups % kAttnXcds == 0 && (int)p.seg_begin.size() == p.n_groups + 1 && p.seg_begin[0] == 0 && p.seg_begin.back() == (int)p.segs.size());
  std::map<std::pair<int, int>, std::vector<AttnSeg>> items;
  int per_xcd_pieces[kAttnXcds] = {};
  for (int g = 0; g < p.n_groups; ++g) {
    const int n = p.seg_begin[g + 1] - p.seg_begin[g];
    CHECK(n == 0 || n == 1);
    if (n == 0) continue;
    const AttnSeg& s = p.segs[p.seg_begin[g]];
    CHECK(s.desc == g % kAttnXcds);     // a unit stays on its XCD
    items[{s.desc, s.q_tile}].push_back(s);
    per_xcd_pieces[g % kAttnXcds] += s.part >= 0;
  }
  std::vector<int> parts(p.n_parts, 0), counters(p.n_counters, 0);
  size_t n_items = 0;
  for (int x = 0; x < kAttnXcds; ++x) {
    CHECK(per_xcd_pieces[x] <= cus);
    n_items += sizes[x];
  }
  CHECK(items.size() == n_items);
  for (auto& kv : items) {
    const auto& v = kv.second;
    const int nb = kv.first.first == kAttnXcds - 1 ? blocks - shorter : blocks;
    if (v.size() == 1) {
      CHECK(v[0].part < 0 && v[0].blk0 == 0 && v[0].blk1 >= nb);
      continue;
    }
    CHECK((int)v.size() <= kTailMaxPieces && v[0].counter >= 0 && v[0].counter < p.n_counters);
    ++counters[v[0].counter];
    for (size_t i = 0; i < v.size(); ++i) {
      CHECK(v[i].blk0 == (i ? v[i - 1].blk1 : 0) && v[i].blk1 > v[i].blk0 && v[i].n_parts == (int)v.size());
      CHECK(v[i].first_part == v[0].part && v[i].part == v[0].part + (int)i && v[i].part < p.n_parts && v[i].counter == v[0].counter);
      ++parts[v[i].part];
    }
    CHECK(v.back().blk1 == nb);
  }
  for (int u : parts) CHECK(u == 1);
  for (int u : counters) CHECK(u == 1);
  return 0;
}

int main() {
  int bad = 0;
  for (int blocks : {40, 41, 47, 201, 1024})
    for (int r = 0; r < 64; ++r)
      for (int q : {0, 1, 2, 5}) {
        const int n = q * 64 + r;
        bad |= check({n, n, n, n, n, n, n, n}, blocks, 0, 32, q > 0 && r > 0 && r <= 16);
        bad |= check({n, n, n, 0, n, n > 3 ? n - 3 : 0, n, n}, blocks, 0, 32, q > 0 && r > 0 && r <= 16);
      }
  bad |= check({72, 72, 72, 72, 72, 72, 72, 72}, 39, 0, 32, false);      // too short to pay for the parts
  bad |= check({72, 72, 72, 72, 72, 72, 72, 72}, 160, 10, 32, true);     // lengths within a sixteenth
  bad |= check({72, 72, 72, 72, 72, 72, 72, 72}, 160, 11, 32, false);
  bad |= check({9, 9, 9, 9, 9, 9, 9, 9}, 100, 0, 4, true);               // four compute units an XCD
  bad |= check({9, 9, 9, 9, 9, 9, 9, 9}, 100, 0, 0, false);
  if (!bad) std::printf("ok\n");
  return bad;
}
