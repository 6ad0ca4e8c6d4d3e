// Content-addressed store of launch tables (per-unit descriptors and work lists).
//
// A table is uploaded the first time its contents are seen and keeps its device
// address until the store is destroyed: kernels that were queued earlier, and HIP
// graphs captured earlier, go on reading the address they were given, so storage
// that has been handed out is never moved, overwritten or reused.  When a chunk
// is full another one is chained behind it; chunks are released together at the
// end.  Growth is bounded by a total limit.
//
// A copy issued on a stream that is being captured is not carried out, it becomes a
// node of the graph.  Such a table is known (it has its address and its host mirror)
// but not uploaded: every call that needs it issues the copy again, to the same
// address with the same bytes, until one outside a capture has done so.
//
// The memory back end is a template parameter, so that the bookkeeping can be
// exercised on the host without a device (the unit test plugs in malloc).
//   struct Backend {
//     bool alloc(size_t bytes, uint8_t** dev, uint8_t** host);   // one chunk: device memory + host mirror
//     void release(uint8_t* dev, uint8_t* host);
//     bool upload(uint8_t* dev, const uint8_t* host, size_t bytes, void* stream);  // asynchronous on stream
//     bool may_alloc(void* stream);                              // false while `stream` is being captured
//   };
#pragma once

#include <stddef.h>
#include <stdint.h>
#include <string.h>

#include <unordered_map>
#include <vector>

namespace hack {

enum class TableStatus { kOk, kTooLarge, kFullDuringCapture, kLimit, kAllocFailed, kUploadFailed };

template <typename Backend>
class TableCache {
 public:
  TableCache(Backend backend, size_t chunk_bytes, size_t limit_bytes)
      : be_(backend), chunk_bytes_(chunk_bytes), limit_bytes_(limit_bytes) {}
  TableCache(const TableCache&) = delete;
  TableCache& operator=(const TableCache&) = delete;
  ~TableCache() {
    for (Chunk& c : chunks_) be_.release(c.dev, c.host);
  }

  // Device address of a table with exactly these bytes, for work that is issued on `stream` next.  id (may be NULL)
  // gets a number for upload() and uploaded(), valid as long as the store.
  TableStatus get(const uint8_t* bytes, size_t n, void* stream, const uint8_t** dev, size_t* id = nullptr) {
    const uint64_t h = hash(bytes, n);
    auto range = index_.equal_range(h);
    for (auto it = range.first; it != range.second; ++it) {
      const Entry& e = entries_[it->second];
      if (e.bytes == n && memcmp(chunks_[e.chunk].host + e.offset, bytes, n) == 0) {
        *dev = chunks_[e.chunk].dev + e.offset;
        if (id) *id = it->second;
        return upload(it->second, stream);
      }
    }
    const size_t need = (n + kAlign - 1) / kAlign * kAlign;
    if (need > chunk_bytes_) return TableStatus::kTooLarge;
    if (chunks_.empty() || chunks_.back().used + need > chunk_bytes_) {
      if (!be_.may_alloc(stream)) return TableStatus::kFullDuringCapture;
      if ((chunks_.size() + 1) * chunk_bytes_ > limit_bytes_) return TableStatus::kLimit;
      if (!add_chunk()) return TableStatus::kAllocFailed;
    }
    Chunk& c = chunks_.back();
    const size_t off = c.used;
    memcpy(c.host + off, bytes, n);
    entries_.push_back(Entry{chunks_.size() - 1, off, n, false});
    const TableStatus st = upload(entries_.size() - 1, stream);
    if (st != TableStatus::kOk) {
      entries_.pop_back();
      return st;
    }
    index_.emplace(h, entries_.size() - 1);
    c.used += need;
    *dev = c.dev + off;
    if (id) *id = entries_.size() - 1;
    return TableStatus::kOk;
  }

  // Issues the copy of table `id` on `stream` unless an earlier one, outside any capture, has been issued.
  TableStatus upload(size_t id, void* stream) {
    Entry& e = entries_[id];
    if (e.uploaded) return TableStatus::kOk;
    Chunk& c = chunks_[e.chunk];
    const bool recorded = !be_.may_alloc(stream);
    if (!be_.upload(c.dev + e.offset, c.host + e.offset, e.bytes, stream)) return TableStatus::kUploadFailed;
    e.uploaded = !recorded;
    return TableStatus::kOk;
  }
  bool uploaded(size_t id) const { return entries_[id].uploaded; }

  // Allocates the first chunk ahead of time (so that a first table seen during a
  // stream capture still finds room).  Returns false if the allocation failed.
  bool reserve_first_chunk() {
    return !chunks_.empty() || add_chunk();
  }

  size_t chunks() const { return chunks_.size(); }
  size_t tables() const { return index_.size(); }

 private:
  static constexpr size_t kAlign = 256;
  struct Chunk {
    uint8_t* dev;
    uint8_t* host;
    size_t used;
  };
  bool add_chunk() {
    chunks_.reserve(chunks_.size() + 1);   // first, so that an exception leaks no chunk
    Chunk c{};
    if (!be_.alloc(chunk_bytes_, &c.dev, &c.host)) return false;
    chunks_.push_back(c);
    return true;
  }
  struct Entry {
    size_t chunk, offset, bytes;
    bool uploaded;   // a copy has been issued outside a capture
  };
  // Four independent 8-byte lanes (multiply, fold the high half down), so that the multiplies overlap: a table of a
  // few hundred kilobytes is hashed at memory speed instead of one multiply latency per byte (960 units: 25 us of
  // 210 for the table of a step).  Equal hashes are told apart by comparing the contents.
  static uint64_t hash(const uint8_t* p, size_t n) {
    constexpr uint64_t kMul = 0x9E3779B97F4A7C15ull;
    uint64_t h[4] = {n, n ^ kMul, n + kMul, ~n};
    auto mix = [](uint64_t a, uint64_t v) {
      a = (a ^ v) * kMul;
      return a ^ (a >> 29);
    };
    size_t i = 0;
    for (; i + 32 <= n; i += 32)
      for (int k = 0; k < 4; ++k) {
        uint64_t v;
        memcpy(&v, p + i + 8 * k, 8);
        h[k] = mix(h[k], v);
      }
    for (; i < n; i += 8) {
      uint64_t v = 0;
      memcpy(&v, p + i, n - i < 8 ? n - i : 8);
      h[0] = mix(h[0], v);
    }
    return mix(mix(mix(h[0], h[1]), h[2]), h[3]);
  }

  Backend be_;
  size_t chunk_bytes_, limit_bytes_;
  std::vector<Chunk> chunks_;
  std::vector<Entry> entries_;
  std::unordered_multimap<uint64_t, size_t> index_;   // hash -> entry
};

}  // namespace hack
