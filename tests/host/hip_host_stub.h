// Stand-in for the HIP runtime and the kernels, so that csrc/hack_api.cpp runs on the host without a device: "device"
// memory is malloc'ed and filled with a pattern no table holds, copies and launches on a stream that is being captured
// are collected in a graph instead of carried out, and a launch looks at the tables it was given when it is carried out.
// Include it once, before hack_api.cpp.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <new>
#include <string>
#include <vector>

#include "../../paper_2504_09261_amd/csrc/hack_internal.h"

namespace stub {

// Allocations of the code under test that succeed before the next one fails (-1: all do); the stand-in's own do not count.
inline long allocations_left = -1;
inline bool allocation_failed = false;
inline int quiet = 0;
struct Quiet {
  Quiet() { ++quiet; }
  ~Quiet() { --quiet; }
};
inline void* allocate(size_t n) {
  if (!quiet && allocations_left >= 0 && allocations_left-- == 0) {
    allocation_failed = true;
    return nullptr;
  }
  return malloc(n ? n : 1);
}

struct Graph {
  std::vector<std::function<void()>> nodes;
  int copies = 0;
};
inline Graph* capture = nullptr;              // graph being recorded, of stream capture_stream
inline void* capture_stream = nullptr;
inline std::vector<int> waves;                // ... of a work-group of each key-split attention launch
inline std::vector<std::string> launches;     // names of the launches carried out
inline int bad_launches = 0;                  // ... over tables that were never written
inline int lds_bytes = 256;                   // of a work-group: no whole steps in one launch unless a check asks for more
struct WholeLaunch { hack::WholeStep step; std::vector<hack::UnitDesc> descs; };
inline std::vector<WholeLaunch> whole_launches;   // launches that do a whole step, with the descriptors they were given
inline int copies = 0;                        // asynchronous copies carried out
inline size_t copied = 0;                     // bytes of the last one
inline std::map<void*, size_t> device_memory; // live allocations

struct ShortUnits { int n_units, n_append; };
inline std::vector<ShortUnits> moving_launches;   // launches that score, select and move the rows of a step

// Whether n bytes from p on lie in one live allocation.
inline bool owned(const void* p, size_t n) {
  const char* at = static_cast<const char*>(p);
  auto it = device_memory.upper_bound(const_cast<void*>(p));
  if (it == device_memory.begin()) return false;
  --it;
  const char* base = static_cast<const char*>(it->first);
  return at >= base && at + n <= base + it->second;
}

inline bool captured(void* stream) { return capture != nullptr && stream == capture_stream; }
inline void submit(void* stream, std::function<void()> f) {
  if (captured(stream)) capture->nodes.push_back(std::move(f));
  else f();
}
inline void begin_capture(Graph* g, void* stream) { capture = g; capture_stream = stream; }
inline void end_capture() { capture = nullptr; }
inline void replay(const Graph& g) {
  for (const auto& f : g.nodes) f();
}

// A launch over n descriptors: all of them must have been written.
inline void launch(const char* name, void* stream, const hack::UnitDesc* descs, const int32_t* list, int n) {
  Quiet q;
  submit(stream, [=] {
    launches.push_back(name);
    for (int i = 0; i < n; ++i) {
      const int at = list ? list[i] : i;
      const bool ok = at >= 0 && at < 65536 && descs[at].unit >= 0 && descs[at].unit < 65536 && descs[at].len_in >= 0 && descs[at].n_out >= 0;
      if (!ok) {
        ++bad_launches;
        return;
      }
    }
  });
}
inline void launch_items(const char* name, void* stream, const hack::AttnItem* items, int n) {
  Quiet q;
  submit(stream, [=] {
    launches.push_back(name);
    for (int i = 0; i < n; ++i)
      if (items[i].desc < -1 || items[i].desc > 65536 || (items[i].desc >= 0 && (items[i].n_out < 1 || items[i].unit < 0))) {
        ++bad_launches;
        return;
      }
  });
}

}  // namespace stub

void* operator new(size_t n) {
  if (void* p = stub::allocate(n)) return p;
  throw std::bad_alloc();
}
void* operator new(size_t n, const std::nothrow_t&) noexcept { return stub::allocate(n); }
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }
void operator delete(void* p, const std::nothrow_t&) noexcept { free(p); }

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
  stub::Quiet q;
  *p = malloc(n);
  if (!*p) return hipErrorOutOfMemory;
  memset(*p, 0xEE, n);
  stub::device_memory[*p] = n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  stub::device_memory.erase(p);
  free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return (*p = malloc(n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipHostFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemset(void* d, int v, size_t n) { memset(d, v, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t stream) {
  stub::Quiet q;
  if (stub::captured(stream)) ++stub::capture->copies;
  stub::submit(stream, [=] { ++stub::copies; stub::copied = n; memcpy(d, s, n); });
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
  *st = stub::captured(s) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeMaxSharedMemoryPerBlock ? stub::lds_bytes : 256;
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stub"; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = nullptr; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = nullptr; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
}

namespace hack {

int score_max_groups() { return 64; }
// as the kernels' registers and LDS have it on a device of 256 compute units
int score_fused_capacity(int head_dim, int item_keys) {
  return 1024 * (head_dim == 128 ? 2 : item_keys == 32 ? 5 : item_keys == 64 ? 4 : item_keys == 96 || item_keys == 192 ? 3 : 2);
}
int attn_stream_slots(int) { return 512; }
int attn_split_q_tile_rows() { return 32; }
int attn_f32_q_tile_rows(int n_units, int N_k) { return n_units * ((N_k + 15) / 16) <= kAttnF32SmallItems ? 16 : 32; }
bool use_score_select(int, int n_units, int max_t_in) { return max_t_in <= 256 || (max_t_in <= 1024 && n_units >= 128); }
hipError_t score_static_setup(int) { return hipSuccess; }

void launch_move(hipStream_t s, int, int, const UnitDesc* d, int n, int, CachePtrs, CachePtrs, const void*, const void*, int, int,
                 const int32_t*, int64_t) { stub::launch("move", s, d, nullptr, n); }
void launch_select(hipStream_t s, const UnitDesc* d, int n, int, const float*, int64_t, int32_t*, int64_t, int32_t*) {
  stub::launch("select", s, d, nullptr, n);
}
void launch_score_fused(hipStream_t s, int, int, bool two_pass, const ScoreItem* items, int n, const void*, const int32_t*, int, int, float,
                        const void*, const void*, unsigned long long*, int, unsigned*, float*, int64_t, int*, int, const unsigned*, int) {
  stub::Quiet q;
  stub::submit(s, [=] {
    stub::launches.push_back(two_pass ? "score_two_pass" : "score_fused");
    for (int i = 0; i < n; ++i)
      if (items[i].t_in < 1 || items[i].n_groups < 1 || items[i].n_groups > 64) { ++stub::bad_launches; return; }
  });
}
void launch_score_select(hipStream_t s, int, const UnitDesc* d, int n, int, const void*, const int32_t*, int, int, float,
                         const void*, const void*, int32_t*, int64_t, int32_t*, int*) { stub::launch("score_select", s, d, nullptr, n); }
// The move of such a launch is recorded as the launch that it stands for.
void launch_score_select_move(hipStream_t s, int, const UnitDesc* d, int n, const UnitDesc* app, int n_app, int max_t, const void*, const int32_t*,
                              int, int, float, CachePtrs, const void*, const void*, int, int32_t*, int64_t, int*) {
  stub::launch("score_select", s, d, nullptr, n);
  stub::launch("move", s, app, nullptr, n_app);
  stub::Quiet q;
  stub::submit(s, [=] {
    stub::moving_launches.push_back({n, n_app});
    for (int i = 0; i < n; ++i) if (d[i].mode != MOVE_GATHER || d[i].len_in + d[i].n_new > max_t || d[i].n_new < 1) ++stub::bad_launches;
    for (int i = 0; i < n_app; ++i) if (app[i].mode != MOVE_APPEND) ++stub::bad_launches;
  });
}
void launch_score_select_f32(hipStream_t s, int, const UnitDesc* d, int n, int max_t, const void*, const int32_t*, int, int, float, const void*,
                             const void*, double* logits, double* stats, unsigned* counters, int32_t*, int64_t, int32_t*) {
  const size_t groups = (size_t)score_f32_groups(n, max_t, 64);
  if (!stub::owned(logits, groups * kF32GroupLogits * sizeof(double)) || !stub::owned(stats, groups * kMaxObs * 2 * sizeof(double)) ||
      !stub::owned(counters, 2 * n * sizeof(unsigned)) || logits == stats)
    ++stub::bad_launches;
  stub::launch("score_select_f32", s, d, nullptr, n);
  stub::Quiet q;
  stub::submit(s, [=] {
    for (int i = 0; i < n; ++i) if (d[i].mode != MOVE_GATHER || d[i].len_in + d[i].n_new > max_t || d[i].n_new < 1) ++stub::bad_launches;
  });
}
void launch_score_f32(hipStream_t s, int, const UnitDesc* d, int n, int, const void*, const int32_t*, int, int, float,
                      const void*, const void*, double*, float*, int64_t) { stub::launch("score_f32", s, d, nullptr, n); }
hipError_t launch_score_static(hipStream_t, int, int, const StaticScorePlan&, const void*, int, int, float, const void*, const void*, float*,
                               int64_t, int*) { return hipSuccess; }
void launch_attn(hipStream_t s, int, const UnitDesc*, const AttnItem* it, int n, const void*, const void*, const void*, int, float, void*, int kernel) {
  stub::launch_items(kernel == kAttnHalves ? "attn_halves" : "attn", s, it, n);
}
void launch_attn_stream(hipStream_t s, int, const UnitDesc*, const AttnSeg*, const int32_t* begin, int n, const void*, const void*,
                        const void*, int, float, void*, float*, float*, unsigned*) {
  stub::Quiet q;
  stub::submit(s, [=] {
    stub::launches.push_back("attn_stream");
    for (int i = 0; i < n; ++i) if (begin[i] < 0 || begin[i + 1] < begin[i]) { ++stub::bad_launches; return; }
  });
}
void launch_attn_split(hipStream_t s, int, const UnitDesc*, const AttnItem* it, int n, const void*, const void*, const void*, const void*,
                       const void*, void*, void*, int32_t*, int, bool append, bool eight, int, float, void*) {
  stub::launch_items(append ? "attn_split_append" : "attn_split", s, it, n);
  stub::Quiet q;
  stub::submit(s, [=] { stub::waves.push_back(eight ? 8 : 4); });
}
void launch_attn_split_gather(hipStream_t s, int, const UnitDesc* descs, const AttnItem* it, int n, const GatherArgs& g, const void*,
                              const void*, const void*, int, float, void*) {
  stub::launch_items("attn_split_gather", s, it, n);
  stub::Quiet q;
  const bool eight = g.eight;
  stub::submit(s, [=] { stub::waves.push_back(eight ? 8 : 4); });
}
void launch_step_units(hipStream_t s, int, const UnitDesc* descs, WholeStep w, const void*, const CachePtrs&, const void*, const void*, int, int, float,
                       void*, int32_t*, int64_t) {
  stub::launch(w.moved ? "attend_whole" : "step_whole", s, descs, nullptr, w.n_units);
  stub::Quiet q;
  stub::submit(s, [=] { stub::whole_launches.push_back({w, std::vector<UnitDesc>(descs, descs + w.n_units)}); });
}
void launch_attn_f32(hipStream_t s, int, const AttnItem* it, int n, int, const void*, const void*, const void*, const void*, const void*,
                     void*, void*, int32_t*, int, int fuse, int, float, void*) {
  stub::launch_items(fuse ? "attn_f32_append" : "attn_f32", s, it, n);
}
void launch_attn_f32_gather(hipStream_t s, int, const UnitDesc*, const AttnItem* it, int n, int, const GatherArgs&, const void*, const void*,
                            const void*, int, float, void*) { stub::launch_items("attn_f32_gather", s, it, n); }
void launch_merge(hipStream_t s, int, const UnitDesc* d, const int32_t* l, int n, int, int, const void*, const void*, const void*, const void*,
                  int, const int32_t*, int64_t, void*, void*, int32_t*, float*, float*, int64_t) { stub::launch("merge", s, d, l, n); }
void launch_head_variance(hipStream_t s, int, const UnitDesc* d, int n, int, const void*, const void*, int, float, float*, double*) {
  stub::launch("head_variance", s, d, nullptr, n);
}

}  // namespace hack
