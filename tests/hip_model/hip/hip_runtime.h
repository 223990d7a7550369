// A model of the HIP host calls that the C ABI makes, for a CPU build of it:
// device memory is host memory, a launch runs at once (or, in a capture, when
// the graph is launched), and what the host has waited for is tracked, so that
// releasing something that work in flight may still use is an error.  Handles
// are heap objects, so AddressSanitizer sees any use after their release.
#pragma once
#include <cstddef>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <vector>

#define __global__
#define __device__
#define __forceinline__ inline
struct int2 { int x, y; };
struct int4 { int x, y, z, w; };
struct float2 { float x, y; };
struct float4 { float x, y, z, w; };
inline int2 make_int2(int x, int y) { return {x, y}; }
inline int4 make_int4(int x, int y, int z, int w) { return {x, y, z, w}; }
struct dim3 {
  unsigned x;
  dim3(unsigned a = 1) : x(a) {}
};
enum hipError_t { hipSuccess, hipErrorInvalidValue, hipErrorOutOfMemory, hipErrorStreamCaptureUnsupported };
enum { hipMemcpyHostToDevice, hipMemcpyDeviceToHost, hipMemcpyDeviceToDevice };
enum { hipStreamNonBlocking = 1, hipEventDisableTiming = 2, hipHostMallocPortable = 1, hipHostMallocMapped = 2 };
enum hipStreamCaptureMode { hipStreamCaptureModeThreadLocal };
enum hipStreamCaptureStatus { hipStreamCaptureStatusNone, hipStreamCaptureStatusActive };

namespace model {
// every call holds it: the model is one object to all threads (its own
// allocations are not the tested code's)
inline std::recursive_mutex mu;
inline thread_local int inside = 0;
struct Lock {
  std::lock_guard<std::recursive_mutex> lk{mu};
  Lock() { ++inside; }
  ~Lock() { --inside; }
};
#define MODEL_LOCK model::Lock model_lock_
[[noreturn]] inline void fault(const std::string& what) {
  std::fprintf(stderr, "model: %s\n", what.c_str());
  std::abort();
}
using Clock = std::map<int, long>;  // stream number -> launches of it that are ordered before
inline void join(Clock& a, const Clock& b) {
  for (const auto& kv : b)
    if (a[kv.first] < kv.second) a[kv.first] = kv.second;
}
struct Capture;
struct Stream {
  int id;
  Clock after;          // what its next launch comes after (its own launches too)
  Capture* cap = nullptr;
};
struct Graph { std::vector<std::function<void()>> nodes; };
struct Capture { Graph* g; std::set<Stream*> streams; };
struct Exec { std::vector<std::function<void()>> nodes; Clock last; };
struct Event { Clock after; Capture* cap = nullptr; };
inline int next_id = 1;
inline Stream null_stream{0, {}, nullptr};
inline std::set<Stream*> live_streams;
inline Clock waited;    // what the host knows to be complete
inline long streams_made = 0, streams_live = 0, events_live = 0, execs_live = 0, host_mallocs = 0, host_frees = 0,
            destroys = 0, graph_calls = 0, memsets_captured = 0;
inline bool host_malloc_fails = false;

inline Stream* of(Stream* s) { return s ? s : &null_stream; }
inline bool done(const Clock& c) {
  for (const auto& kv : c) {
    auto it = waited.find(kv.first);
    if ((it == waited.end() ? 0 : it->second) < kv.second) return false;
  }
  return true;
}
template <class F> void launch(Stream* st, F fn) {
  MODEL_LOCK;
  Stream* s = of(st);
  if (s->cap) {
    s->cap->g->nodes.push_back(fn);
    return;
  }
  ++s->after[s->id];
  fn();
}
}  // namespace model

using hipStream_t = model::Stream*;
using hipEvent_t = model::Event*;
using hipGraph_t = model::Graph*;
using hipGraphExec_t = model::Exec*;

#define hipLaunchKernelGGL(kernel, grid, block, shmem, stream, ...) \
  model::launch(stream, [=] { kernel(__VA_ARGS__); })

inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
inline hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  MODEL_LOCK;
  *s = new model::Stream{model::next_id++, {}, nullptr};
  model::live_streams.insert(*s);
  ++model::streams_made;
  ++model::streams_live;
  return hipSuccess;
}
inline hipError_t hipStreamDestroy(hipStream_t s) {
  MODEL_LOCK;
  if (s->cap) model::fault("a capturing stream is destroyed");
  if (!model::done(s->after)) model::fault("a stream with work in flight is destroyed");
  model::live_streams.erase(s);
  --model::streams_live;
  ++model::destroys;
  delete s;
  return hipSuccess;
}
inline hipError_t hipStreamSynchronize(hipStream_t st) {
  MODEL_LOCK;
  hipStream_t s = model::of(st);
  if (s->cap) model::fault("a capturing stream is waited for");
  model::join(model::waited, s->after);
  return hipSuccess;
}
inline hipError_t hipStreamWaitEvent(hipStream_t st, hipEvent_t e, unsigned) {
  MODEL_LOCK;
  hipStream_t s = model::of(st);
  if (e->cap && !s->cap) {
    s->cap = e->cap;
    e->cap->streams.insert(s);
  }
  if (!s->cap) model::join(s->after, e->after);
  return hipSuccess;
}
inline hipError_t hipStreamIsCapturing(hipStream_t st, hipStreamCaptureStatus* out) {
  MODEL_LOCK;
  *out = model::of(st)->cap ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  MODEL_LOCK;
  *e = new model::Event();
  ++model::events_live;
  return hipSuccess;
}
inline hipError_t hipEventDestroy(hipEvent_t e) {
  MODEL_LOCK;
  if (!model::done(e->after)) model::fault("an event with work in flight is destroyed");
  --model::events_live;
  ++model::destroys;
  delete e;
  return hipSuccess;
}
inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t st) {
  MODEL_LOCK;
  hipStream_t s = model::of(st);
  e->cap = s->cap;
  if (!s->cap) e->after = s->after;
  return hipSuccess;
}
inline hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
  MODEL_LOCK;
  ++model::graph_calls;
  s->cap = new model::Capture{new model::Graph(), {s}};
  return hipSuccess;
}
inline hipError_t hipStreamEndCapture(hipStream_t s, hipGraph_t* g) {
  MODEL_LOCK;
  model::Capture* c = s->cap;
  *g = c->g;
  for (auto* x : c->streams) x->cap = nullptr;
  delete c;
  return hipSuccess;
}
inline hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t g, void*, char*, size_t) {
  MODEL_LOCK;
  *x = new model::Exec{g->nodes, {}};
  ++model::execs_live;
  return hipSuccess;
}
inline hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t st) {
  MODEL_LOCK;
  hipStream_t s = model::of(st);
  if (s->cap) return hipErrorStreamCaptureUnsupported;
  ++model::graph_calls;
  ++s->after[s->id];
  model::join(x->last, s->after);
  for (auto& n : x->nodes) n();
  return hipSuccess;
}
inline hipError_t hipGraphExecDestroy(hipGraphExec_t x) {
  MODEL_LOCK;
  if (!model::done(x->last)) model::fault("a graph in flight is destroyed");
  --model::execs_live;
  ++model::destroys;
  delete x;
  return hipSuccess;
}
inline hipError_t hipGraphDestroy(hipGraph_t g) {
  MODEL_LOCK;
  ++model::destroys;
  delete g;
  return hipSuccess;
}
inline hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  MODEL_LOCK;
  if (model::host_malloc_fails) return hipErrorOutOfMemory;
  *p = std::malloc(n);
  ++model::host_mallocs;
  return hipSuccess;
}
inline hipError_t hipHostFree(void* p) {
  MODEL_LOCK;
  ++model::host_frees;
  ++model::destroys;
  std::free(p);
  return hipSuccess;
}
inline hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, int, hipStream_t st) {
  model::launch(st, [=] { std::memcpy(d, s, n); });
  return hipSuccess;
}
inline hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t st) {
  {
    MODEL_LOCK;
    if (model::of(st)->cap) ++model::memsets_captured;
  }
  model::launch(st, [=] { std::memset(d, v, n); });
  return hipSuccess;
}
