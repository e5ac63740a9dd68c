// Host-only stand-in for the HIP runtime calls of runtime.cpp, and a C
// interface to Workspace on it: streams and events whose work ends when the
// test says so, and a device memory of a set capacity.  Pointers handed out
// are never dereferenced.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdint>
#include <map>
#include <mutex>
#include <set>
#include <thread>
#include <vector>

#include "runtime.h"

namespace {
struct Stream {
  int dev = 0;
  bool capturing = false;
  uint64_t issued = 0, finished = 0;  // work enqueued and completed
};
struct Event {
  Stream* on = nullptr;
  uint64_t at = 0;  // done once on->finished >= at
  bool done() const { return !on || on->finished >= at; }
};
struct State {
  std::recursive_mutex mu;
  std::vector<Stream*> streams;
  int device = 0;
  size_t capacity = SIZE_MAX, used = 0, peak = 0;
  uintptr_t next = 1 << 20;
  std::map<void*, size_t> live;
  int64_t mallocs = 0, frees = 0, cross_waits = 0, unsafe_calls = 0, host_waits = 0, trims = 0;
  bool any_capture = false;
};
State& S() {
  static State* s = new State();
  return *s;
}
thread_local hipStreamCaptureMode g_mode = hipStreamCaptureModeGlobal;
Stream g_null[8];
Stream* of(hipStream_t s) {
  if (s) return reinterpret_cast<Stream*>(s);
  return &g_null[S().device];
}
// a call that a capture in the global mode on any stream forbids
void unsafe() {
  if (S().any_capture && g_mode != hipStreamCaptureModeRelaxed) ++S().unsafe_calls;
}
hipError_t take(void** p, size_t bytes) {
  State& s = S();
  if (s.used > s.capacity || bytes > s.capacity - s.used) {
    *p = nullptr;
    return hipErrorOutOfMemory;
  }
  s.used += bytes;
  s.peak = std::max(s.peak, s.used);
  *p = reinterpret_cast<void*>(s.next);
  s.next += (bytes + 4095) / 4096 * 4096;
  s.live[*p] = bytes;
  ++s.mallocs;
  return hipSuccess;
}
}  // namespace

#define LOCK std::lock_guard<std::recursive_mutex> lk(S().mu)

extern "C" {
hipError_t hipGetDevice(int* d) { LOCK; *d = S().device; return hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t* d) { LOCK; *d = s ? of(s)->dev : S().device; return hipSuccess; }
hipError_t hipDeviceGetDefaultMemPool(hipMemPool_t* p, int) { *p = reinterpret_cast<hipMemPool_t>(8); return hipSuccess; }
hipError_t hipMemPoolSetAttribute(hipMemPool_t, hipMemPoolAttr, void*) { return hipSuccess; }
hipError_t hipMemPoolTrimTo(hipMemPool_t, size_t) { LOCK; ++S().trims; return hipSuccess; }
hipError_t hipMalloc(void** p, size_t bytes) { LOCK; unsafe(); return take(p, bytes); }
hipError_t hipMallocAsync(void** p, size_t bytes, hipStream_t) { LOCK; return take(p, bytes); }
hipError_t hipFreeAsync(void* p, hipStream_t) {
  LOCK;
  auto it = S().live.find(p);
  if (it == S().live.end()) return hipErrorInvalidValue;
  S().used -= it->second;
  S().live.erase(it);
  ++S().frees;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = reinterpret_cast<hipEvent_t>(new Event()); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t e) { delete reinterpret_cast<Event*>(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  LOCK;
  Event* ev = reinterpret_cast<Event*>(e);
  ev->on = of(s);
  ev->at = ev->on->issued;
  return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) { LOCK; unsafe(); return reinterpret_cast<Event*>(e)->done() ? hipSuccess : hipErrorNotReady; }
hipError_t hipEventSynchronize(hipEvent_t e) {
  LOCK;
  unsafe();
  Event* ev = reinterpret_cast<Event*>(e);
  if (!ev->done()) {
    ++S().host_waits;
    ev->on->finished = ev->at;
  }
  return hipSuccess;
}
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0.0f; return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  LOCK;
  Event* ev = reinterpret_cast<Event*>(e);
  if (!ev->done() && ev->on != of(s)) ++S().cross_waits;
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
  LOCK;
  *st = of(s)->capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) { LOCK; unsafe(); of(s)->finished = of(s)->issued; return hipSuccess; }
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode* m) { std::swap(*m, g_mode); return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "mock"; }

// --- the test's interface ---------------------------------------------------
void* mock_stream(int dev) {
  LOCK;
  Stream* s = new Stream();
  s->dev = dev;
  S().streams.push_back(s);
  return s;
}
void mock_set_device(int dev) { LOCK; S().device = dev; }
void mock_capacity(size_t bytes) { LOCK; S().capacity = bytes; }
void mock_capture(void* s, int on) { LOCK; of((hipStream_t)s)->capturing = on != 0; S().any_capture = on != 0; }
void mock_work(void* s) { LOCK; ++of((hipStream_t)s)->issued; }
void mock_finish(void* s) { LOCK; of((hipStream_t)s)->finished = of((hipStream_t)s)->issued; }
int64_t mock_count(int what) {
  LOCK;
  const State& s = S();
  const int64_t v[] = {s.mallocs, s.frees, s.cross_waits, s.unsafe_calls, s.host_waits, s.trims, (int64_t)s.used,
                       (int64_t)s.peak};
  return v[what];
}
void* ws_new(void* stream) { return new stag::Workspace((hipStream_t)stream); }
int ws_alloc(void* w, size_t bytes, void** p) { return (int)static_cast<stag::Workspace*>(w)->alloc_bytes(p, bytes); }
void ws_delete(void* w) { delete static_cast<stag::Workspace*>(w); }
int dev_alloc(size_t bytes, void** p) { return (int)stag::cached_alloc(p, bytes); }

// `threads` threads, each on a stream of its own, take and return workspaces
// `rounds` times; returns how often two held the same block at once.
int64_t mock_hammer(int threads, int rounds) {
  std::mutex mu;
  std::set<void*> held;
  std::atomic<int64_t> clashes{0};
  std::vector<std::thread> t;
  for (int k = 0; k < threads; ++k)
    t.emplace_back([&, k] {
      void* s = mock_stream(0);
      for (int r = 0; r < rounds; ++r) {
        void* p = nullptr;
        stag::Workspace ws((hipStream_t)s);
        if (ws.alloc_bytes(&p, (size_t)(40 + 8 * ((k + r) % 3)) << 20) != STAG_OK) continue;
        {
          std::lock_guard<std::mutex> lk(mu);
          if (!held.insert(p).second) ++clashes;
        }
        mock_work(s);
        if (r % 2) mock_finish(s);
        std::lock_guard<std::mutex> lk(mu);
        held.erase(p);
      }
    });
  for (auto& x : t) x.join();
  return clashes;
}
}  // extern "C"
