// Host runtime: last-error storage, stream-ordered workspace, small
// host-only entry points of the C ABI.
#include "runtime.h"

#include <cstring>

#include <atomic>
#include <cmath>
#include <map>
#include <mutex>
#include <vector>

namespace stag {

namespace {
thread_local std::string g_last_error;
}

stag_status fail(stag_status st, const char* fmt, ...) {
  char buf[1024];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  g_last_error = buf;
  return st;
}

void clear_error() { g_last_error.clear(); }

stag_status check_launch(const char* what) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(STAG_E_DEVICE, "launch of %s failed: %s", what, hipGetErrorString(e));
  return STAG_OK;
}

namespace {
std::mutex g_pool_mu;
bool g_pool_done[64] = {};
}  // namespace

void keep_pool_memory() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return;
  std::lock_guard<std::mutex> lk(g_pool_mu);
  if (g_pool_done[dev]) return;
  g_pool_done[dev] = true;
  hipMemPool_t pool = nullptr;
  if (hipDeviceGetDefaultMemPool(&pool, dev) == hipSuccess && pool) {
    uint64_t thr = UINT64_MAX;
    (void)hipMemPoolSetAttribute(pool, hipMemPoolAttrReleaseThreshold, &thr);
  }
  (void)hipGetLastError();
}

namespace {
std::mutex g_cache_mu;
std::map<int, std::multimap<size_t, void*>> g_cache;
}  // namespace

// Gives the idle workspace blocks of device dev back to the system (see
// BlockCache); st: a stream of that device.  False if there were none.
static bool release_idle(int dev, hipStream_t st);

stag_status cached_alloc(void** p, size_t bytes) {
  *p = nullptr;
  int dev = 0;
  (void)hipGetDevice(&dev);
  {
    std::lock_guard<std::mutex> lk(g_cache_mu);
    auto& c = g_cache[dev];
    auto it = c.lower_bound(bytes);
    if (it != c.end() && it->first <= 2 * bytes) {
      *p = it->second;
      c.erase(it);
      return STAG_OK;
    }
  }
  hipError_t e = hipMalloc(p, bytes);
  if (e == hipErrorOutOfMemory && release_idle(dev, nullptr)) {
    (void)hipGetLastError();
    e = hipMalloc(p, bytes);
  }
  if (e != hipSuccess) {
    *p = nullptr;
    (void)hipGetLastError();
    return fail(e == hipErrorOutOfMemory ? STAG_E_NOMEM : STAG_E_DEVICE, "device allocation of %zu bytes: %s", bytes,
                hipGetErrorString(e));
  }
  return STAG_OK;
}

void cached_free(void* p, size_t bytes) {
  if (!p) return;
  int dev = 0;
  (void)hipGetDevice(&dev);
  std::lock_guard<std::mutex> lk(g_cache_mu);
  g_cache[dev].emplace(bytes, p);
}

// Runs a query of an event's state, which a capture in the global mode on
// any other stream would otherwise forbid (and be ended by).
class RelaxedCapture {
 public:
  RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode_); }
  ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode_); }

 private:
  hipStreamCaptureMode mode_ = hipStreamCaptureModeRelaxed;
};

// Blocks returned by workspaces, per device, for the next ones.  A pool
// allocation cost 40 us and a stream-ordered free 150 us of host time on
// average (1 ms at times) on the caller's critical path, more than all the
// launches of a small call.  A block carries an event, recorded on the stream
// that used it last when it is returned, which is when the host has enqueued
// the call, long before the device has run it.  So a stream is given a block
// that it used last itself, or one whose work is done; a block that another
// stream still works on would tie the two streams together (four calls of
// 100,000 points and 300 queries took 291 us on four streams and 229 on one;
// on four streams now 174).
// At most kMaxIdle bytes per device lie idle (the blocks returned longest ago
// make room for a new one, unless they are still at work) and no block above
// kMaxBlock is kept; the rest goes back to the pool, and when an allocation of any size
// fails, a workspace's or an index's, everything idle goes back to the system
// before it is tried again.  Requests on a capturing stream bypass the cache
// both ways: a graph owns its memory.
class BlockCache {
 public:
  static constexpr size_t kMaxIdle = (size_t)2 << 30, kMaxBlock = (size_t)1 << 30;

  // An idle block of at least `bytes` and at most twice as many: the smallest
  // that st used last, else the smallest whose work is done.
  bool take(int dev, size_t bytes, hipStream_t st, Workspace::Block* out) {
    {
      std::lock_guard<std::mutex> lk(mu_);
      auto& d = dev_[dev];
      const auto lo = d.idle.lower_bound(bytes), hi = d.idle.upper_bound(2 * bytes);
      auto it = lo;
      while (it != hi && it->second.last != st) ++it;
      if (it == hi && lo != hi) {
        RelaxedCapture relaxed;
        for (it = lo; it != hi && hipEventQuery(it->second.ev) != hipSuccess; ++it) (void)hipGetLastError();
      }
      if (it == hi) return false;
      *out = it->second;
      d.idle.erase(it);
      d.idle_bytes -= out->bytes;
    }
    // (also for its own stream: the handle may be that of a newer stream)
    if (hipStreamWaitEvent(st, out->ev, 0) == hipSuccess) return true;
    (void)hipGetLastError();
    RelaxedCapture relaxed;
    give_back(*out, st);
    return false;
  }

  void put(Workspace::Block b, hipStream_t st) {
    b.last = st;
    if (b.ev == nullptr || hipEventRecord(b.ev, st) != hipSuccess) {
      (void)hipFreeAsync(b.p, st);
      drop_event(b.ev);
      return;
    }
    std::vector<Workspace::Block> out;
    {
      std::lock_guard<std::mutex> lk(mu_);
      auto& d = dev_[b.dev];
      while (d.idle_bytes + b.bytes > kMaxIdle && evict_oldest(&d, &out)) {
      }
      if (d.idle_bytes + b.bytes <= kMaxIdle) {
        b.returned = ++returns_;
        d.idle.emplace(b.bytes, b);
        d.idle_bytes += b.bytes;
      } else {
        out.push_back(b);
      }
    }
    for (const Workspace::Block& o : out) {
      (void)hipFreeAsync(o.p, st);
      drop_event(o.ev);
    }
  }

  // Returns every idle block of the device to the system once its work is done.
  bool trim(int dev, hipStream_t st) {
    std::multimap<size_t, Workspace::Block> idle;
    {
      std::lock_guard<std::mutex> lk(mu_);
      idle.swap(dev_[dev].idle);
      dev_[dev].idle_bytes = 0;
    }
    if (idle.empty()) return false;
    RelaxedCapture relaxed;
    for (auto& kv : idle) give_back(kv.second, st);
    (void)hipStreamSynchronize(st);
    hipMemPool_t pool = nullptr;
    if (hipDeviceGetDefaultMemPool(&pool, dev) == hipSuccess && pool) (void)hipMemPoolTrimTo(pool, 0);
    (void)hipGetLastError();
    return true;
  }

  static void drop_event(hipEvent_t ev) {
    if (ev) (void)hipEventDestroy(ev);
  }

 private:
  // Frees a block on stream st after its last use.
  void give_back(const Workspace::Block& b, hipStream_t st) {
    (void)hipEventSynchronize(b.ev);
    (void)hipFreeAsync(b.p, st);
    drop_event(b.ev);
    (void)hipGetLastError();
  }

  struct Device {
    std::multimap<size_t, Workspace::Block> idle;
    size_t idle_bytes = 0;
  };

  // Takes the idle block that was returned first among those whose work is
  // done; false if there is none.
  bool evict_oldest(Device* d, std::vector<Workspace::Block>* out) {
    RelaxedCapture relaxed;
    auto oldest = d->idle.end();
    for (auto it = d->idle.begin(); it != d->idle.end(); ++it) {
      if (oldest != d->idle.end() && oldest->second.returned < it->second.returned) continue;
      if (hipEventQuery(it->second.ev) == hipSuccess) oldest = it;
      else (void)hipGetLastError();
    }
    if (oldest == d->idle.end()) return false;
    out->push_back(oldest->second);
    d->idle_bytes -= oldest->second.bytes;
    d->idle.erase(oldest);
    return true;
  }

  std::mutex mu_;
  std::map<int, Device> dev_;
  uint64_t returns_ = 0;
};

namespace {
// Never destroyed: its blocks go with the process, after the runtime may have.
BlockCache& block_cache() {
  static BlockCache* c = new BlockCache();
  return *c;
}
}  // namespace

static bool release_idle(int dev, hipStream_t st) { return block_cache().trim(dev, st); }

Workspace::~Workspace() {
  for (const Block& b : blocks_) block_cache().put(b, stream_);
}

std::vector<void*> Workspace::release() {
  std::vector<void*> v;
  for (const Block& b : blocks_) {
    v.push_back(b.p);
    BlockCache::drop_event(b.ev);
  }
  blocks_.clear();
  cur_ = nullptr;
  used_ = cap_ = 0;
  return v;
}

stag_status Workspace::raw_alloc(void** p, size_t bytes) {
  *p = nullptr;
  keep_pool_memory();
  Block b = {nullptr, bytes, 0, nullptr, stream_, 0};
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  // the stream's device, which need not be the current one
  const bool cached = hipStreamGetDevice(stream_, &b.dev) == hipSuccess &&
                      hipStreamIsCapturing(stream_, &cap) == hipSuccess && cap == hipStreamCaptureStatusNone;
  if (cached && bytes <= BlockCache::kMaxBlock) {
    if (block_cache().take(b.dev, bytes, stream_, &b)) {
      blocks_.push_back(b);
      *p = b.p;
      return STAG_OK;
    }
    if (hipEventCreateWithFlags(&b.ev, hipEventDisableTiming) != hipSuccess) b.ev = nullptr;
  }
  (void)hipGetLastError();
  hipError_t e = hipMallocAsync(&b.p, bytes, stream_);
  if (e == hipErrorOutOfMemory && cached && release_idle(b.dev, stream_)) {
    (void)hipGetLastError();
    e = hipMallocAsync(&b.p, bytes, stream_);
  }
  if (e != hipSuccess) {
    (void)hipGetLastError();
    BlockCache::drop_event(b.ev);
    return fail(e == hipErrorOutOfMemory ? STAG_E_NOMEM : STAG_E_DEVICE, "workspace allocation of %zu bytes: %s",
                bytes, hipGetErrorString(e));
  }
  blocks_.push_back(b);
  *p = b.p;
  return STAG_OK;
}

stag_status Workspace::alloc_bytes(void** p, size_t bytes) {
  *p = nullptr;
  bytes = (bytes + 255) / 256 * 256;
  if (bytes == 0) bytes = 256;
  if (mode_ == kCount) {
    used_ += bytes;
    return STAG_OK;
  }
  if (mode_ == kArena) {
    if (used_ + bytes > cap_)
      return fail(STAG_E_NOMEM, "scratch arena exhausted: %zu + %zu bytes > %zu", used_, bytes, cap_);
    *p = cur_ + used_;
    used_ += bytes;
    return STAG_OK;
  }
  if (bytes >= kSmallBytes) return raw_alloc(p, bytes);
  if (cur_ == nullptr || used_ + bytes > cap_) {
    void* blk = nullptr;
    STAG_TRY(raw_alloc(&blk, kBlockBytes));
    cur_ = static_cast<char*>(blk);
    used_ = 0;
    cap_ = kBlockBytes;
  }
  *p = cur_ + used_;
  used_ += bytes;
  return STAG_OK;
}

namespace {
struct TimerRec {
  const char* name;
  hipEvent_t a, b;
};
std::mutex g_timer_mu;
std::vector<TimerRec> g_timer_recs;
std::atomic<int> g_timing{0};
}  // namespace

bool timing_enabled() { return g_timing.load(std::memory_order_relaxed) != 0; }

ScopedTimer::ScopedTimer(const char* name, hipStream_t s) : name_(name), stream_(s) {
  if (!timing_enabled()) return;
  if (hipEventCreate(&start_) != hipSuccess || hipEventRecord(start_, stream_) != hipSuccess) {
    if (start_) (void)hipEventDestroy(start_);
    start_ = nullptr;
    (void)hipGetLastError();
  }
}

ScopedTimer::~ScopedTimer() {
  if (!start_) return;
  hipEvent_t end = nullptr;
  if (hipEventCreate(&end) != hipSuccess || hipEventRecord(end, stream_) != hipSuccess) {
    if (end) (void)hipEventDestroy(end);
    (void)hipEventDestroy(start_);
    (void)hipGetLastError();
    return;
  }
  std::lock_guard<std::mutex> lk(g_timer_mu);
  g_timer_recs.push_back({name_, start_, end});
}

}  // namespace stag

extern "C" {

void stag_timing_enable(int32_t on) { stag::g_timing.store(on ? 1 : 0); }

// Waits for every recorded launch, then writes "name count total_ms\n" lines
// (one per kernel name, sorted) into buf and clears the records.  Returns
// the number of bytes the full report needs (excluding the terminator).
size_t stag_timing_report(char* buf, size_t len) {
  std::vector<stag::TimerRec> recs;
  {
    std::lock_guard<std::mutex> lk(stag::g_timer_mu);
    recs.swap(stag::g_timer_recs);
  }
  std::map<std::string, std::pair<long, double>> agg;
  for (auto& r : recs) {
    float ms = 0.0f;
    if (hipEventSynchronize(r.b) == hipSuccess && hipEventElapsedTime(&ms, r.a, r.b) == hipSuccess) {
      auto& e = agg[r.name];
      e.first += 1;
      e.second += ms;
    }
    (void)hipGetLastError();
    (void)hipEventDestroy(r.a);
    (void)hipEventDestroy(r.b);
  }
  std::string out;
  char line[256];
  for (auto& kv : agg) {
    snprintf(line, sizeof(line), "%s %ld %.6f\n", kv.first.c_str(), kv.second.first, kv.second.second);
    out += line;
  }
  if (buf && len > 0) {
    size_t k = out.size() < len - 1 ? out.size() : len - 1;
    memcpy(buf, out.data(), k);
    buf[k] = 0;
  }
  return out.size();
}

const char* stag_last_error(void) { return stag::g_last_error.c_str(); }

const char* stag_version(void) { return "0.1.0 gfx950"; }

// Closed form of the single-function collision probability (Sec. "Random
// Projection"), written without the overflowing factor exp(8/c^2), boosted
// over K concatenated functions and L tables (Sec. "Boosting the
// Probability").
double stag_e2lsh_collision_probability(double c, int32_t K, int32_t L) {
  if (!(c >= 0.0) || K < 1 || L < 1) return NAN;
  double p = 1.0;
  if (c > 0.0) {
    const double inv_sqrt_2pi = 0.39894228040143267794;  // 1/sqrt(2 pi)
    p = std::erf(2.0 * std::sqrt(2.0) / c) - 0.5 * inv_sqrt_2pi * c * (-std::expm1(-8.0 / (c * c)));
  }
  const double pk = std::pow(p, (double)K);
  if (pk >= 1.0) return 1.0;
  return -std::expm1((double)L * std::log1p(-pk));
}

}  // extern "C"
