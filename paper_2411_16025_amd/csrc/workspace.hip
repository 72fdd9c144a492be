// Device memory: the graphs' arrays and the calls' temporaries.

#include <algorithm>
#include <atomic>
#include <cstdlib>
#include <iterator>
#include <list>
#include <map>
#include <mutex>
#include <new>
#include <unordered_map>
#include <utility>

#include "workspace.h"

namespace gcn {

void dfree(void* p) {
  if (p) (void)hipFree(p);
}

// Temporaries. hipFreeAsync waits for the work enqueued on its stream (20
// buffers of 64 MiB written by 20 kernels: 698 us with hipMallocAsync and
// hipFreeAsync around them, 363 us with kept buffers), so a call that released
// its temporaries with it ran in step with the host. Released blocks are
// kept here instead, per device and stream: the next call on that stream takes
// them without waiting, since its work is ordered behind the work that used them.
//  * A caller's stream may be destroyed with its work pending and a new one
//    created at its address. So a call that released blocks ends with an event
//    on its stream, and a later call at that address waits for it before it takes
//    a block and before it records the event again: nothing to wait for on the
//    stream itself, and a real dependency on another. (A call that finds no block
//    of its size waits too, or the event would no longer cover the work of the
//    stream before.) The NULL stream and the library's own are not destroyed and
//    need no event.
//  * A block goes to another stream only through the driver.
//  * The partial rows of an aggregation come from the device's default memory pool
//    and belong to their graph: they are kept for its next aggregation and given
//    back with it. All other kept blocks come from a pool of the library's own, so
//    that the default pool holds nothing of a graph that was only built (what
//    calls that promise to take nothing from it are measured by).
//  * While a stream is being captured, its temporaries are nodes of the graph
//    (hipMallocAsync / hipFreeAsync), as a graph may be replayed on any stream.
//  * At most a quarter of the device's memory is kept idle (or GCN_IDLE_MAX bytes,
//    if that is less when a graph is built), the oldest blocks going first; all of
//    it is given back when an allocation fails, and all but kKeepIdle when the
//    last graph on the device is freed.
namespace {

struct Block {
  void* ptr;
  size_t bytes;
  int dev;
  hipStream_t stream;
  const void* owner;  // the graph it belongs to, or null
};

hipMemPool_t g_pool[64] = {};  // set once per device, under g_cache_mu
std::mutex g_cache_mu;
std::list<Block> g_idle;                  // oldest first
std::unordered_map<void*, Block> g_live;  // handed out
std::map<std::pair<int, hipStream_t>, hipEvent_t> g_last_use;  // callers' streams
size_t g_idle_bytes[64] = {};
size_t g_idle_max[64] = {};
int g_graphs[64] = {};
constexpr size_t kKeepIdle = size_t(256) << 20;

thread_local CallScope* t_scope = nullptr;

// The bytes that may be kept idle on the current device, dev.
size_t idle_max(int dev) {
  static std::atomic<size_t> memory[64] = {};
  size_t free_b = 0, total = memory[dev];
  if (!total) {
    if (hipMemGetInfo(&free_b, &total) != hipSuccess) {
      (void)hipGetLastError();
      total = size_t(64) << 30;
    }
    memory[dev] = total;
  }
  const char* s = std::getenv("GCN_IDLE_MAX");
  const long long v = s && *s ? std::atoll(s) : 0;
  return v > 0 && (size_t)v < total / 4 ? (size_t)v : total / 4;
}

// A block from the driver, of the library's own pool or (pool = false) of the
// default one.
hipError_t driver_alloc(void** p, size_t bytes, int dev, hipStream_t stream, bool pool) {
  hipMemPool_t own = nullptr;
  if (pool) {
    std::lock_guard<std::mutex> lk(g_cache_mu);
    if (!g_pool[dev]) {
      hipMemPoolProps props = {};
      props.allocType = hipMemAllocationTypePinned;
      props.location.type = hipMemLocationTypeDevice;
      props.location.id = dev;
      if (hipMemPoolCreate(&g_pool[dev], &props) != hipSuccess) {
        (void)hipGetLastError();
        g_pool[dev] = nullptr;
      }
    }
    own = g_pool[dev];
  }
  return own ? hipMallocFromPoolAsync(p, bytes, own, stream) : hipMallocAsync(p, bytes, stream);
}

// The current device; false where blocks cannot be kept (a capturing stream,
// the special handles, a stream the runtime refuses).
bool may_keep(hipStream_t stream, int* dev) {
  if (hipGetDevice(dev) != hipSuccess || *dev < 0 || *dev >= 64) return false;
  if (!stream) return true;
  if (stream == hipStreamPerThread || stream == hipStreamLegacy) return false;
  return !stream_capturing(stream);
}

}  // namespace

bool stream_capturing(hipStream_t stream) {
  if (!stream || stream == hipStreamLegacy) return false;
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(stream, &cs) != hipSuccess) {
    (void)hipGetLastError();
    return true;
  }
  return cs != hipStreamCaptureStatusNone;
}

namespace {

bool callers_stream(int dev, hipStream_t stream) { return stream && stream != side_stream(dev); }

// Give a block back (the caller holds no lock). Where the stream is the
// caller's own, it orders the release; otherwise hipFree waits for the device.
void give_back(const Block& b, hipStream_t stream) {
  if (!stream && !b.stream)
    (void)hipFreeAsync(b.ptr, stream);
  else
    (void)hipFree(b.ptr);
}

// The lists never throw (the caller holds the lock): a block that cannot be
// noted as handed out, or as idle, goes back to the driver when it is released.
void track(const Block& b) {
  try {
    g_live.emplace(b.ptr, b);
  } catch (const std::bad_alloc&) {
  }
}

bool push_idle(const Block& b) {
  try {
    g_idle.push_back(b);
    return true;
  } catch (const std::bad_alloc&) {
    return false;
  }
}

// Idle blocks of a device, oldest first, until at most keep bytes are left.
std::list<Block> take_idle(int dev, size_t keep) {
  std::list<Block> out;
  std::lock_guard<std::mutex> lk(g_cache_mu);
  for (auto it = g_idle.begin(); it != g_idle.end() && g_idle_bytes[dev] > keep;) {
    auto next = std::next(it);
    if (it->dev == dev) {
      g_idle_bytes[dev] -= it->bytes;
      out.splice(out.end(), g_idle, it);
    }
    it = next;
  }
  return out;
}

// The stream waits for the event at its address (the caller holds the lock).
void wait_last_use(int dev, hipStream_t stream) {
  auto ev = g_last_use.find({dev, stream});
  if (ev == g_last_use.end() || !ev->second) return;
  if (hipStreamWaitEvent(stream, ev->second, 0) != hipSuccess) {
    (void)hipGetLastError();
    (void)hipEventSynchronize(ev->second);
  }
}

// The event that ends the last call on a caller's stream that released blocks
// (waited: the call has waited for the one before).
void mark_last_use(int dev, hipStream_t stream, bool waited) {
  std::lock_guard<std::mutex> lk(g_cache_mu);
  if (!waited) wait_last_use(dev, stream);
  hipEvent_t ev = nullptr;
  try {
    hipEvent_t& e = g_last_use[{dev, stream}];
    if (!e && hipEventCreateWithFlags(&e, hipEventDisableTiming) != hipSuccess) e = nullptr;
    ev = e;
  } catch (const std::bad_alloc&) {
  }
  if (!ev || hipEventRecord(ev, stream) != hipSuccess) {
    (void)hipGetLastError();
    (void)hipStreamSynchronize(stream);  // without an event the work is waited for
  }
}

}  // namespace

gcn_status dmalloc(void** p, size_t bytes, const char* what) {
  *p = nullptr;
  hipError_t e = hipMalloc(p, bytes);
  int dev = 0;
  if (e != hipSuccess && hipGetDevice(&dev) == hipSuccess && dev >= 0 && dev < 64) {
    (void)hipGetLastError();
    for (const Block& b : take_idle(dev, 0)) (void)hipFree(b.ptr);
    e = hipMalloc(p, bytes);
  }
  if (e != hipSuccess) {
    *p = nullptr;
    (void)hipGetLastError();
    set_error("device allocation of %zu bytes for %s failed: %s", bytes, what,
              hipGetErrorString(e));
    return GCN_ENOMEM;
  }
  return GCN_OK;
}

CallScope::CallScope(void* s) : stream((hipStream_t)s), outer(t_scope) { t_scope = this; }

CallScope::~CallScope() {
  t_scope = outer;
  if (released) mark_last_use(dev, stream, waited);
}

gcn_status tmalloc(void** p, size_t bytes, hipStream_t stream, const char* what,
                   const void* owner) {
  *p = nullptr;
  int dev = 0;
  const bool keep = may_keep(stream, &dev);
  if (keep) {
    // whole 64 KiB (2 MiB above 1 MiB), so that nearly equal sizes share blocks
    const size_t unit = bytes > (size_t(1) << 20) ? size_t(2) << 20 : size_t(64) << 10;
    bytes = (bytes + unit - 1) / unit * unit;
    std::lock_guard<std::mutex> lk(g_cache_mu);
    auto best = g_idle.end();
    for (auto it = g_idle.begin(); it != g_idle.end(); ++it)
      if (it->dev == dev && it->stream == stream && it->owner == owner && it->bytes >= bytes &&
          it->bytes <= bytes + bytes / 4 && (best == g_idle.end() || it->bytes < best->bytes))
        best = it;
    if (best != g_idle.end()) {
      CallScope* sc = t_scope && t_scope->stream == stream ? t_scope : nullptr;
      if (callers_stream(dev, stream) && !(sc && sc->waited)) {
        wait_last_use(dev, stream);
        if (sc) sc->waited = true;
      }
      *p = best->ptr;
      g_idle_bytes[dev] -= best->bytes;
      track(*best);
      g_idle.erase(best);
      return GCN_OK;
    }
  }
  hipError_t e = driver_alloc(p, bytes, dev, stream, keep && !owner);
  if (e != hipSuccess && keep) {
    (void)hipGetLastError();
    for (const Block& b : take_idle(dev, 0)) give_back(b, stream);
    (void)hipStreamSynchronize(stream);
    e = driver_alloc(p, bytes, dev, stream, !owner);
  }
  if (e != hipSuccess) {
    *p = nullptr;
    (void)hipGetLastError();
    set_error("stream-ordered allocation of %zu bytes for %s failed: %s", bytes, what,
              hipGetErrorString(e));
    return GCN_ENOMEM;
  }
  if (keep) {
    std::lock_guard<std::mutex> lk(g_cache_mu);
    track(Block{*p, bytes, dev, stream, owner});
  }
  return GCN_OK;
}

void tfree(void* p, hipStream_t stream) {
  if (!p) return;
  int dev = 0;
  const bool keep = may_keep(stream, &dev);
  size_t over = 0;
  bool kept = false, mark = false;
  {
    std::lock_guard<std::mutex> lk(g_cache_mu);
    auto it = g_live.find(p);
    if (it != g_live.end()) {
      if (keep && it->second.dev == dev && it->second.stream == stream) kept = push_idle(it->second);
      if (kept) {
        if (callers_stream(dev, stream)) {
          if (t_scope && t_scope->stream == stream) {
            t_scope->released = true;
            t_scope->dev = dev;
          } else {
            mark = true;
          }
        }
        g_idle_bytes[dev] += it->second.bytes;
        if (!g_idle_max[dev]) g_idle_max[dev] = idle_max(dev);
        if (g_idle_bytes[dev] > g_idle_max[dev]) over = g_idle_max[dev];
      }
      g_live.erase(it);
    }
  }
  if (!kept) {
    (void)hipFreeAsync(p, stream);
    return;
  }
  if (mark) mark_last_use(dev, stream, false);
  if (over)
    for (const Block& b : take_idle(dev, over)) give_back(b, stream);
}

void graph_opened(int dev) {
  if (dev < 0 || dev >= 64) return;
  const size_t max = idle_max(dev);
  std::lock_guard<std::mutex> lk(g_cache_mu);
  ++g_graphs[dev];
  g_idle_max[dev] = max;
}

void graph_closed(int dev, const void* graph) {
  std::list<Block> own;
  {
    std::lock_guard<std::mutex> lk(g_cache_mu);
    if (dev < 0 || dev >= 64) return;
    for (auto it = g_idle.begin(); it != g_idle.end();) {
      auto next = std::next(it);
      if (it->owner == graph) {
        g_idle_bytes[dev] -= it->bytes;
        own.splice(own.end(), g_idle, it);
      }
      it = next;
    }
    --g_graphs[dev];
  }
  for (const Block& b : own) (void)hipFree(b.ptr);
  {
    std::lock_guard<std::mutex> lk(g_cache_mu);
    if (g_graphs[dev] > 0) return;
  }
  int cur = -1;
  if (hipGetDevice(&cur) != hipSuccess || cur != dev) return;
  for (const Block& b : take_idle(dev, std::min(kKeepIdle, idle_max(dev)))) (void)hipFree(b.ptr);
}

}  // namespace gcn
