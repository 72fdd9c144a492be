// A model of the HIP calls that the library's device memory code makes, for a
// build on the CPU: streams, events and allocations with vector clocks.
#pragma once

#include <cstddef>
#include <cstdint>
#include <map>
#include <vector>

enum hipError_t { hipSuccess = 0, hipErrorOutOfMemory = 2, hipErrorUnknown = 999 };
enum hipStreamCaptureStatus { hipStreamCaptureStatusNone = 0 };
enum hipMemAllocationType { hipMemAllocationTypePinned = 1 };
enum hipMemLocationType { hipMemLocationTypeDevice = 1 };
struct hipMemLocation {
  hipMemLocationType type;
  int id;
};
struct hipMemPoolProps {
  hipMemAllocationType allocType;
  int handleTypes;
  hipMemLocation location;
};
typedef struct hipMemPool* hipMemPool_t;
constexpr unsigned hipEventDisableTiming = 2;

namespace model {

// What has happened before: work items of each stream that are ordered before.
typedef std::map<int, int> Clock;
inline void join(Clock& a, const Clock& b) {
  for (auto& kv : b)
    if (a[kv.first] < kv.second) a[kv.first] = kv.second;
}
inline bool before(const Clock& a, const Clock& b) {
  for (auto& kv : a) {
    auto it = b.find(kv.first);
    if (it == b.end() || it->second < kv.second) return false;
  }
  return true;
}

struct Stream {
  int id;  // of this incarnation; the address may have had others
  Clock clock;
};
struct Event {
  Clock clock;
};

struct State {
  int next_id = 1;
  Stream null_stream{0, {}};
  Clock host;                       // what the host has waited for
  Clock all;                        // all work
  std::map<char*, size_t> mem;      // live allocations
  std::map<char*, size_t> pooled;   // those of the default pool
  std::map<char*, Clock> last_use;  // of the work that touched each
  size_t allocated = 0, total = 0, limit = 0;
  int allocs = 0, frees = 0, faults = 0;
  uintptr_t next = 1 << 20;
};
inline State& st() {
  static State s;
  return s;
}
// The model's own bookkeeping, which does not fail when host memory runs out.
inline int& own_depth() {
  static int d = 0;
  return d;
}
struct Own {
  Own() { ++own_depth(); }
  ~Own() { --own_depth(); }
};

}  // namespace model

typedef model::Stream* hipStream_t;
typedef model::Event* hipEvent_t;
#define hipStreamLegacy ((hipStream_t)1)
#define hipStreamPerThread ((hipStream_t)2)

namespace model {

inline Stream& at(hipStream_t s) { return s ? *s : st().null_stream; }
inline Clock now(hipStream_t s) {
  Clock c = at(s).clock;
  join(c, st().host);
  return c;
}
// A kernel on the stream that reads and writes the block.
inline void use(void* p, hipStream_t s) {
  Own own;
  Stream& t = at(s);
  join(t.clock, st().host);
  Clock& last = st().last_use[(char*)p];
  if (!before(last, t.clock)) ++st().faults;  // runs beside the work before it
  t.clock[t.id] += 1;
  last = t.clock;
  join(st().all, t.clock);
}
inline hipError_t alloc(void** p, size_t n) {
  Own own;
  State& s = st();
  if (s.limit && s.allocated + n > s.limit) {
    *p = nullptr;
    return hipErrorOutOfMemory;
  }
  char* q = (char*)s.next;
  s.next += n + 4096;
  s.mem[q] = n;
  s.allocated += n;
  ++s.allocs;
  *p = q;
  return hipSuccess;
}
inline hipError_t release(void* p) {
  Own own;
  State& s = st();
  auto it = s.mem.find((char*)p);
  if (it == s.mem.end()) {
    ++s.faults;  // not allocated, or released twice
    return hipErrorUnknown;
  }
  s.allocated -= it->second;
  s.last_use.erase(it->first);
  s.pooled.erase(it->first);
  s.mem.erase(it);
  ++s.frees;
  return hipSuccess;
}

}  // namespace model

inline hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
inline hipError_t hipGetLastError() { return hipSuccess; }
inline const char* hipGetErrorString(hipError_t) { return "model"; }
inline hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* c) {
  *c = hipStreamCaptureStatusNone;
  return hipSuccess;
}
inline hipError_t hipMemGetInfo(size_t* f, size_t* t) {
  *t = model::st().total;
  *f = *t - model::st().allocated;
  return hipSuccess;
}
inline hipError_t hipMalloc(void** p, size_t n) { return model::alloc(p, n); }
inline hipError_t hipMallocAsync(void** p, size_t n, hipStream_t) {
  model::Own own;
  const hipError_t e = model::alloc(p, n);
  if (e == hipSuccess) model::st().pooled[(char*)*p] = n;
  return e;
}
inline hipError_t hipMemPoolCreate(hipMemPool_t* p, const hipMemPoolProps*) {
  *p = (hipMemPool_t)1;
  return hipSuccess;
}
inline hipError_t hipMallocFromPoolAsync(void** p, size_t n, hipMemPool_t, hipStream_t) {
  return model::alloc(p, n);
}
inline hipError_t hipFree(void* p) {  // waits for the device
  model::Own own;
  model::join(model::st().host, model::st().all);
  return model::release(p);
}
inline hipError_t hipFreeAsync(void* p, hipStream_t s) {
  model::Own own;
  if (!model::before(model::st().last_use[(char*)p], model::now(s))) ++model::st().faults;
  return model::release(p);
}
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  model::Own own;
  *e = new model::Event();
  return hipSuccess;
}
inline hipError_t hipEventDestroy(hipEvent_t e) {
  model::Own own;
  delete e;
  return hipSuccess;
}
inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  model::Own own;
  e->clock = model::now(s);
  return hipSuccess;
}
inline hipError_t hipEventSynchronize(hipEvent_t e) {
  model::Own own;
  model::join(model::st().host, e->clock);
  return hipSuccess;
}
inline hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  model::Own own;
  model::join(model::at(s).clock, e->clock);
  return hipSuccess;
}
inline hipError_t hipStreamSynchronize(hipStream_t s) {
  model::Own own;
  model::join(model::st().host, model::at(s).clock);
  return hipSuccess;
}
