// Device memory of the library (workspace.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "../../include/gcnagg.h"

namespace gcn {

void set_error(const char* fmt, ...) __attribute__((format(printf, 1, 2)));
hipStream_t side_stream(int dev);

// ---- arrays that live as long as a graph -----------------------------------------
gcn_status dmalloc(void** p, size_t bytes, const char* what);
template <class T>
gcn_status dalloc(T** p, int64_t count, const char* what) {
  return dmalloc(reinterpret_cast<void**>(p), (size_t)(count > 0 ? count : 1) * sizeof(T), what);
}
void dfree(void* p);

// ---- temporaries ------------------------------------------------------------------
// Temporaries of the work enqueued on `stream`, kept for later calls on it, or
// for later calls on it with the same owner, a graph (workspace.hip).
gcn_status tmalloc(void** p, size_t bytes, hipStream_t stream, const char* what,
                   const void* owner = nullptr);
template <class T>
gcn_status talloc(T** p, int64_t count, hipStream_t stream, const char* what,
                  const void* owner = nullptr) {
  return tmalloc(reinterpret_cast<void**>(p), (size_t)(count > 0 ? count : 1) * sizeof(T), stream,
                 what, owner);
}
void tfree(void* p, hipStream_t stream);
// Whether work on the stream is being recorded (or the runtime cannot tell).
bool stream_capturing(hipStream_t stream);
// One per entry point that takes temporaries, from its start to its end (see
// workspace.hip); calls without one are ordered block by block.
struct CallScope {
  hipStream_t stream;
  CallScope* outer;
  int dev = 0;
  bool waited = false, released = false;
  explicit CallScope(void* stream);
  CallScope(const CallScope&) = delete;
  CallScope& operator=(const CallScope&) = delete;
  ~CallScope();
};
// Graphs alive per device: a graph's idle temporaries are given back with it, the
// others with the last one. graph_closed is called before the graph's address
// can be another's.
void graph_opened(int dev);
void graph_closed(int dev, const void* graph);

}  // namespace gcn
