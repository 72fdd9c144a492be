// Runs the library's device memory code against the model of the HIP calls:
// no block may be used, or given back, while earlier work on it may be running.
// usage: model SCENARIO SEED; prints the number of faults.
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>

#include "../../paper_2411_16025_amd/csrc/workspace.hip"

// Host memory that runs out: inside the library, every n-th allocation fails.
static int g_fail_every = 0, g_news = 0, g_failed = 0;
void* operator new(size_t n) {
  if (g_fail_every && !model::own_depth() && ++g_news % g_fail_every == 0) {
    ++g_failed;
    throw std::bad_alloc();
  }
  return malloc(n ? n : 1);
}
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }

namespace gcn {
void set_error(const char*, ...) {}
static model::Stream g_side_stream{-1, {}};
hipStream_t side_stream(int) { return &g_side_stream; }
}  // namespace gcn

using namespace gcn;

// Streams whose addresses are taken again after they are destroyed.
struct Streams {
  std::vector<model::Stream> slot = std::vector<model::Stream>(3);
  std::vector<bool> live = std::vector<bool>(3, false);
  hipStream_t create(int i) {
    slot[i] = model::Stream{model::st().next_id++, {}};
    live[i] = true;
    return &slot[i];
  }
};

static void call(hipStream_t s, const std::vector<size_t>& sizes, bool scoped = true,
                 bool side = false, const void* graph = nullptr) {
  model::Own own;  // but for the calls of the library itself
  auto lib = [](auto f) {
    const int depth = model::own_depth();
    model::own_depth() = 0;
    f();
    model::own_depth() = depth;
  };
  alignas(CallScope) char buf[sizeof(CallScope)];
  CallScope* sc = scoped ? new (buf) CallScope(s) : nullptr;
  std::vector<void*> p(sizes.size());
  for (size_t i = 0; i < sizes.size(); ++i)
    lib([&] { tmalloc(&p[i], sizes[i], s, "block", i % 2 ? nullptr : graph); });
  for (void* q : p)
    if (q) model::use(q, s);
  if (side) {  // fork, a block of the side stream and one of the caller's, join
    hipStream_t s2 = side_stream(0);
    model::join(s2->clock, model::now(s));
    void* q = nullptr;
    lib([&] { tmalloc(&q, sizes[0], s2, "side block"); });
    if (q) model::use(q, s2);
    lib([&] { tfree(q, s2); });
    if (p[0]) model::use(p[0], s2);
    model::join(model::at(s).clock, s2->clock);
  }
  for (void* q : p) lib([&] { tfree(q, s); });
  if (sc) lib([&] { sc->~CallScope(); });
}

static size_t kib(int n) { return (size_t)n << 10; }

int main(int argc, char** argv) {
  model::State& st = model::st();
  st.total = kib(64 << 10);  // at most 16 MiB idle
  const char* what = argv[1];
  std::mt19937 rng(argc > 2 ? atoi(argv[2]) : 0);
  Streams S;
  if (!strcmp(what, "address")) {
    // a stream destroyed with its work pending; the first call at its address
    // finds no block of its size, the second one does
    call(S.create(0), {kib(64)});
    hipStream_t s = S.create(0);
    call(s, {kib(640)});
    call(s, {kib(64)});
  } else if (!strcmp(what, "address_unscoped")) {
    call(S.create(0), {kib(64)}, false);
    hipStream_t s = S.create(0);
    call(s, {kib(640)}, false);
    call(s, {kib(64)}, false);
  } else if (!strcmp(what, "graphs")) {
    // the default pool holds the partial rows of the graphs that ran, no more
    char g[2];
    graph_opened(0);
    graph_opened(0);
    call(nullptr, {kib(64), kib(128)});
    if (!st.pooled.empty()) ++st.faults;
    for (int k = 0; k < 2; ++k) {
      call(nullptr, {kib(64), kib(128)}, true, false, &g[k]);
      call(S.create(k), {kib(64), kib(128)}, true, false, &g[k]);
      call(&S.slot[k], {kib(64), kib(128)}, true, false, &g[k]);
    }
    if (st.pooled.size() != 4) ++st.faults;
    graph_closed(0, &g[0]);
    if (st.pooled.size() != 2) ++st.faults;
    graph_closed(0, &g[1]);
    if (!st.pooled.empty()) ++st.faults;
  } else if (!strcmp(what, "memory")) {
    // 40 MiB of memory, 12 of them idle: both kinds of allocation find room
    st.limit = kib(40 << 10);
    void *a = nullptr, *b = nullptr;
    call(nullptr, {kib(4 << 10), kib(8 << 10)});
    if (dmalloc(&a, kib(32 << 10), "array") != GCN_OK) ++st.faults;
    if (dmalloc(&b, kib(16 << 10), "array") != GCN_ENOMEM || b) ++st.faults;
    dfree(a);
    call(S.create(0), {kib(4 << 10), kib(8 << 10)});
    call(nullptr, {kib(32 << 10)});
    if (st.allocated > st.limit || st.allocs != 6) ++st.faults;
  } else if (!strcmp(what, "limits")) {
    // idle memory stays within the limit and the oldest blocks go first, whatever
    // stream their work is on
    graph_opened(0);
    for (int i = 0; i < 12; ++i) call(i % 2 ? nullptr : S.create(i / 2 % 3), {kib((2 + i) << 10)});
    if (st.allocated > st.total / 4 || st.allocated < kib(12 << 10)) ++st.faults;
    setenv("GCN_IDLE_MAX", "4194304", 1);
    graph_opened(0);
    call(nullptr, {kib(1 << 10), kib(4 << 10), kib(2 << 10)});
    if (st.allocated > kib(4 << 10)) ++st.faults;
    setenv("GCN_IDLE_MAX", "1048576", 1);
    char g[2];
    graph_closed(0, &g[0]);
    if (st.allocated <= kib(1 << 10)) ++st.faults;
    graph_closed(0, &g[1]);
    if (st.allocated > kib(1 << 10)) ++st.faults;
  } else if (!strcmp(what, "random") || !strcmp(what, "host_memory")) {
    if (!strcmp(what, "host_memory")) g_fail_every = 2 + rng() % 5;
    char graphs[3];
    char limit[32];
    snprintf(limit, sizeof(limit), "%zu", kib(64 << rng() % 8));
    setenv("GCN_IDLE_MAX", limit, 1);
    for (int k = 0; k < 3; ++k) graph_opened(0);
    for (int step = 0; step < 400; ++step) {
      model::Own own;
      const int i = rng() % 4;
      if (i < 3 && (!S.live[i] || rng() % 6 == 0)) S.create(i);
      hipStream_t s = i < 3 ? &S.slot[i] : nullptr;
      std::vector<size_t> sizes(1 + rng() % 4);
      for (size_t& b : sizes) b = kib(64 << rng() % 7);
      const int k = rng() % 4;
      call(s, sizes, rng() % 4 != 0, rng() % 3 == 0, k < 3 ? &graphs[k] : nullptr);
      if (k < 3 && rng() % 20 == 0) {  // freed, and another at its address
        graph_closed(0, &graphs[k]);
        if (rng() % 2) graph_opened(0);
      }
      if (rng() % 15 == 0) hipStreamSynchronize(s);
    }
  } else {
    return 2;
  }
  if (g_fail_every && !g_failed) ++st.faults;
  g_fail_every = 0;
  printf("faults %d allocs %d frees %d\n", st.faults, st.allocs, st.frees);
  return st.faults != 0;
}
