// The library's device memory (buffers of a call, cached checkpoints, workspaces, the refusal of an
// allocation) on a device that exists only here: a counted heap behind the few runtime calls that
// this code makes.  api.hip is compiled as host C++ and the rest of the library is left out (its
// symbols stay unresolved and are never called).  argv[1] names the check; prints "ok".
#include "../../paper_1603_00937_amd/csrc/api.hip"

#include <cstdio>
#include <cstdlib>
#include <new>
#include <set>

namespace {
size_t g_capacity = (size_t)1 << 40, g_used = 0, g_pooled = 0;
int g_mallocs = 0, g_frees = 0, g_events = 0, g_progress_trims = 0;
bool g_no_host_memory = false, g_running = false;  // running: work that nobody waited for
std::map<void*, size_t> g_live;

#define CHECK(c)                                                              \
  do {                                                                        \
    if (!(c)) {                                                               \
      std::fprintf(stderr, "check failed: %s (line %d)\n", #c, __LINE__);     \
      std::exit(1);                                                           \
    }                                                                         \
  } while (0)
}  // namespace

// host allocations fail on demand
void* operator new(std::size_t n) {
  if (g_no_host_memory) throw std::bad_alloc();
  void* p = std::malloc(n ? n : 1);
  if (!p) throw std::bad_alloc();
  return p;
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }

extern "C" {
hipError_t hipMallocAsync(void** p, size_t n, hipStream_t) {
  *p = nullptr;
  if (g_used + n > g_capacity) return hipErrorOutOfMemory;
  *p = std::malloc(16);
  g_live[*p] = n;
  g_used += n;
  ++g_mallocs;
  return hipSuccess;
}
hipError_t hipFreeAsync(void* p, hipStream_t) {  // the pool keeps it until it is trimmed
  CHECK(g_live.count(p) == 1);
  g_pooled += g_live[p];
  g_live.erase(p);
  std::free(p);
  ++g_frees;
  return hipSuccess;
}
hipError_t hipMemPoolTrimTo(hipMemPool_t, size_t) {
  g_used -= g_pooled;
  g_pooled = 0;
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceSynchronize(void) {
  g_running = false;
  return hipSuccess;
}
hipError_t hipStreamQuery(hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipDeviceGetDefaultMemPool(hipMemPool_t* p, int) {
  *p = nullptr;
  return hipSuccess;
}
hipError_t hipMemPoolSetAttribute(hipMemPool_t, hipMemPoolAttr, void*) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = reinterpret_cast<hipEvent_t>(std::malloc(16));
  ++g_events;
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
  std::free(e);
  --g_events;
  return hipSuccess;
}
}
namespace gbi {  // what gb_trim asks of the rest of the library
void ml_trim() {}
void progress_trim() { ++g_progress_trims; }
}  // namespace gbi

namespace {

constexpr size_t MiB = (size_t)1 << 20;
const hipStream_t kStream = reinterpret_cast<hipStream_t>((uintptr_t)64);

// What earlier calls left idle, however small, is back on the device before a call is refused.
int refusal() {
  CHECK(guarded([] {
          WsLease ws;
          for (int i = 0; i < 8; ++i) (void)ws->get_bytes(i, 20 * MiB, kStream);  // slabs below 32 MiB
        }) == GB_OK);
  const size_t slabs = g_used;
  CHECK(slabs >= 160 * MiB);
  g_capacity = 300 * MiB;
  CHECK(guarded([] {
          { DBuf<char> freed(30 * MiB, kStream); }  // put aside by this very call
          DBuf<char> large(280 * MiB, kStream);
          CHECK(large.get() != nullptr);
        }) == GB_OK);
  CHECK(guarded([] { DBuf<char> too_large(301 * MiB, kStream); }) == GB_ENOMEM);
  return 0;
}

// The same through a registered allocator.
size_t g_hook_used = 0;
std::map<void*, size_t> g_hook_live;
void* hook_alloc(size_t n, void*, void*) {
  if (g_hook_used + n > 300 * MiB) return nullptr;
  void* p = std::malloc(16);
  g_hook_live[p] = n;
  g_hook_used += n;
  return p;
}
void hook_free(void* p, void*, void*) {
  g_hook_used -= g_hook_live[p];
  g_hook_live.erase(p);
  std::free(p);
}
int hook_refusal() {
  CHECK(gb_set_allocator(hook_alloc, hook_free, nullptr) == GB_OK);
  CHECK(guarded([] {
          WsLease ws;
          for (int i = 0; i < 4; ++i) (void)ws->get_bytes(i, 50 * MiB, kStream);
        }) == GB_OK);
  CHECK(g_hook_used >= 200 * MiB);
  CHECK(guarded([] {
          DBuf<char> large(280 * MiB, kStream);
          CHECK(large.get() != nullptr);
        }) == GB_OK);
  CHECK(guarded([] { DBuf<char> too_large(301 * MiB, kStream); }) == GB_ENOMEM);
  CHECK(g_hook_used == 0);
  return 0;
}

// A checkpoint whose list has no memory for its entry is freed, once, and the list stays usable.
int no_host_memory() {
  {
    std::vector<CachedBuf> held;
    for (int i = 0; i < 40; ++i) held.emplace_back(40 * MiB, kStream);
    g_no_host_memory = true;
    held.clear();
    g_no_host_memory = false;
  }
  CHECK(g_frees > 0);  // the list had no room for all of them
  const int kept = 40 - g_frees, mallocs = g_mallocs;
  {
    std::vector<CachedBuf> again;
    for (int i = 0; i < 40; ++i) again.emplace_back(40 * MiB, kStream);
    CHECK(g_mallocs == mallocs + 40 - kept);
  }
  cached_trim();
  CHECK(g_live.empty());
  return 0;
}

// The process may end with idle checkpoints (nothing is freed then: the runtime may be gone).
int idle_at_exit() {
  const int frees = g_frees;
  {
    std::vector<CachedBuf> held;
    for (int i = 0; i < 5; ++i) held.emplace_back(40 * MiB, kStream);
  }
  CHECK(g_frees == frees);
  return 0;
}

// Full lists follow the sizes in use.
int full_lists() {
  auto call = [](int count, size_t each) {
    const int before = g_mallocs;
    CHECK(guarded([&] {
            std::vector<DBuf<char>> b;
            for (int i = 0; i < count; ++i) b.emplace_back(each, kStream);
          }) == GB_OK);
    return g_mallocs - before;
  };
  CHECK(call(8, 32 * MiB) == 8);  // all that the list holds
  CHECK(call(8, 32 * MiB) == 0);
  CHECK(call(20, MiB) == 20);
  CHECK(call(20, MiB) == 0);  // twenty of these and seven of the others
  CHECK(call(8, 32 * MiB) == 1);
  auto checkpoints = [](int count, size_t each) {
    const int before = g_mallocs;
    std::vector<CachedBuf> b;
    for (int i = 0; i < count; ++i) b.emplace_back(each, kStream);
    return g_mallocs - before;
  };
  CHECK(checkpoints(22, 2048 * MiB) == 22);
  CHECK(checkpoints(22, 2048 * MiB) == 0);
  CHECK(checkpoints(30, 200 * MiB) == 30);
  CHECK(checkpoints(30, 200 * MiB) == 0);
  const size_t idle = g_used - g_pooled;
  CHECK(idle <= (48 << 10) * MiB + 256 * MiB);
  CHECK(checkpoints(1, (60 << 10) * MiB) == 1);  // larger than the list: freed, and nothing else is
  CHECK(g_used - g_pooled == idle);
  return 0;
}

// What a failed call leaves running is waited for before another call can take its buffers.
int failed_call() {
  void* held = nullptr;
  CHECK(guarded([&] {
          WsLease ws;
          held = ws->get_bytes(0, 64 * MiB, kStream);
        }) == GB_OK);
  CHECK(guarded([&] {
          WsLease ws;
          CHECK(ws->get_bytes(0, 64 * MiB, kStream) == held);
          g_running = true;
          fail(GB_EHIP, "a call fails in between");
        }) == GB_EHIP);
  CHECK(!g_running);
  CHECK(guarded([&] {
          CachedBuf b(64 * MiB, kStream);
          g_running = true;
          fail(GB_EHIP, "a call fails in between");
        }) == GB_EHIP);
  CHECK(!g_running);
  g_running = true;  // another stream's: no business of a call that succeeds
  CHECK(guarded([&] {
          WsLease ws;
          CachedBuf b(64 * MiB, kStream);
        }) == GB_OK);
  CHECK(g_running);
  return 0;
}

// gb_trim gives everything back that calls have kept, the events of their timings among it.
int trim() {
  {
    Timer a, b;
    WsLease ws;
    (void)ws->get_bytes(0, 64 * MiB, kStream);
    CachedBuf c(64 * MiB, kStream);
  }
  CHECK(guarded([] { DBuf<char> small(MiB, kStream); }) == GB_OK);
  CHECK(g_events == 4 && g_live.size() == 3);
  {
    Timer again;
    CHECK(g_events == 4);
  }
  CHECK(gb_trim() == GB_OK);
  CHECK(g_events == 0 && g_progress_trims == 1 && g_live.empty());
  Timer after;
  CHECK(g_events == 2);
  return 0;
}

}  // namespace

int main(int argc, char** argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  int rc = 2;
  if (what == "refusal") rc = refusal();
  if (what == "hook_refusal") rc = hook_refusal();
  if (what == "no_host_memory") rc = no_host_memory();
  if (what == "idle_at_exit") rc = idle_at_exit();
  if (what == "full_lists") rc = full_lists();
  if (what == "failed_call") rc = failed_call();
  if (what == "trim") rc = trim();
  if (rc == 0) std::printf("ok\n");
  return rc;
}
