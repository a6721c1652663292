// HostCopyRing (csrc/vklb_hostcopy.hpp) over a stand-in for the few HIP calls it
// makes, on the CPU: what is copied, how often the host is asked for the ring,
// and that a failure of any call ends the copy with nothing left behind. The
// stand-in's copies run when an event or the stream is waited for, in order.
#include <stdio.h>
#include <stdlib.h>

#include <atomic>
#include <deque>
#include <functional>

#include "vklb_hostcopy.hpp"

namespace {
std::mutex g_mu;
std::deque<std::function<void()>> g_queue;  // the stream's work
hipError_t g_last = hipSuccess;             // HIP's last error
struct Event {
  long long pos = 0;
};
long long g_pushed = 0, g_run = 0, g_events = 0, g_buffers = 0;  // live objects: events, pinned buffers
int g_copies = 0, g_event_calls = 0, g_malloc_calls = 0;
// the call of each kind that fails (-1: none), counted from 0
int fail_event = -1, fail_malloc = -1, fail_copy = -1, fail_wait = -1, fail_record = -1;
std::atomic<int> n_wait{0};
int n_record = 0;

hipError_t err(hipError_t e) { return g_last = e; }
void run_to(long long pos) {
  std::lock_guard<std::mutex> lk(g_mu);
  while (g_run < pos) {
    g_queue.front()();
    g_queue.pop_front();
    ++g_run;
  }
}
}  // namespace

extern "C" {
hipError_t hipGetLastError() {
  const hipError_t e = g_last;
  g_last = hipSuccess;
  return e;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void*) {
  a->type = hipMemoryTypeUnregistered;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  if (g_event_calls++ == fail_event) return err(hipErrorOutOfMemory);
  *e = reinterpret_cast<hipEvent_t>(new Event);
  ++g_events;
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
  delete reinterpret_cast<Event*>(e);
  --g_events;
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  if (g_malloc_calls++ == fail_malloc) return err(hipErrorOutOfMemory);
  *p = malloc(n);
  ++g_buffers;
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  free(p);
  --g_buffers;
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  if (g_copies++ == fail_copy) return err(hipErrorInvalidValue);
  std::lock_guard<std::mutex> lk(g_mu);
  g_queue.push_back([=] { memcpy(d, s, n); });
  ++g_pushed;
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
  if (n_record++ == fail_record) return err(hipErrorInvalidValue);
  std::lock_guard<std::mutex> lk(g_mu);
  reinterpret_cast<Event*>(e)->pos = g_pushed;
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
  if (n_wait++ == fail_wait) return hipErrorUnknown;
  long long pos;
  {
    std::lock_guard<std::mutex> lk(g_mu);
    pos = reinterpret_cast<Event*>(e)->pos;
  }
  run_to(pos);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) {
  long long pos;
  {
    std::lock_guard<std::mutex> lk(g_mu);
    pos = g_pushed;
  }
  run_to(pos);
  return hipSuccess;
}
}

#define CHECK(c)                                                      \
  do {                                                                \
    if (!(c)) {                                                       \
      printf("line %d: %s does not hold (%s)\n", __LINE__, #c, what); \
      exit(1);                                                        \
    }                                                                 \
  } while (0)

static void reset() {
  g_last = hipSuccess;
  g_copies = g_event_calls = g_malloc_calls = n_record = 0;
  n_wait = 0;
  fail_event = fail_malloc = fail_copy = fail_wait = fail_record = -1;
}

// Copies `bytes` through `ring`; a successful copy has every byte.
static hipError_t copy(vklb::HostCopyRing& ring, size_t bytes, const char* what) {
  std::vector<unsigned char> src(bytes), dst(bytes + 16, 0xee);
  unsigned x = unsigned(bytes) * 2654435761u + 1;
  for (auto& c : src) c = (unsigned char)((x = x * 1664525u + 1013904223u) >> 24);
  const hipError_t e = ring.copy(dst.data(), src.data(), bytes, nullptr, 0);
  if (bytes >= vklb::HostCopyRing::kAbove && g_buffers) CHECK(g_queue.empty());
  (void)hipStreamSynchronize(nullptr);
  CHECK(g_queue.empty());  // nothing in flight, whatever happened
  if (e == hipSuccess) CHECK(memcmp(src.data(), dst.data(), bytes) == 0);
  for (int i = 0; i < 16; ++i) CHECK(dst[bytes + i] == 0xee);
  return e;
}

int main() {
  using R = vklb::HostCopyRing;
  const char* what = "sizes";
  {
    R ring;
    reset();
    for (size_t b : {size_t(1), R::kAbove - 1}) CHECK(copy(ring, b, what) == hipSuccess);
    CHECK(g_event_calls == 0 && g_malloc_calls == 0 && g_copies == 2);
    for (size_t b : {R::kAbove, R::kAbove + 1, 9 * R::kChunk, 24 * R::kChunk - 1, 41 * R::kChunk + 4097})
      CHECK(copy(ring, b, what) == hipSuccess);
    CHECK(g_event_calls == R::kSlots && g_malloc_calls == 1);  // made once
    CHECK(g_events == R::kSlots && g_buffers == 1);
    ring.release();
    CHECK(g_events == 0 && g_buffers == 0);
  }
  // A host that refuses an event or the pinned memory: the copy is made by the
  // one call, HIP's last error is clear, and the host is not asked again.
  for (int k = 0; k <= R::kSlots; ++k) {
    what = k < R::kSlots ? "event refused" : "pinned memory refused";
    R ring;
    reset();
    (k < R::kSlots ? fail_event : fail_malloc) = k < R::kSlots ? k : 0;
    CHECK(copy(ring, R::kAbove + 5, what) == hipSuccess);
    CHECK(hipGetLastError() == hipSuccess);
    CHECK(g_events == 0 && g_buffers == 0);
    const int events = g_event_calls, mallocs = g_malloc_calls;
    CHECK(copy(ring, R::kAbove + 6, what) == hipSuccess);
    CHECK(g_event_calls == events && g_malloc_calls == mallocs && g_copies == 2);
    ring.release();
  }
  // Any call that fails on the way ends the copy with its error; the next works.
  for (int k : {0, 9, 23}) {
    for (int* f : {&fail_copy, &fail_record, &fail_wait}) {
      what = f == &fail_copy ? "copy fails" : f == &fail_record ? "record fails" : "wait fails";
      R ring;
      reset();
      *f = k;
      CHECK(copy(ring, 24 * R::kChunk, what) != hipSuccess);
      reset();
      CHECK(copy(ring, 24 * R::kChunk, what) == hipSuccess);
      ring.release();
    }
  }
  CHECK(g_events == 0 && g_buffers == 0);
  printf("ok\n");
  return 0;
}
