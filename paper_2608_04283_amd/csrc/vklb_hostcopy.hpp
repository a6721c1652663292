// Large copies from device memory to pageable host memory.
//
// hipMemcpyAsync to pageable memory runs its copy engine, the page faults of a
// fresh destination and its host copy one after another, at 9-10 GB/s (the
// fields of Euler 2048^2, 134 MB: 14.5 ms). Here the device copies into a ring of
// pinned chunks while worker threads move finished ones on, so the three
// overlap: 56 GB/s of a pinned copy, 14 GB/s a thread into fresh pages, 4.7 ms for
// the same fields. Small copies, pinned destinations, and hosts that give no
// threads, events or pinned memory take the one call.
#pragma once

#include <hip/hip_runtime_api.h>
#include <string.h>

#include <algorithm>
#include <condition_variable>
#include <mutex>
#include <thread>
#include <vector>

namespace vklb {

// Not thread safe, as the solver that owns it. Its pinned memory (8 MiB) and
// events are made by the first copy that needs them and kept until release();
// worker threads end before a copy returns, and wait on a condition variable
// or an event, not in a loop.
class HostCopyRing {
 public:
  static constexpr size_t kChunk = size_t(1) << 20;
  static constexpr int kSlots = 8, kWorkers = 4;
  static constexpr size_t kAbove = size_t(8) << 20;  // smaller copies: one call

  // Copies in the order of `stream` (of `device`); the copy is complete when the
  // stream is. (It is not waited for here: a caller that reads more behind it
  // would wait twice, 20 us of the 65 that a small grid's moments take.)
  hipError_t copy(void* dst, const void* src, size_t bytes, hipStream_t stream, int device) {
    const int workers = std::min<int>(kWorkers, int(std::thread::hardware_concurrency()) - 1);
    if (bytes >= kAbove && workers >= 2 && !is_pinned(dst) && make()) {
      bool started = false;
      const hipError_t r = through_ring(dst, src, bytes, stream, device, workers, &started);
      if (started) return r;
    }
    return hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, stream);
  }

  void release() {
    for (hipEvent_t& e : ev_) {
      if (e) (void)hipEventDestroy(e);
      e = nullptr;
    }
    if (pin_) (void)hipHostFree(pin_);
    pin_ = nullptr;
  }

 private:
  static bool is_pinned(const void* p) {
    hipPointerAttribute_t at;
    if (hipPointerGetAttributes(&at, p) == hipSuccess) return at.type != hipMemoryTypeUnregistered;
    (void)hipGetLastError();
    return false;
  }

  // The ring, made once; a host that refuses any part of it is not asked again.
  bool make() {
    if (pin_) return true;
    if (refused_) return false;
    bool ok = true;
    for (hipEvent_t& e : ev_) ok = ok && hipEventCreateWithFlags(&e, hipEventDisableTiming) == hipSuccess;
    void* p = nullptr;
    ok = ok && hipHostMalloc(&p, kChunk * kSlots, hipHostMallocDefault) == hipSuccess;
    if (!ok) {
      (void)hipGetLastError();  // the one-call copy reports its own
      release();
      refused_ = true;
      return false;
    }
    pin_ = static_cast<char*>(p);
    return true;
  }

  // *started stays false if no thread was to be had: nothing was copied then.
  hipError_t through_ring(void* dst, const void* src, size_t bytes, hipStream_t stream, int device, int workers,
                          bool* started) {
    const long long chunks = (long long)((bytes + kChunk - 1) / kChunk);
    std::mutex mu;
    std::condition_variable to_move, to_issue;  // the workers wait for the one, the caller for the other
    long long issued = 0;          // chunks handed to the device
    long long moved[kSlots] = {};  // per slot: chunks moved on
    hipError_t failed = hipSuccess;
    bool stop = false;
    auto give_up = [&](hipError_t e) {
      std::lock_guard<std::mutex> lk(mu);
      if (failed == hipSuccess) failed = e;
      stop = true;
      to_move.notify_all();
      to_issue.notify_all();
    };
    auto work = [&](int w) {
      hipError_t e = hipSetDevice(device);
      for (long long i = w; i < chunks && e == hipSuccess; i += workers) {
        {
          std::unique_lock<std::mutex> lk(mu);
          to_move.wait(lk, [&] { return issued > i || stop; });
          if (stop) return;
        }
        const int slot = int(i % kSlots);
        if ((e = hipEventSynchronize(ev_[slot])) != hipSuccess) break;
        const size_t off = size_t(i) * kChunk;
        memcpy(static_cast<char*>(dst) + off, pin_ + size_t(slot) * kChunk, std::min(kChunk, bytes - off));
        std::lock_guard<std::mutex> lk(mu);
        ++moved[slot];
        to_issue.notify_one();
      }
      if (e != hipSuccess) give_up(e);
    };
    std::vector<std::thread> pool;
    try {
      pool.reserve(workers);
      for (int w = 0; w < workers; ++w) pool.emplace_back(work, w);
    } catch (...) {
      give_up(hipSuccess);
      for (std::thread& t : pool) t.join();
      return hipSuccess;
    }
    *started = true;
    // the work before the copy is waited for by this thread alone
    const hipError_t before = hipStreamSynchronize(stream);
    if (before != hipSuccess) give_up(before);
    for (long long i = 0; i < chunks; ++i) {
      const int slot = int(i % kSlots);
      {
        std::unique_lock<std::mutex> lk(mu);
        to_issue.wait(lk, [&] { return moved[slot] == i / kSlots || stop; });
        if (stop) break;
      }
      const size_t off = size_t(i) * kChunk;
      hipError_t e = hipMemcpyAsync(pin_ + size_t(slot) * kChunk, static_cast<const char*>(src) + off,
                                    std::min(kChunk, bytes - off), hipMemcpyDeviceToHost, stream);
      if (e == hipSuccess) e = hipEventRecord(ev_[slot], stream);
      if (e != hipSuccess) {
        give_up(e);
        break;
      }
      std::lock_guard<std::mutex> lk(mu);
      issued = i + 1;
      to_move.notify_all();
    }
    for (std::thread& t : pool) t.join();
    if (failed != hipSuccess) (void)hipStreamSynchronize(stream);  // no copy into the ring is left in flight
    return failed;
  }

  char* pin_ = nullptr;
  hipEvent_t ev_[kSlots] = {};
  bool refused_ = false;
};

}  // namespace vklb
