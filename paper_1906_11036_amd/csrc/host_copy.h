// Device-to-host copies into ordinary (pageable) memory.
//
// The runtime's own copy moves such memory through a pinned buffer with one
// thread: about 10 GB/s.  Large copies go through two pinned chunks here, each
// filled by the copy engine while a few threads empty the other: a pass that
// reads 2^24 binary64 values back 22.9 -> 14.3 ms.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <string.h>

#include <atomic>
#include <thread>

namespace dugks {

// Owned by one context and used by one call at a time, as the context is; the
// pinned memory is taken at the first large copy and freed with the context.
class HostCopy {
 public:
  HostCopy() = default;
  HostCopy(const HostCopy&) = delete;
  HostCopy& operator=(const HostCopy&) = delete;
  ~HostCopy() {
    for (int b = 0; b < 2; ++b) {
      if (pin_[b]) (void)hipHostFree(pin_[b]);
      if (ev_[b]) (void)hipEventDestroy(ev_[b]);
    }
  }

  // n bytes from device memory to dst, after the work enqueued on s; complete
  // when it returns.
  hipError_t out(void* dst, const void* src, size_t n, hipStream_t s) {
    if (n < kLeast || !pageable(dst) || !ready(s)) return plain(dst, src, n, s);
    const size_t chunks = (n + kChunk - 1) / kChunk;
    std::atomic<size_t> filled{0}, emptied{0};   // chunks filled; slices emptied
    std::atomic<bool> stop{false};
    auto slice = [&](size_t i, int w) {
      const size_t at = i * kChunk, len = n - at < kChunk ? n - at : kChunk;
      const size_t lo = len * w / kThreads, hi = len * (w + 1) / kThreads;
      memcpy((char*)dst + at + lo, (const char*)pin_[i & 1] + lo, hi - lo);
      emptied.fetch_add(1, std::memory_order_release);
    };
    auto work = [&](int w) {
      for (size_t i = 0; i < chunks; ++i) {
        while (filled.load(std::memory_order_acquire) <= i) {
          if (stop.load(std::memory_order_relaxed)) return;
          std::this_thread::yield();
        }
        slice(i, w);
      }
    };
    auto fill = [&](size_t i) {
      const size_t at = i * kChunk, len = n - at < kChunk ? n - at : kChunk;
      hipError_t e = hipMemcpyAsync(pin_[i & 1], (const char*)src + at, len, hipMemcpyDeviceToHost, s);
      return e == hipSuccess ? hipEventRecord(ev_[i & 1], s) : e;
    };
    // The first chunk comes after all the work enqueued on s, which may be long:
    // the threads start when it is there, so that nothing spins until then.
    hipError_t e = fill(0);
    if (e == hipSuccess && chunks > 1) e = fill(1);
    if (e == hipSuccess) e = hipEventSynchronize(ev_[0]);
    std::thread team[kThreads - 1];
    int started = 0;
    if (e == hipSuccess) {
      try {
        for (; started < kThreads - 1; ++started) team[started] = std::thread(work, started + 1);
      } catch (...) {   // no threads to be had: the plain copy
        stop = true;
        for (int t = 0; t < started; ++t) team[t].join();
        return plain(dst, src, n, s);
      }
    }
    for (size_t i = 0; i < chunks && e == hipSuccess; ++i) {
      if (i > 0) e = hipEventSynchronize(ev_[i & 1]);
      if (e != hipSuccess) break;
      filled.store(i + 1, std::memory_order_release);
      slice(i, 0);
      while (emptied.load(std::memory_order_acquire) < (i + 1) * kThreads) std::this_thread::yield();
      if (i + 2 < chunks) e = fill(i + 2);
    }
    stop = true;
    for (int t = 0; t < started; ++t) team[t].join();
    const hipError_t d = hipStreamSynchronize(s);   // nothing may still write the pinned chunks
    return e == hipSuccess ? d : e;
  }

 private:
  static constexpr size_t kChunk = size_t(4) << 20;
  static constexpr size_t kLeast = size_t(16) << 20;   // below, the first use's pinning costs what the threads gain
  static constexpr int kThreads = 4;
  void* pin_[2] = {nullptr, nullptr};
  hipEvent_t ev_[2] = {nullptr, nullptr};
  int ev_device_[2] = {0, 0};

  static hipError_t plain(void* dst, const void* src, size_t n, hipStream_t s) {
    const hipError_t e = hipMemcpyAsync(dst, src, n, hipMemcpyDeviceToHost, s);
    return e == hipSuccess ? hipStreamSynchronize(s) : e;
  }
  // Memory that the runtime knows (pinned, managed) is written by the copy engine itself.
  static bool pageable(const void* p) {
    hipPointerAttribute_t a;
    if (hipPointerGetAttributes(&a, p) == hipSuccess) return a.type == hipMemoryTypeUnregistered;
    (void)hipGetLastError();   // (an address that is not the runtime's may also be an error)
    return true;
  }
  // The pinned chunks and the events, which belong to the device of the stream
  // that they are recorded on (the caller's current device may be another).
  bool ready(hipStream_t s) {
    int now = 0;
    hipDevice_t dev = 0;
    bool ok = hipGetDevice(&now) == hipSuccess && hipStreamGetDevice(s, &dev) == hipSuccess;
    const bool move = ok && dev != now;
    if (move) ok = hipSetDevice(dev) == hipSuccess;
    for (int b = 0; b < 2 && ok; ++b) {
      if (!pin_[b] && hipHostMalloc(&pin_[b], kChunk, hipHostMallocDefault) != hipSuccess) {
        pin_[b] = nullptr;
        ok = false;
      }
      if (ev_[b] && ev_device_[b] != dev) {
        (void)hipEventDestroy(ev_[b]);
        ev_[b] = nullptr;
      }
      if (ok && !ev_[b]) {
        ok = hipEventCreateWithFlags(&ev_[b], hipEventDisableTiming) == hipSuccess;
        if (!ok) ev_[b] = nullptr;
        ev_device_[b] = dev;
      }
    }
    if (move) (void)hipSetDevice(now);
    if (!ok) (void)hipGetLastError();
    return ok;
  }
};

}  // namespace dugks
