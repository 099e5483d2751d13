#include "host_copy.h"

#include <stdlib.h>
#include <string.h>

#include <atomic>
#include <exception>
#include <thread>
#include <vector>

namespace sbt {

HostCopy::~HostCopy() {
  free(tmp_);
  for (hipEvent_t &e : ev_)
    if (e) (void)hipEventDestroy(e);
  if (pin_) (void)hipHostFree(pin_);
}

bool HostCopy::ready() {
  if (pin_ || failed_) return pin_ != nullptr;
  void *p = nullptr;
  failed_ = hipHostMalloc(&p, kWorkers * kChunk, hipHostMallocDefault) != hipSuccess;
  for (int i = 0; i < kWorkers && !failed_; ++i)
    failed_ = hipEventCreateWithFlags(&ev_[i], hipEventDisableTiming) != hipSuccess;
  if (failed_) {
    if (p) (void)hipHostFree(p);
    (void)hipGetLastError();  // the runtime copies instead
    return false;
  }
  pin_ = static_cast<char *>(p);
  return true;
}

hipError_t HostCopy::to_host(const Piece *p, int n, hipStream_t s) {
  size_t total = 0;
  bool joined = n > 1;  // the pieces follow one another on the device
  for (int i = 0; i < n; ++i) {
    joined = joined && (i == 0 || p[i].dev == static_cast<const char *>(p[i - 1].dev) + p[i - 1].bytes);
    total += p[i].bytes;
  }
  if (joined && total <= kSmall) {  // one transfer, then a copy per piece
    char *buf = pin_;
    if (!buf) {
      if (!tmp_) tmp_ = static_cast<char *>(malloc(kSmall));
      buf = tmp_;
    }
    if (buf) {
      hipError_t e = hipMemcpyAsync(buf, p[0].dev, total, hipMemcpyDeviceToHost, s);
      if (e == hipSuccess) e = hipStreamSynchronize(s);
      if (e != hipSuccess) return e;
      for (int i = 0; i < n; buf += p[i++].bytes) memcpy(p[i].host, buf, p[i].bytes);
      return hipSuccess;
    }
  }
  int dev = 0;
  // the per-thread stream is another one in each worker, which would not wait
  // for what the caller's holds: the caller copies by itself
  if (total < kLarge || s == hipStreamPerThread || !ready() || hipGetDevice(&dev) != hipSuccess) {
    for (int i = 0; i < n; ++i) {
      const hipError_t e = hipMemcpyAsync(p[i].host, p[i].dev, p[i].bytes, hipMemcpyDeviceToHost, s);
      if (e != hipSuccess) return e;
    }
    return hipStreamSynchronize(s);
  }
  std::atomic<size_t> next{0};
  std::atomic<int> err{(int)hipSuccess};
  auto work = [&](int w) {
    char *buf = pin_ + (size_t)w * kChunk;
    hipError_t e = hipSetDevice(dev);
    while (e == hipSuccess && err.load() == (int)hipSuccess) {
      // chunk `next` over the pieces, each cut from its start
      size_t c = next.fetch_add(1), off = 0;
      int i = 0;
      for (; i < n; ++i) {
        const size_t k = (p[i].bytes + kChunk - 1) / kChunk;
        if (c < k) {
          off = c * kChunk;
          break;
        }
        c -= k;
      }
      if (i == n) break;
      const size_t m = p[i].bytes - off < kChunk ? p[i].bytes - off : kChunk;
      e = hipMemcpyAsync(buf, static_cast<const char *>(p[i].dev) + off, m, hipMemcpyDeviceToHost, s);
      if (e == hipSuccess) e = hipEventRecord(ev_[w], s);
      if (e == hipSuccess) e = hipEventSynchronize(ev_[w]);
      if (e == hipSuccess) memcpy(static_cast<char *>(p[i].host) + off, buf, m);
    }
    if (e != hipSuccess) err.store((int)e);
  };
  std::vector<std::thread> crew;
  try {
    crew.reserve(kWorkers - 1);
    for (int w = 1; w < kWorkers; ++w) crew.emplace_back(work, w);
  } catch (const std::exception &) {  // fewer threads than asked for: those there do the work
  }
  work(0);
  for (std::thread &t : crew) t.join();
  const hipError_t e = hipStreamSynchronize(s);
  return err.load() != (int)hipSuccess ? (hipError_t)err.load() : e;
}

}  // namespace sbt
