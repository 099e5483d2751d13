// Device-to-host copies of whole fields into the caller's (pageable) arrays.
#pragma once
#include <hip/hip_runtime.h>

#include <stddef.h>

namespace sbt {

// A pageable copy through the runtime is one thread's memcpy out of its
// staging buffer, page faults of a fresh array included: 226 MB of fields
// took 20 ms, two thirds of that in the faults.  Here kWorkers threads (the
// caller's among them) each take pieces of kChunk bytes in turn through a
// pinned buffer of their own, so one's copy out overlaps the others'
// transfers.  Buffers are made at the first large copy and freed with the
// object; without them, below kLarge bytes, or on the per-thread stream the
// runtime copies, up to kSmall bytes that lie together on the device in one
// transfer (four fields of 16^3 cells, 131 kB, 49 us, 71 in four transfers; of
// 32^3, 1 MB, 120 and 100).
class HostCopy {
 public:
  struct Piece {
    const void *dev;
    void *host;
    size_t bytes;
  };
  HostCopy() = default;
  HostCopy(const HostCopy &) = delete;
  HostCopy &operator=(const HostCopy &) = delete;
  ~HostCopy();
  // Copies the pieces in stream order and waits for them.
  hipError_t to_host(const Piece *p, int n, hipStream_t s);

 private:
  static constexpr int kWorkers = 8;
  static constexpr size_t kChunk = (size_t)1 << 20, kLarge = (size_t)4 << 20,
                          kSmall = (size_t)1 << 19;
  char *pin_ = nullptr;  // [kWorkers][kChunk]
  char *tmp_ = nullptr;  // [kSmall] where pin_ has not been needed yet
  hipEvent_t ev_[kWorkers] = {};
  bool failed_ = false;
  bool ready();
};

}  // namespace sbt
