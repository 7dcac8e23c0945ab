// Device -> host copies of whole weight vectors into ordinary (pageable) memory.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>
#include <mutex>

namespace cdp {

// Four threads, each with two pinned buffers: a thread requests its next piece into one while it empties the other into the
// caller's memory.  A plain copy into pageable memory does the same from one thread, and what it waits for is mostly the
// host: copying, and the page faults of memory that is written for the first time.  The read alone, the device idle before it
// (24 vectors of 67 MB, 1.63 GB; the link moves 57 GB/s into pinned memory): 160 -> 54 ms into fresh memory, 88 -> 41 ms (38
// GB/s) into memory in use; one vector of 16.8 MB 0.92 -> 0.53 ms.
class HostReader {
 public:
  HostReader() = default;
  HostReader(const HostReader&) = delete;
  HostReader& operator=(const HostReader&) = delete;
  ~HostReader();
  // Copies after everything enqueued on `stream` so far; returns when dst is written.
  hipError_t read(void* dst, const void* src, size_t bytes, hipStream_t stream);

 private:
  static constexpr int THREADS = 4, DEPTH = 2;
  static constexpr size_t PIECE = 2u << 20;
  // From here on the threads pay for 16 MiB of pinned memory (below it one plain copy).
  static constexpr size_t WORTH = 16u << 20;
  bool prepare(int device);
  void release();
  hipError_t work(int thread, char* dst, const char* src, size_t bytes);
  std::mutex in_use_;
  int device_ = 0;
  char* pinned_ = nullptr;
  hipEvent_t event_[THREADS * DEPTH] = {};
};

}  // namespace cdp
