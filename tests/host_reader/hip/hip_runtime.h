// The few HIP calls of host_copy.cpp, on the CPU: a stream is a list of work that runs when somebody waits for it, so a copy
// that was not ordered after the work before it reads what that work has not written yet.
#pragma once
#include <atomic>
#include <chrono>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <map>
#include <mutex>
#include <thread>
#include <utility>
#include <vector>

enum hipError_t { hipSuccess = 0, hipErrorInvalidValue = 1, hipErrorInvalidHandle = 400, hipErrorUnknown = 999 };
enum { hipHostMallocDefault = 0, hipEventDisableTiming = 2 };
enum hipMemcpyKind { hipMemcpyDeviceToHost = 2 };

namespace stub {
struct Stream;
}
typedef stub::Stream* hipStream_t;
#define hipStreamPerThread (reinterpret_cast<hipStream_t>(2))

namespace stub {
inline thread_local int device = 0;            // the current device is the thread's own
inline thread_local int quiet = 0;             // > 0: inside a stub call
struct Quiet {
  Quiet() { ++quiet; }
  ~Quiet() { --quiet; }
};

struct Stream {
  int device = 0;
  size_t done = 0;
  std::vector<std::function<void()>> work;
};
struct Event {
  int device = 0;
  Stream* stream = nullptr;
  size_t upto = 0;
};

inline std::recursive_mutex mutex;
inline std::map<int, Stream> legacy;                                      // per device: the null stream
inline std::map<std::pair<std::thread::id, int>, Stream> per_thread;      // hipStreamPerThread
inline std::vector<Stream*> created;
inline std::thread::id late;                                              // a thread whose copies come last
inline const void* pinned_by_caller = nullptr;
inline int pinned_now = 0, events_now = 0, plain_copies = 0, async_copies = 0, fail_copy = -1;

inline Stream* find(hipStream_t s) {
  if (s == nullptr) {
    Stream& x = legacy[device];
    x.device = device;
    return &x;
  }
  if (s == hipStreamPerThread) {
    Stream& x = per_thread[{std::this_thread::get_id(), device}];
    x.device = device;
    return &x;
  }
  return s;
}
inline void run(Stream* s, size_t upto) {
  while (s->done < upto) {
    const size_t k = s->done++;
    s->work[k]();
  }
}
// Everything that was enqueued on the device's other streams so far: the null stream waits for it.
inline std::vector<std::pair<Stream*, size_t>> others(int dev) {
  std::vector<std::pair<Stream*, size_t>> v;
  for (auto& t : per_thread)
    if (t.second.device == dev) v.push_back({&t.second, t.second.work.size()});
  for (Stream* s : created)
    if (s->device == dev) v.push_back({s, s->work.size()});
  return v;
}
inline void push(hipStream_t h, std::function<void()> f) {
  Stream* s = find(h);
  if (h == nullptr) {
    auto before = others(s->device);
    s->work.push_back([before, f] {
      for (auto& b : before) run(b.first, b.second);
      f();
    });
  } else {
    s->work.push_back(std::move(f));
  }
}
}  // namespace stub

typedef stub::Event* hipEvent_t;

enum hipMemoryType { hipMemoryTypeUnregistered = 0, hipMemoryTypeHost = 1 };
struct hipPointerAttribute_t {
  hipMemoryType type;
};

inline hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void* p) {
  if (p != stub::pinned_by_caller) return hipErrorInvalidValue;
  a->type = hipMemoryTypeHost;
  return hipSuccess;
}
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipGetDevice(int* d) { *d = stub::device; return hipSuccess; }
inline hipError_t hipSetDevice(int d) { stub::device = d; return hipSuccess; }
inline hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  stub::Quiet q;
  std::lock_guard<std::recursive_mutex> l(stub::mutex);
  ++stub::pinned_now;
  *p = std::malloc(n);
  return hipSuccess;
}
inline hipError_t hipHostFree(void* p) {
  stub::Quiet q;
  std::lock_guard<std::recursive_mutex> l(stub::mutex);
  --stub::pinned_now;
  std::free(p);
  return hipSuccess;
}
inline hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  stub::Quiet q;
  std::lock_guard<std::recursive_mutex> l(stub::mutex);
  ++stub::events_now;
  *e = new stub::Event;
  (*e)->device = stub::device;
  return hipSuccess;
}
inline hipError_t hipEventDestroy(hipEvent_t e) {
  stub::Quiet q;
  std::lock_guard<std::recursive_mutex> l(stub::mutex);
  --stub::events_now;
  delete e;
  return hipSuccess;
}
inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t h) {
  stub::Quiet q;
  std::lock_guard<std::recursive_mutex> l(stub::mutex);
  stub::Stream* s = stub::find(h);
  if (s->device != e->device) return hipErrorInvalidHandle;
  e->stream = s;
  e->upto = s->work.size();
  return hipSuccess;
}
inline hipError_t hipEventSynchronize(hipEvent_t e) {
  stub::Quiet q;
  {
    std::lock_guard<std::recursive_mutex> l(stub::mutex);
    if (e->stream) stub::run(e->stream, e->upto);
  }
  std::this_thread::sleep_for(std::chrono::milliseconds(2));  // the host is slow to see it: others run in between
  return hipSuccess;
}
inline hipError_t hipStreamSynchronize(hipStream_t h) {
  stub::Quiet q;
  std::lock_guard<std::recursive_mutex> l(stub::mutex);
  stub::Stream* s = stub::find(h);
  stub::run(s, s->work.size());
  return hipSuccess;
}
inline hipError_t hipMemcpyAsync(void* dst, const void* src, size_t n, hipMemcpyKind, hipStream_t h) {
  if (std::this_thread::get_id() == stub::late) std::this_thread::sleep_for(std::chrono::milliseconds(20));  // the others are well ahead
  stub::Quiet q;
  std::lock_guard<std::recursive_mutex> l(stub::mutex);
  if (stub::async_copies++ == stub::fail_copy) return hipErrorUnknown;
  stub::push(h, [dst, src, n] { std::memcpy(dst, src, n); });
  return hipSuccess;
}
inline hipError_t hipMemcpy(void* dst, const void* src, size_t n, hipMemcpyKind) {
  stub::Quiet q;
  std::lock_guard<std::recursive_mutex> l(stub::mutex);
  ++stub::plain_copies;
  stub::Stream* s = stub::find(nullptr);
  stub::push(nullptr, [dst, src, n] { std::memcpy(dst, src, n); });
  stub::run(s, s->work.size());
  return hipSuccess;
}
