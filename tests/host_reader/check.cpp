// HostReader (host_copy.cpp) against the HIP stand-in beside this file.  check NAME: exit code 0 when it holds.
#include "host_copy.h"

#include <cstdio>
#include <cstring>
#include <new>
#include <string>

// Allocations of the thread that armed this, outside the stand-in, until one of them fails (-1: none does).
static thread_local int allocations_left = -1;
void* operator new(size_t n) {
  if (!stub::quiet && allocations_left >= 0 && allocations_left-- == 0) throw std::bad_alloc();
  if (void* p = std::malloc(n ? n : 1)) return p;
  throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

using cdp::HostReader;

namespace {

constexpr size_t BIG = (33u << 20) + 12;  // above the size from which threads copy, and not a whole number of pieces
std::vector<char> device_memory(BIG), host_memory(BIG);

void fill(std::vector<char>& v, unsigned seed) {
  for (size_t i = 0; i < v.size(); ++i) v[i] = (char)((i * 2654435761u + seed) >> 13);
}
// Work that writes the weights, enqueued on `s`, and what it writes.
std::vector<char> enqueue_update(hipStream_t s, unsigned seed) {
  std::vector<char> want(BIG);
  fill(want, seed);
  std::lock_guard<std::recursive_mutex> l(stub::mutex);
  stub::push(s, [want] { std::memcpy(device_memory.data(), want.data(), BIG); });
  return want;
}
bool reads(HostReader& r, hipStream_t s, const std::vector<char>& want, size_t bytes = BIG) {
  fill(host_memory, 99);
  const hipError_t e = r.read(host_memory.data(), device_memory.data(), bytes, s);
  if (e != hipSuccess) { std::printf("read: error %d\n", (int)e); return false; }
  if (std::memcmp(host_memory.data(), want.data(), bytes)) { std::printf("read: stale or wrong bytes\n"); return false; }
  return true;
}

// Every kind of stream handle that a context can be given, twice each, and a size that one plain copy serves.
bool order() {
  stub::Stream own;
  stub::created.push_back(&own);
  for (hipStream_t s : {(hipStream_t) nullptr, hipStreamPerThread, &own}) {
    HostReader r;
    for (unsigned k = 1; k < 3; ++k)
      if (!reads(r, s, enqueue_update(s, k))) return false;
    if (!reads(r, s, enqueue_update(s, 7), 4096)) return false;
  }
  return stub::pinned_now == 0 && stub::events_now == 0;
}

// A copy that fails is reported, and nothing writes into the buffers afterwards.
bool failing_copy() {
  for (int n : {0, 3, 9}) {
    HostReader r;
    auto want = enqueue_update(hipStreamPerThread, 3);
    stub::fail_copy = stub::async_copies + n;
    if (r.read(host_memory.data(), device_memory.data(), BIG, hipStreamPerThread) == hipSuccess) return false;
    stub::fail_copy = -1;
    for (auto& t : stub::per_thread)
      if (t.second.done != t.second.work.size()) return false;
    for (auto& t : stub::legacy)
      if (t.second.done != t.second.work.size()) return false;
    if (!reads(r, hipStreamPerThread, want)) return false;
  }
  return true;
}

// No memory for the k-th helper thread: the call does without it, and nothing is thrown.
bool no_memory_for_threads() {
  for (int k = 0; k < 3; ++k) {
    HostReader r;
    if (!reads(r, nullptr, enqueue_update(nullptr, 1))) return false;  // buffers and events are there
    auto want = enqueue_update(nullptr, 20 + k);
    fill(host_memory, 99);
    allocations_left = k;
    const hipError_t e = r.read(host_memory.data(), device_memory.data(), BIG, nullptr);
    const bool fired = allocations_left < 0;
    allocations_left = -1;
    if (!fired || e != hipSuccess || std::memcmp(host_memory.data(), want.data(), BIG)) return false;
  }
  return true;
}

// Calling threads whose current device differs from call to call; the context's stream is on device 0.
bool other_device() {
  stub::Stream own;
  stub::created.push_back(&own);
  HostReader r;
  bool ok = true;
  for (int d : {0, 1, 0, 1}) {
    stub::device = d;
    ok = ok && reads(r, &own, enqueue_update(&own, 30 + d));
  }
  stub::device = 0;
  return ok;
}

// Two threads that read different vectors of one context at a time.
bool two_callers() {
  std::vector<char> source[2] = {std::vector<char>(BIG), std::vector<char>(BIG)};
  for (int k = 0; k < 4; ++k) {
    HostReader r;
    bool ok[2] = {false, false};
    std::thread t[2];
    for (int c = 0; c < 2; ++c) fill(source[c], 40 + 2 * k + c);
    for (int c = 0; c < 2; ++c) {
      t[c] = std::thread([&, c] {
        std::vector<char> host(BIG);
        ok[c] = r.read(host.data(), source[c].data(), BIG, nullptr) == hipSuccess && host == source[c];
      });
    }
    for (auto& x : t) x.join();
    if (!ok[0] || !ok[1]) return false;
  }
  return true;
}

// Memory that the device reaches by itself needs no help from the host: one copy.
bool pinned_by_caller() {
  HostReader r;
  stub::pinned_by_caller = host_memory.data();
  const bool ok = reads(r, nullptr, enqueue_update(nullptr, 50));
  stub::pinned_by_caller = nullptr;
  if (!ok || stub::async_copies != 0 || stub::plain_copies != 1) return false;
  return reads(r, nullptr, enqueue_update(nullptr, 51)) && stub::async_copies > 0 && stub::plain_copies == 1;
}

}  // namespace

int main(int argc, char** argv) {
  const std::string name = argc > 1 ? argv[1] : "";
  bool ok = false;
  stub::late = std::this_thread::get_id();
  if (name == "order") ok = order();
  else if (name == "failing_copy") ok = failing_copy();
  else if (name == "no_memory_for_threads") ok = no_memory_for_threads();
  else if (name == "other_device") ok = other_device();
  else if (name == "two_callers") ok = two_callers();
  else if (name == "pinned_by_caller") ok = pinned_by_caller();
  else std::printf("no such check\n");
  std::printf("%s: %s\n", name.c_str(), ok ? "holds" : "FAILS");
  return ok ? 0 : 1;
}
