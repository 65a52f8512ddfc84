// Host-sanitizer driver of the library's buffer cache
// (paper_2310_15668_amd/csrc/cache.cpp), built by tests/test_cache_cpu.py with
// ThreadSanitizer and with AddressSanitizer.  The runtime's allocator is a stub
// over malloc that counts what is out and refuses more than a set amount.
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <deque>
#include <mutex>
#include <thread>
#include <unordered_map>
#include <vector>

#include "common.h"

extern const size_t kNoallocBytes = 4096;

namespace {
std::mutex mu;
std::unordered_map<void*, size_t> out;
size_t held = 0, room = size_t(1) << 40;
std::atomic<long> calls{0};

hipError_t take(void** p, size_t n) {
  std::lock_guard<std::mutex> lock(mu);
  ++calls;
  if (held + n > room) return hipErrorOutOfMemory;
  *p = std::malloc(16);
  out[*p] = n;
  held += n;
  return hipSuccess;
}
hipError_t give(void* p) {
  std::lock_guard<std::mutex> lock(mu);
  auto it = out.find(p);
  if (it == out.end()) std::abort();  // freed twice, or never allocated
  held -= it->second;
  out.erase(it);
  std::free(p);
  return hipSuccess;
}
}  // namespace

extern "C" {
hipError_t hipMallocAsync(void** p, size_t n, hipStream_t) { return take(p, n); }
hipError_t hipMalloc(void** p, size_t n) { return take(p, n); }
hipError_t hipFreeAsync(void* p, hipStream_t) { return give(p); }
hipError_t hipFree(void* p) { return give(p); }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stub"; }
}

#define CHECK(x) \
  if (!(x)) { std::printf("line %d: " #x "\n", __LINE__); return 1; }

int main() {
  mochy_ctx ctx;
  ctx.async_alloc = true;
  cache_set_limit(&ctx, int64_t(1) << 30);
  // a freed block is handed out again where at most half of it is unused
  void *a, *b;
  CHECK(device_alloc(&ctx, &a, 1000) == MOCHY_OK);
  device_free(&ctx, a);
  CHECK(cache_held(&ctx) >= 1000 && held == size_t(cache_held(&ctx)));
  CHECK(device_alloc(&ctx, &b, 900) == MOCHY_OK && b == a);
  device_free(&ctx, b);
  CHECK(device_alloc(&ctx, &b, 300) == MOCHY_OK && b != a);
  device_free(&ctx, b);
  // a limit of 0 gives all of it back and keeps nothing more
  cache_set_limit(&ctx, 0);
  CHECK(held == 0 && cache_held(&ctx) == 0);
  CHECK(device_alloc(&ctx, &a, 5000) == MOCHY_OK);
  device_free(&ctx, a);
  CHECK(held == 0);
  // a block taken before the limit fell is not kept above it
  cache_set_limit(&ctx, int64_t(1) << 20);
  CHECK(device_alloc(&ctx, &a, 700000) == MOCHY_OK);
  cache_set_limit(&ctx, 1000);
  device_free(&ctx, a);
  CHECK(held == 0);
  // an allocation that fails has the kept blocks released, then is refused
  cache_set_limit(&ctx, int64_t(1) << 30);
  CHECK(device_alloc(&ctx, &a, 8 << 20) == MOCHY_OK);
  device_free(&ctx, a);
  CHECK(held > 0);
  room = 20 << 20;
  CHECK(device_alloc(&ctx, &a, 18 << 20) == MOCHY_OK);
  CHECK(device_alloc(&ctx, &b, 18 << 20) == MOCHY_ENOMEM && b == nullptr);
  device_free(&ctx, a);
  room = size_t(1) << 40;
  cache_set_limit(&ctx, 0);
  CHECK(held == 0);

  // one thread allocates, another frees, a third sets the limit and reads
  cache_set_limit(&ctx, int64_t(1) << 22);
  std::deque<void*> passed;
  std::mutex pm;
  std::atomic<bool> done{false};
  std::thread freer([&] {
    for (;;) {
      void* p = nullptr;
      {
        std::lock_guard<std::mutex> lock(pm);
        if (!passed.empty()) {
          p = passed.front();
          passed.pop_front();
        } else if (done) {
          return;
        }
      }
      if (p) device_free(&ctx, p);
      else std::this_thread::yield();
    }
  });
  std::thread setter([&] {
    for (int x = 0; !done; ++x) {
      cache_set_limit(&ctx, x % 3 ? int64_t(1) << (18 + x % 7) : 0);
      if (cache_held(&ctx) < 0) std::abort();
    }
  });
  for (int x = 0; x < 20000; ++x) {
    void* p;
    if (device_alloc(&ctx, &p, size_t(1) << (x % 20)) != MOCHY_OK) std::abort();
    std::lock_guard<std::mutex> lock(pm);
    passed.push_back(p);
  }
  done = true;
  freer.join();
  setter.join();
  cache_set_limit(&ctx, 0);
  CHECK(held == 0 && cache_held(&ctx) == 0 && ctx.cache_live.empty());
  std::printf("cache ok: %ld allocator calls\n", long(calls));
  return 0;
}
