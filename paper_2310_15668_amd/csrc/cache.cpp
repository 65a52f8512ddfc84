// Device buffers of a context: allocation and release ordered on its stream, and
// the freed buffers it keeps.  Host code only.
#include <algorithm>
#include <string>

#include "common.h"

namespace {

// Graph and scratch buffers are stream-ordered allocations on the context's
// stream when the device has memory pools, so that a free never waits for
// work queued by other contexts on other streams.
hipError_t raw_alloc(mochy_ctx* ctx, void** p, size_t n) {
  return ctx->async_alloc ? hipMallocAsync(p, n, ctx->stream) : hipMalloc(p, n);
}

void raw_free(mochy_ctx* ctx, void* p) {
  if (ctx->async_alloc) (void)hipFreeAsync(p, ctx->stream);
  else (void)hipFree(p);
}

void release_cached(mochy_ctx* ctx) {  // with cache_mu held
  for (auto& kv : ctx->cache_free) {
    ctx->cache_live.erase(kv.second);
    raw_free(ctx, kv.second);
  }
  ctx->cache_free.clear();
  ctx->cache_bytes = 0;
}

}  // namespace

void cache_release(mochy_ctx* ctx) {
  std::lock_guard<std::mutex> lock(ctx->cache_mu);
  release_cached(ctx);
}

void cache_set_limit(mochy_ctx* ctx, int64_t bytes) {
  std::lock_guard<std::mutex> lock(ctx->cache_mu);
  ctx->cache_limit = bytes;
  if (ctx->cache_bytes > bytes) release_cached(ctx);
}

int64_t cache_held(mochy_ctx* ctx) {
  std::lock_guard<std::mutex> lock(ctx->cache_mu);
  return ctx->cache_bytes;
}

namespace {

// Buffers go through a per-context cache: a freed block is kept (up to
// cache_limit bytes in all) and handed to a later request that it fits with at
// most half of it unused.  Freeing and mapping again the hundred-odd GB that a
// batch of 65 graphs holds costs up to seconds per call; reusing the blocks
// costs nothing.  A context works on one
// stream, so a reused block's earlier readers are ordered before its new
// writers.
// Small blocks as well: a call on 4,009 hyperedges takes and gives back 37, and
// the stream-ordered allocator's calls were 1.36 ms of its 3.69 (hipFreeAsync
// 23 us, hipMallocAsync 14 us each).  Sizes come in steps of a quarter of a
// power of two, whole 2 MiB pages from there on, so that calls of about the same
// size find each other's blocks; the number kept is bounded by what the calls
// use at once of each step.
size_t cache_size(size_t n) {
  size_t step = size_t(2) << 20;
  if (n < step) {
    step = 64;
    while (step * 8 < n) step <<= 1;  // n in (4, 8] steps
    if (n <= 256) return 256;
  }
  return (n + step - 1) / step * step;
}

}  // namespace

mochy_status device_alloc(mochy_ctx* ctx, void** p, size_t bytes) {
  *p = nullptr;
  size_t n = std::max<size_t>(bytes, 8);
  if (ctx->arena) {  // allocation-free call: carve from the static scratch array
    const size_t at = (ctx->arena_used + 255) & ~size_t(255);
    if (at + n > ctx->arena_cap) {
      ctx->err = "the allocation-free call needs more than its " + std::to_string(ctx->arena_cap) +
                 "-byte scratch array (" + std::to_string(at + n) + " bytes so far)";
      return MOCHY_ERANGE;
    }
    *p = ctx->arena + at;
    ctx->arena_used = at + n;
    return MOCHY_OK;
  }
  // a graph may be freed by another thread than the one that runs a call on its
  // context (a caller's garbage collector)
  std::lock_guard<std::mutex> lock(ctx->cache_mu);
  const bool cached = ctx->cache_limit > 0;
  if (cached) {
    n = cache_size(n);
    auto it = ctx->cache_free.lower_bound(n);
    if (it != ctx->cache_free.end() && it->first / 2 <= n) {
      *p = it->second;
      ctx->cache_bytes -= int64_t(it->first);
      ctx->cache_free.erase(it);
      return MOCHY_OK;
    }
  }
  hipError_t e = raw_alloc(ctx, p, n);
  if (e != hipSuccess && !ctx->cache_free.empty()) {  // give the cached blocks back and retry
    (void)hipGetLastError();
    release_cached(ctx);
    (void)hipStreamSynchronize(ctx->stream);
    e = raw_alloc(ctx, p, n);
  }
  if (e != hipSuccess) {
    *p = nullptr;
    (void)hipGetLastError();
    ctx->err = "device allocation of " + std::to_string(bytes) + " bytes failed: " + hipGetErrorString(e);
    return MOCHY_ENOMEM;
  }
  if (cached) ctx->cache_live[*p] = n;
  return MOCHY_OK;
}

void device_free(mochy_ctx* ctx, void* p) {
  if (!p) return;
  const char* const arena = static_cast<const char*>(ctx->noalloc_scratch);
  if (arena && p >= arena && p < arena + kNoallocBytes) return;  // released with its call
  std::lock_guard<std::mutex> lock(ctx->cache_mu);
  auto it = ctx->cache_live.find(p);
  if (it != ctx->cache_live.end() && ctx->cache_bytes + int64_t(it->second) <= ctx->cache_limit) {
    ctx->cache_free.emplace(it->second, p);  // stays in cache_live until released
    ctx->cache_bytes += int64_t(it->second);
    return;
  }
  if (it != ctx->cache_live.end()) ctx->cache_live.erase(it);
  raw_free(ctx, p);
}
