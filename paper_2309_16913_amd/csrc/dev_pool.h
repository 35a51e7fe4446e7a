// Device memory kept between calls.
#pragma once

#include <hip/hip_runtime_api.h>

#include <cstdint>

namespace rtk {

// Device workspaces kept per device between calls, each with a few pinned host
// words and an event recorded behind its last use: one is handed out again only
// when that has completed, so calls on different streams or threads never
// share one while it is in use.
struct PoolWs {
    void *d = nullptr;
    uint64_t bytes = 0;
    uint64_t *host = nullptr;     // 8 pinned words
    hipEvent_t done = nullptr;
};
constexpr int kPoolDevices = 64;

// Idle workspaces hold at most this much device memory together, or what the
// one released last holds; the longest idle are freed first.
constexpr uint64_t kIdleMax = 8ull << 30;

// A workspace of at least `bytes`, and of `bytes + extra` if the device has that
// much: what is extra is only worth having.  More is taken for growth unless exact.
hipError_t pool_acquire(int dev, uint64_t bytes, uint64_t extra, PoolWs **out, bool exact = false);
// Hands a workspace back once everything enqueued on s so far has finished.
// keep: device memory above this is freed first (the caller has waited for s).
void pool_release(int dev, PoolWs *w, hipStream_t s, uint64_t keep = ~0ull);

// Plain device blocks; freed ones are kept up to a bound.
hipError_t block_alloc(int dev, uint64_t bytes, void **p, uint64_t *got);
void block_free(int dev, void *p, uint64_t bytes);

// hipMalloc on device dev (the current one) for memory that is hipFree'd.  When
// the device is out of memory, every kept block and idle workspace is given
// back first; all of the library's allocations come through here.
hipError_t dev_malloc(int dev, void **p, uint64_t bytes);

}  // namespace rtk
