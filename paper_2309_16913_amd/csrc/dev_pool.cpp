// Device memory kept between calls: workspaces (with pinned host words and an
// event) and plain blocks.  hipMalloc and hipFree cost tens of microseconds
// to milliseconds each and hipFree waits for the whole device, so calls that
// would allocate each time take their memory from here.  What is kept is
// bounded and goes back to the device as soon as an allocation of the library
// fails for lack of memory.
#include "dev_pool.h"

#include <algorithm>
#include <mutex>
#include <new>
#include <vector>

namespace rtk {
namespace {

// Freed blocks kept per device: so many, so large, so much in all.
constexpr int kBlocksKept = 16;
constexpr uint64_t kBlockMax = 512ull << 20, kBlocksMax = 1ull << 30;

struct Block {
    void *p;
    uint64_t bytes;
};
struct DevPool {
    std::mutex mu;
    std::vector<PoolWs *> idle;   // longest idle first; room for every workspace there is (see pool_acquire)
    size_t made = 0;              // workspaces there are, idle or handed out
    Block blocks[kBlocksKept];    // freed blocks, none in use by the device; longest kept first
    int nblocks = 0;
    uint64_t block_bytes = 0;
};
DevPool g_pool[kPoolDevices];

bool pooled(int dev) { return dev >= 0 && dev < kPoolDevices; }

// Takes the device memory of an idle workspace that the device is done with.
void *take_memory(PoolWs *w) {
    if (!w->d || hipEventQuery(w->done) != hipSuccess) return nullptr;
    void *d = w->d;
    w->d = nullptr;
    w->bytes = 0;
    return d;
}

// Gives every kept block and every idle workspace's memory back to the device.
void trim(int dev) {
    DevPool &p = g_pool[dev];
    Block old[kBlocksKept];
    int n = 0;
    {
        std::lock_guard<std::mutex> lk(p.mu);
        std::swap(n, p.nblocks);
        std::copy(p.blocks, p.blocks + n, old);
        p.block_bytes = 0;
    }
    for (int i = 0; i < n; ++i) (void)hipFree(old[i].p);
    for (;;) {   // one at a time: freed outside the lock, without a list of its own
        void *d = nullptr;
        {
            std::lock_guard<std::mutex> lk(p.mu);
            for (PoolWs *w : p.idle)
                if ((d = take_memory(w))) break;
        }
        if (!d) break;
        (void)hipFree(d);
    }
}

hipError_t ws_alloc(int dev, PoolWs *w, uint64_t bytes) {
    if (w->d) (void)hipFree(w->d);
    w->d = nullptr;
    w->bytes = 0;
    hipError_t e = dev_malloc(dev, &w->d, bytes);
    if (e == hipSuccess) w->bytes = bytes;
    else w->d = nullptr;
    return e;
}

}  // namespace

hipError_t dev_malloc(int dev, void **p, uint64_t bytes) {
    hipError_t e = hipMalloc(p, bytes);
    if (e == hipErrorOutOfMemory && pooled(dev)) {
        (void)hipGetLastError();
        trim(dev);
        e = hipMalloc(p, bytes);
    }
    return e;
}

// The smallest idle workspace that is large enough, else an idle one (grown) or
// a new one.
hipError_t pool_acquire(int dev, uint64_t bytes, uint64_t extra, PoolWs **out, bool exact) {
    if (!pooled(dev)) return hipErrorInvalidDevice;
    DevPool &p = g_pool[dev];
    const uint64_t want = bytes + extra;
    PoolWs *w = nullptr;
    {
        std::lock_guard<std::mutex> lk(p.mu);
        size_t at = 0;
        for (size_t i = 0; i < p.idle.size(); ++i) {
            PoolWs *c = p.idle[i];
            const bool fits = c->bytes >= want;
            if (w && (w->bytes >= want ? (!fits || c->bytes >= w->bytes) : !fits)) continue;
            if (hipEventQuery(c->done) != hipSuccess) continue;
            w = c;
            at = i;
        }
        if (w) {
            p.idle.erase(p.idle.begin() + (long)at);
        } else {
            p.idle.reserve(p.made + 1);   // so that handing one back never allocates
            p.made += 1;
        }
    }
    hipError_t e = hipSuccess;
    if (!w) {
        w = new (std::nothrow) PoolWs();
        if (!w) e = hipErrorMemoryAllocation;
        if (e == hipSuccess) e = hipEventCreateWithFlags(&w->done, hipEventDisableTiming);
        if (e == hipSuccess) e = hipHostMalloc(reinterpret_cast<void **>(&w->host), 64, hipHostMallocDefault);
        if (e != hipSuccess) {
            if (w && w->done) (void)hipEventDestroy(w->done);
            delete w;
            std::lock_guard<std::mutex> lk(p.mu);
            p.made -= 1;
            return e;
        }
    }
    if (w->bytes < want) {
        // by half again for the next larger call, but not by much of the device
        e = ws_alloc(dev, w, exact ? want : want + std::min<uint64_t>(want / 2, 256ull << 20));
        if (e == hipErrorOutOfMemory && !exact) {
            (void)hipGetLastError();
            e = ws_alloc(dev, w, want);
        }
        if (e == hipErrorOutOfMemory && extra) {
            (void)hipGetLastError();
            e = ws_alloc(dev, w, bytes);
        }
    }
    if (e != hipSuccess) {   // its event and pinned words stay valid for a later call
        std::lock_guard<std::mutex> lk(p.mu);
        p.idle.push_back(w);
        return e;
    }
    *out = w;
    return hipSuccess;
}

void pool_release(int dev, PoolWs *w, hipStream_t s, uint64_t keep) {
    if (!w) return;
    if (w->bytes > keep) {
        (void)hipFree(w->d);
        w->d = nullptr;
        w->bytes = 0;
    }
    (void)hipEventRecord(w->done, s);
    DevPool &p = g_pool[dev];
    {
        std::lock_guard<std::mutex> lk(p.mu);
        p.idle.push_back(w);
    }
    // what other workspaces hold makes room; those still in use by the device
    // are left, and looked at again by the next call
    for (;;) {
        void *d = nullptr;
        {
            std::lock_guard<std::mutex> lk(p.mu);
            uint64_t sum = 0;
            for (const PoolWs *c : p.idle) sum += c->bytes;
            if (sum <= kIdleMax) break;
            for (PoolWs *c : p.idle)
                if (c != w && (d = take_memory(c))) break;
        }
        if (!d) break;
        (void)hipFree(d);
    }
}

// A kept block of at least `bytes` and at most a quarter (or 1 MiB) more, else
// a new one; *got receives its size.
hipError_t block_alloc(int dev, uint64_t bytes, void **p, uint64_t *got) {
    if (pooled(dev)) {
        DevPool &d = g_pool[dev];
        std::lock_guard<std::mutex> lk(d.mu);
        int best = -1;
        for (int i = 0; i < d.nblocks; ++i) {
            const uint64_t b = d.blocks[i].bytes;
            if (b >= bytes && b <= bytes + bytes / 4 + (1u << 20) && (best < 0 || b < d.blocks[best].bytes)) best = i;
        }
        if (best >= 0) {
            *p = d.blocks[best].p;
            *got = d.blocks[best].bytes;
            d.block_bytes -= *got;
            std::copy(d.blocks + best + 1, d.blocks + d.nblocks, d.blocks + best);
            d.nblocks -= 1;
            return hipSuccess;
        }
    }
    *got = bytes;
    return dev_malloc(dev, p, bytes);
}

// Waits for the device (which must be current), as hipFree does: work of any
// stream may still read the block.
void block_free(int dev, void *p, uint64_t bytes) {
    if (!p) return;
    if (pooled(dev) && bytes <= kBlockMax && hipDeviceSynchronize() == hipSuccess) {
        // the longest kept make room: a program that moved on to other sizes
        // reuses its own blocks again
        Block old[kBlocksKept];
        int n = 0;
        {
            DevPool &d = g_pool[dev];
            std::lock_guard<std::mutex> lk(d.mu);
            while (d.nblocks - n >= kBlocksKept || d.block_bytes + bytes > kBlocksMax) {
                old[n] = d.blocks[n];
                d.block_bytes -= d.blocks[n].bytes;
                n += 1;
            }
            std::copy(d.blocks + n, d.blocks + d.nblocks, d.blocks);
            d.nblocks -= n;
            d.blocks[d.nblocks++] = Block{p, bytes};
            d.block_bytes += bytes;
        }
        for (int i = 0; i < n; ++i) (void)hipFree(old[i].p);
        return;
    }
    (void)hipFree(p);
}

}  // namespace rtk
