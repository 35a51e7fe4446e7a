// Device memory kept between calls: workspaces (with pinned host words and an
// event) and plain blocks.  hipMalloc and hipFree cost tens of microseconds
// to milliseconds each and hipFree waits for the whole device, so calls that
// would allocate each time take their memory from here.
#include <mutex>
#include <new>
#include <vector>

#include "rt_api_internal.h"

namespace rtk {
namespace {

struct Block {
    void *p;
    uint64_t bytes;
};
struct DevPool {
    std::mutex mu;
    std::vector<PoolWs *> idle;
    std::vector<Block> blocks;   // freed blocks, none in use by the device
    uint64_t block_bytes = 0;
};
DevPool g_pool[kPoolDevices];

// Freed blocks kept per device: so many, so large, so much in all.
constexpr size_t kBlocksKept = 16;
constexpr uint64_t kBlockMax = 512ull << 20, kBlocksMax = 1ull << 30;

// Gives every kept block back to the device.
void trim(int dev) {
    std::vector<Block> old;
    {
        std::lock_guard<std::mutex> lk(g_pool[dev].mu);
        old.swap(g_pool[dev].blocks);
        g_pool[dev].block_bytes = 0;
    }
    for (const Block &b : old) (void)hipFree(b.p);
}

hipError_t dev_malloc(int dev, void **p, uint64_t bytes) {
    hipError_t e = hipMalloc(p, bytes);
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        trim(dev);
        e = hipMalloc(p, bytes);
    }
    return e;
}

hipError_t ws_alloc(int dev, PoolWs *w, uint64_t bytes) {
    if (w->d) (void)hipFree(w->d);
    w->d = nullptr;
    w->bytes = 0;
    hipError_t e = dev_malloc(dev, &w->d, bytes);
    if (e == hipSuccess) w->bytes = bytes;
    return e;
}

}  // namespace

// The smallest idle workspace that is large enough, else an idle one (grown;
// by half again unless exact) or a new one.
hipError_t pool_acquire(int dev, uint64_t bytes, PoolWs **out, bool exact) {
    if (dev < 0 || dev >= kPoolDevices) return hipErrorInvalidDevice;
    DevPool &p = g_pool[dev];
    PoolWs *w = nullptr;
    {
        std::lock_guard<std::mutex> lk(p.mu);
        size_t at = 0;
        for (size_t i = 0; i < p.idle.size(); ++i) {
            PoolWs *c = p.idle[i];
            const bool fits = c->bytes >= bytes;
            if (w && (w->bytes >= bytes ? (!fits || c->bytes >= w->bytes) : !fits)) continue;
            if (hipEventQuery(c->done) != hipSuccess) continue;
            w = c;
            at = i;
        }
        if (w) p.idle.erase(p.idle.begin() + (long)at);
    }
    hipError_t e = hipSuccess;
    if (!w) {
        w = new PoolWs();
        e = hipEventCreateWithFlags(&w->done, hipEventDisableTiming);
        if (e == hipSuccess) e = hipHostMalloc(reinterpret_cast<void **>(&w->host), 64, hipHostMallocDefault);
    }
    if (e == hipSuccess && w->bytes < bytes) e = ws_alloc(dev, w, exact ? bytes : bytes + bytes / 2);
    if (e != hipSuccess) {
        // keep the object: its event and pinned words stay valid for a later call
        if (w->done && w->host) {
            std::lock_guard<std::mutex> lk(p.mu);
            p.idle.push_back(w);
        } else {
            if (w->done) (void)hipEventDestroy(w->done);
            delete w;
        }
        return e;
    }
    *out = w;
    return hipSuccess;
}

// Hands a workspace back once everything enqueued on s so far has finished.
// keep: device memory above this is freed first (the caller has waited for s).
void pool_release(int dev, PoolWs *w, hipStream_t s, uint64_t keep) {
    if (!w) return;
    if (w->bytes > keep) {
        (void)hipFree(w->d);
        w->d = nullptr;
        w->bytes = 0;
    }
    (void)hipEventRecord(w->done, s);
    std::lock_guard<std::mutex> lk(g_pool[dev].mu);
    g_pool[dev].idle.push_back(w);
}

// A kept block of at least `bytes` and at most a quarter (or 1 MiB) more, else
// a new one; *got receives its size.
hipError_t block_alloc(int dev, uint64_t bytes, void **p, uint64_t *got) {
    if (dev >= 0 && dev < kPoolDevices) {
        DevPool &d = g_pool[dev];
        std::lock_guard<std::mutex> lk(d.mu);
        size_t best = d.blocks.size();
        for (size_t i = 0; i < d.blocks.size(); ++i) {
            const uint64_t b = d.blocks[i].bytes;
            if (b >= bytes && b <= bytes + bytes / 4 + (1u << 20) &&
                (best == d.blocks.size() || b < d.blocks[best].bytes))
                best = i;
        }
        if (best < d.blocks.size()) {
            *p = d.blocks[best].p;
            *got = d.blocks[best].bytes;
            d.block_bytes -= *got;
            d.blocks.erase(d.blocks.begin() + (long)best);
            return hipSuccess;
        }
    }
    *got = bytes;
    return dev >= 0 && dev < kPoolDevices ? dev_malloc(dev, p, bytes) : hipMalloc(p, bytes);
}

// Waits for the device (which must be current), as hipFree does: work of any
// stream may still read the block.
void block_free(int dev, void *p, uint64_t bytes) {
    if (!p) return;
    if (dev >= 0 && dev < kPoolDevices && bytes <= kBlockMax && hipDeviceSynchronize() == hipSuccess) {
        // the longest kept make room: a program that moved on to other sizes
        // reuses its own blocks again
        std::vector<Block> old;
        {
            DevPool &d = g_pool[dev];
            std::lock_guard<std::mutex> lk(d.mu);
            size_t n = 0;
            while (d.blocks.size() - n >= kBlocksKept || d.block_bytes + bytes > kBlocksMax)
                d.block_bytes -= d.blocks[n++].bytes;
            old.assign(d.blocks.begin(), d.blocks.begin() + (long)n);
            d.blocks.erase(d.blocks.begin(), d.blocks.begin() + (long)n);
            d.blocks.push_back(Block{p, bytes});
            d.block_bytes += bytes;
        }
        for (const Block &b : old) (void)hipFree(b.p);
        return;
    }
    (void)hipFree(p);
}

}  // namespace rtk
