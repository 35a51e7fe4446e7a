// rt_range_select_async: a range select into caller-owned device buffers
// whose workspace the library keeps in a per-device pool.
//
// The call enqueues the count stage, waits for the total (which the scan
// writes to pinned host memory), and either refuses the select (RT_ENOMEM, the ids buffer untouched)
// or enqueues the fill stage and the sort and returns while they run.  A
// pooled workspace is handed to a later call only after the event recorded
// behind its last use has completed, so calls on different streams never
// share one while it is in use.
#include <new>

#include "../../include/rt.h"
#include "rt_api_internal.h"
#include "rt_internal.h"

using namespace rtk;

namespace {
// d_total = total, or all ones when a kernel-side check failed
__global__ void total_word(const uint64_t *__restrict__ status, uint64_t *__restrict__ d_total) {
    d_total[0] = (status[1] & 2u) ? ~0ull : status[0];
}
}  // namespace

extern "C" int rt_range_select_async(const rt_tree *t, const float *d_queries, uint64_t nq, uint64_t *d_offsets,
                                     uint32_t *d_ids, uint64_t ids_capacity, uint64_t *d_total, void *stream) {
    if (!t || (nq && !d_queries) || !d_offsets || !d_total || (ids_capacity && !d_ids))
        return fail(RT_EINVAL, "NULL argument");
    if (nq > 0xFFF00000ull) return fail(RT_EINVAL, "nq = %llu too large", (unsigned long long)nq);
    if ((reinterpret_cast<uintptr_t>(d_queries) & 15) != 0) return fail(RT_EINVAL, "queries not 16-byte aligned");
    if (t->device < 0 || t->device >= kPoolDevices) return fail(RT_EINVAL, "device %d out of range", t->device);
    try {
        DevSet ds(t->device);
        hipStream_t s = static_cast<hipStream_t>(stream);
        const int dev = t->device;
        // the count stage's part and room for its records, so that the fill
        // replays them instead of walking the tree again (50k windows on 1.2M
        // rectangles: fill 457 -> 45 us); whatever more the workspace has is used too
        const uint64_t ws0 = select_ws_bytes(nq, 0);
        PoolWs *w = nullptr, *w2 = nullptr;
        hipError_t e = pool_acquire(dev, ws0, select_rec_guess(t, nq, ids_capacity), &w);
        if (e != hipSuccess) return hip_fail(e, "select workspace");
        // hands both workspaces back behind everything enqueued so far (a
        // moved fill stage still replays the records of the first)
        auto done = [&](int rc) {
            pool_release(dev, w, s);
            pool_release(dev, w2, s);
            return rc;
        };
        w->host[0] = 0;
        int rc = enqueue_select_stage(t, reinterpret_cast<const float4 *>(d_queries), nq, d_offsets, nullptr, 0,
                                      w->d, nullptr, s, 1, nullptr, nullptr, w->bytes - ws0, w->host);
        if (rc == RT_OK) {
            e = hipStreamSynchronize(s);
            if (e != hipSuccess) rc = hip_fail(e, "count stage");
        }
        if (rc != RT_OK) return done(rc);
        const uint64_t total = w->host[0];
        if (total > ids_capacity) {
            e = hipMemcpyAsync(d_total, d_offsets + nq, 8, hipMemcpyDeviceToDevice, s);
            if (e == hipSuccess) e = hipStreamSynchronize(s);
            if (e != hipSuccess) return done(hip_fail(e, "count stage"));
            return done(fail(RT_ENOMEM, "the result has %llu ids, the buffer holds %llu", (unsigned long long)total,
                             (unsigned long long)ids_capacity));
        }
        const uint64_t need = select_ws_bytes(nq, total) + 256;   // and the status words
        void *work = w->d;
        uint64_t end = w->bytes;
        if (w->bytes < need) {
            // the sort needs more scratch than this workspace has: move the
            // count stage's part (order, split plan) into a larger one
            e = pool_acquire(dev, need, 0, &w2);
            if (e == hipSuccess) e = hipMemcpyAsync(w2->d, w->d, ws0, hipMemcpyDeviceToDevice, s);
            if (e != hipSuccess) return done(hip_fail(e, "select workspace"));
            work = w2->d;
            end = w2->bytes;
        }
        uint64_t *st = reinterpret_cast<uint64_t *>(static_cast<uint8_t *>(work) + (end - 256) / 256 * 256);
        rc = enqueue_select_stage(t, reinterpret_cast<const float4 *>(d_queries), nq, d_offsets, d_ids, total, work,
                                  st, s, 2, nullptr, nullptr);
        if (rc == RT_OK) {
            hipLaunchKernelGGL(total_word, dim3(1), dim3(1), 0, s, st, d_total);
            e = hipGetLastError();
            if (e != hipSuccess) rc = hip_fail(e, "fill stage");
        }
        return done(rc);
    } catch (const std::bad_alloc &) {
        return fail(RT_ENOMEM, "host allocation failed");
    } catch (...) {
        return fail(RT_EDEVICE, "unexpected failure");
    }
}
