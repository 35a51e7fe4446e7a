// Sort of the join's pair keys ((idA << 32) | idB, all distinct) by their top
// digit: the keys are split into kPairBuckets buckets by key >> shift (the
// bucket order is the key order), and every bucket is then sorted on its own
// in LDS (a bucket over the LDS cap in runs, merged through global memory).
// Four launches where an LSD radix sort of two 21-bit ids needs four passes
// of five.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace rtk {

constexpr uint32_t kPairBuckets = 2048;      // 11-bit top digit
constexpr uint32_t kPairBucketCap = 4096;    // keys a bucket may hold to be sorted in LDS

// Workspace (uint32 words) of launch_pair_bucket_sort: counts, starts and
// cursors.
constexpr uint64_t kPairSortWords = 3 * kPairBuckets + 8;

// What a replayed join's sort reads from and leaves on the device.
struct Ctrl;
struct PairsOut {
    const uint64_t *n_dev = nullptr;   // the key count (at most n)
    uint64_t capacity = 0;             // (a, b) words are written to pairs if it fits this
    const uint32_t *skip = nullptr;    // and bit 0 here is clear
    uint32_t *pairs = nullptr;         // may be the keys' own buffer
    const Ctrl *ctrl = nullptr;        // ctrl->err is copied to err_out
    uint32_t *err_out = nullptr;
};

// keys (n) -> out (n), sorted; keys is overwritten (merge space for buckets
// over the LDS cap).  shift: every key is below 2^(shift + 11).  ws:
// kPairSortWords uint32.  po (if not NULL): the count is on the device (n then
// only sizes the grids), ws holds zeroed bucket counts, and the result are (a,
// b) words (out is left unsorted).
hipError_t launch_pair_bucket_sort(uint64_t *keys, uint64_t n, int shift, uint64_t *out, uint32_t *ws,
                                   hipStream_t s, const PairsOut *po = nullptr);

// Join status for a single read: *dst = ctrl->err (one thread).
hipError_t launch_copy_err(const Ctrl *ctrl, uint32_t *dst, hipStream_t s);

}  // namespace rtk
