// How much room the records of a count pass are given.  Plain arithmetic
// without device types, so that the host can check it.
#pragma once

#include <algorithm>
#include <cstdint>

#include "replay_units.h"

namespace rtk {

// records a lane group collects in LDS before storing them (128 measured no
// faster for groups of 64 lanes)
constexpr uint32_t kRecBuf = 64;

// Lane groups of `width` lanes that run at once on `cus` CUs.
constexpr uint64_t resident_groups(uint32_t cus, uint32_t width) { return (uint64_t)cus * 8 * (256 / width); }

// The record arena: chunks of kRecChunk 16-byte records (the items of a shared
// walk fill it from its end instead, see replay_units.h), then one count per
// chunk.  Sized for cap / 16 + 16 nq records (leaf visits with hits and
// contained subtrees: about cap / 64 at 10M rectangles / 1M windows, fanout
// 64), a third more for chunks closed early (a node's records never straddle
// two chunks), and a chunk for every window or every lane group that can run at
// once (of the narrowest, 16 lanes), whichever is less, as each may end the pass
// with a partly used one; a count pass that needs more sets the overflow flag
// and the fill walks the tree instead.  (10 to 10k windows of 1e-6 to 1e-4 ..
// 1e-2 of the space, shared, on 0.2M to 50M rectangles at fanouts 16 to 64 take
// 7% to 90% of it.)
// Small results get the chunks that cannot run out: a record has at least one
// id, a chunk is closed with at most kRecBuf - 1 records free, and each
// window's group may hold a partly used one.
constexpr uint64_t rec_chunks_sure(uint64_t nq, uint64_t cap) { return cap / (kRecChunk - kRecBuf + 1) + nq + 1; }
constexpr uint64_t kRecSureIds = 65536;

inline uint64_t rec_arena_bytes(uint32_t cus, uint64_t nq, uint64_t cap) {
    const uint64_t recs = (cap / 16 + 16 * nq) * 4 / 3, groups = resident_groups(cus, 16);
    uint64_t chunks = (recs + kRecChunk - 1) / kRecChunk + std::min(nq, groups);
    if (cap <= kRecSureIds && nq <= groups) chunks = std::max(chunks, rec_chunks_sure(nq, cap));
    const auto align256 = [](uint64_t b) { return (b + 255) & ~255ull; };
    return align256(16 * kRecChunk * chunks) + align256(4 * chunks) + 512;
}

// The same for selects whose result, of at most cap ids, is not known yet, on a
// tree of groups of `width` lanes: up to 512 ids per window on average, 2048
// where large windows are expected (shared), and a chunk for every lane group of
// that width that can run at once.  Records are only worth having, so never more
// than 1 GiB.
constexpr uint64_t kRecGuessMax = 1ull << 30;
inline uint64_t rec_arena_guess(uint32_t cus, uint32_t width, bool shared, uint64_t nq, uint64_t cap) {
    const uint64_t ids = std::min<uint64_t>(cap, (shared ? 2048 : 512) * nq + 65536);
    const uint64_t all = rec_arena_bytes(cus, nq, ids);
    // rec_arena_bytes counts the groups of the narrowest trees
    const uint64_t less =
        (std::min(nq, resident_groups(cus, 16)) - std::min(nq, resident_groups(cus, width))) * (16ull * kRecChunk);
    return std::min(ids <= kRecSureIds ? all : all - less, kRecGuessMax);
}

// Chunks of an arena of `bytes` bytes.
constexpr uint32_t rec_chunks_in(uint64_t bytes) {
    const uint64_t per = 16 * kRecChunk + 4, c = bytes > 512 ? (bytes - 512) / per : 0;
    return (uint32_t)(c < 0xFFFFFFF0ull ? c : 0xFFFFFFF0ull);
}

}  // namespace rtk
