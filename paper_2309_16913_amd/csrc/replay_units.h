// Which records a wave of the replay reads: work units of 64 records, one per
// lane.  Plain arithmetic without device types, so that the host can check it.
//
// The arena is filled from both ends: chunks of kRecChunk records from the
// front, each with a count of its own, and from the back single records, the
// tail, record r of it at place nrec - 1 - r.  The tail's records count as
// further chunks behind the taken ones, all full but the last.
#pragma once

#include <cstdint>

namespace rtk {

constexpr uint32_t kRecChunk = 256;          // records per chunk a lane group takes
constexpr uint32_t kUnitRecs = 64;           // records per unit: a quarter of a chunk
constexpr uint32_t kChunkUnits = kRecChunk / kUnitRecs;

constexpr uint32_t units_of(uint32_t chunks, uint32_t tail) {
    return chunks * kChunkUnits + (tail + kUnitRecs - 1) / kUnitRecs;
}

// Records of chunk c behind the `chunks` taken ones.
constexpr uint32_t tail_count(uint32_t c, uint32_t chunks, uint32_t tail) {
    const uint64_t before = (uint64_t)(c - chunks) * kRecChunk;
    return tail <= before ? 0 : tail - before < kRecChunk ? (uint32_t)(tail - before) : kRecChunk;
}

// Place in the arena of nrec records of a lane's record of unit v.
constexpr uint64_t unit_place(uint32_t v, uint32_t lane, uint32_t chunks, uint64_t nrec) {
    const uint64_t at = (uint64_t)v * kUnitRecs + lane, front = (uint64_t)chunks * kRecChunk;
    return at < front ? at : nrec - 1 - (at - front);
}

// Records that the tail may have: those of the chunks that are not taken.
constexpr uint32_t tail_limit(uint32_t taken, uint32_t nchunks) {
    const uint64_t r = taken < nchunks ? (uint64_t)(nchunks - taken) * kRecChunk : 0;
    return r < 0xF0000000u ? (uint32_t)r : 0xF0000000u;
}

// The unit whose records are loaded for unit u: a wave reads one unit ahead,
// past the last one the last one again.  nunits > 0.
constexpr uint32_t unit_loaded(uint32_t u, uint32_t nunits) { return u < nunits ? u : nunits - 1; }

// Whether unit u holds a record for a lane: count is that of the chunk of
// unit_loaded(u), of a taken one or of one in the tail.  A unit past the last one has none, whatever was loaded.
constexpr bool unit_has(uint32_t u, uint32_t nunits, uint32_t lane, uint32_t count) {
    return u < nunits && (u % kChunkUnits) * kUnitRecs + lane < (count < kRecChunk ? count : kRecChunk);
}

}  // namespace rtk
