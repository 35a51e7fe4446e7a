// Which records a wave of the replay reads: work units of 64 records, one per
// lane.  Plain arithmetic without device types, so that the host can check it.
#pragma once

#include <cstdint>

namespace rtk {

constexpr uint32_t kRecChunk = 256;          // records per chunk a lane group takes
constexpr uint32_t kUnitRecs = 64;           // records per unit: a quarter of a chunk
constexpr uint32_t kChunkUnits = kRecChunk / kUnitRecs;

// The unit whose records are loaded for unit u: a wave reads one unit ahead,
// past the last one the last one again.  nunits > 0.
constexpr uint32_t unit_loaded(uint32_t u, uint32_t nunits) { return u < nunits ? u : nunits - 1; }

// Whether unit u holds a record for a lane: count is that of the chunk of
// unit_loaded(u).  A unit past the last one has none, whatever was loaded.
constexpr bool unit_has(uint32_t u, uint32_t nunits, uint32_t lane, uint32_t count) {
    return u < nunits && (u % kChunkUnits) * kUnitRecs + lane < (count < kRecChunk ? count : kRecChunk);
}

}  // namespace rtk
