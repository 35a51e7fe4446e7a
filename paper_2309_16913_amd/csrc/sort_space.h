// Where the segmented sort keeps its lists of long (class-L) segments: behind
// the ids of its scratch.  Plain arithmetic without device types, so that the
// host can check it.
#pragma once

#include <cstdint>

namespace rtk {

constexpr uint32_t kMidMax = 32768;     // longest segment sorted by one block at once; longer ones are class L
constexpr uint32_t kPart = 16384;       // ids per part of a class-L segment
constexpr uint32_t kLongDigits = 256;
// descriptor of a class-L segment: its digit counts, which become the write
// cursors of its groups; the digits per group (0: the segment went to the
// fallback), its place in ids (two words), its id range
constexpr uint32_t kDescGroup = kLongDigits, kDescOff = kLongDigits + 1, kDescRange = kLongDigits + 3;
constexpr uint32_t kDesc = kLongDigits + 4;

// Class-L segments and parts that cap ids can hold at most.
constexpr uint64_t most_long(uint64_t cap) { return cap / (kMidMax + 1) + 1; }
constexpr uint64_t most_parts(uint64_t cap) { return cap / kPart + most_long(cap); }

// Words of scratch for cap ids: the ids, then for each possible class-L segment
// its descriptor and room for 256 groups, about three parts of four words and
// what aligns those: at most 540 words per segment.  The size is that of an
// earlier layout of 770, which keeps the sizes that a fixed scratch accepts.
constexpr uint64_t kLongWords = 770;
static_assert(4 * 4 + 3 + kDesc + kLongDigits <= kLongWords, "class-L work space");
constexpr uint64_t sort_scratch_words(uint64_t cap) { return cap + most_long(cap) * kLongWords; }

// Word offsets in the scratch at address `scratch` (a multiple of 4: a caller's
// scratch may begin at any id): parts (at a multiple of 16 bytes, as they are
// read as four words at once), descriptors, groups, end.
struct LongSpace {
    uint64_t parts, desc, sub, end;
};
constexpr LongSpace long_space(uint64_t scratch, uint64_t cap) {
    const uint64_t parts = ((scratch + 4 * cap + 15) / 16 * 16 - scratch) / 4;
    const uint64_t desc = parts + 4 * most_parts(cap), sub = desc + kDesc * most_long(cap);
    return LongSpace{parts, desc, sub, sub + kLongDigits * most_long(cap)};
}

}  // namespace rtk
