"""An arena filled from both ends: the replay's waves take every record of the
chunks and of the tail exactly once, and nothing else, up to a tail that meets
the chunks.  The kernel's own arithmetic, compiled for the host."""

import os
import subprocess

from test_replay_units_cpu import CSRC

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "replay_units.h"
using namespace rtk;
int main() {
    for (uint32_t nchunks = 1; nchunks <= 7; ++nchunks)
        for (uint32_t taken = 0; taken <= nchunks; ++taken) {
            const uint32_t limit = tail_limit(taken, nchunks);
            if (limit != (nchunks - taken) * kRecChunk) return std::puts("limit"), 1;
            for (uint32_t tail : {0u, 1u, 63u, 64u, 65u, 255u, 256u, 257u, 700u, limit})
                for (uint32_t step : {1u, 4u, 12u}) {
                    if (tail > limit) continue;
                    const uint64_t nrec = (uint64_t)nchunks * kRecChunk;
                    const uint32_t nunits = units_of(taken, tail);
                    std::vector<uint32_t> count(taken), times(nrec, 0);
                    for (uint32_t c = 0; c < taken; ++c) count[c] = (c * 97 + 5) % (kRecChunk + 1);
                    for (uint32_t first = 0; first < step && first < nunits; ++first)
                        for (uint32_t u = first;; u += step) {
                            const uint32_t v = unit_loaded(u, nunits), c = v / kChunkUnits;
                            const uint32_t n = c < taken ? count[c] : tail_count(c, taken, tail);
                            for (uint32_t lane = 0; lane < kUnitRecs; ++lane) {
                                const uint64_t at = unit_place(v, lane, taken, nrec);
                                if (at >= nrec) return std::puts("read outside the arena"), 1;
                                if (unit_has(u, nunits, lane, n)) times[at] += 1;
                            }
                            if (u >= nunits) break;
                        }
                    for (uint64_t i = 0; i < nrec; ++i) {
                        const bool there = i < (uint64_t)taken * kRecChunk ? i % kRecChunk < count[i / kRecChunk]
                                                                          : nrec - 1 - i < tail;
                        if (times[i] != (there ? 1u : 0u))
                            return std::printf("place %u of %u, %u taken, tail %u: %u times\n", (unsigned)i, (unsigned)nrec, taken, tail, times[i]), 1;
                    }
                }
        }
    if (tail_limit(9, 4) != 0 || tail_limit(0, 0xFFFFFFF0u) != 0xF0000000u) return std::puts("limit at the ends"), 1;
    return 0;
}
"""


def test_both_ends(tmp_path):
    (tmp_path / "tail.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC, str(tmp_path / "tail.cpp"), "-o",
                    str(tmp_path / "tail")], check=True)
    r = subprocess.run([str(tmp_path / "tail")], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
