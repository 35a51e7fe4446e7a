"""Which records the replay's waves take: every record of every chunk exactly
once, and never a place behind a chunk's records, also in the units that are
read ahead past the last one (whose place there is of another quarter).  The
kernel's own arithmetic, compiled for the host."""

import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2309_16913_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "replay_units.h"
using namespace rtk;
int main() {
    for (uint32_t nchunks = 1; nchunks <= 9; ++nchunks)
        for (uint32_t last : {0u, 1u, 63u, 64u, 65u, 191u, 192u, 255u, 256u, 300u})
            for (uint32_t step : {1u, 4u, 8u, 12u, 64u}) {
                std::vector<uint32_t> count(nchunks, kRecChunk), taken(nchunks * kRecChunk, 0);
                count[nchunks - 1] = last;
                const uint32_t nunits = nchunks * kChunkUnits;
                for (uint32_t first = 0; first < step && first < nunits; ++first)   // a wave each
                    for (uint32_t u = first;; u += step) {
                        const uint32_t v = unit_loaded(u, nunits), c = v / kChunkUnits;
                        for (uint32_t lane = 0; lane < kUnitRecs; ++lane) {
                            const uint32_t at = (v % kChunkUnits) * kUnitRecs + lane;
                            if (c >= nchunks || at >= kRecChunk) return std::puts("read outside the arena"), 1;
                            if (!unit_has(u, nunits, lane, count[c])) continue;
                            if (at >= count[c]) return std::printf("unit %u of %u takes record %u of %u\n", u, nunits, at, count[c]), 1;
                            taken[c * kRecChunk + at] += 1;
                        }
                        if (u >= nunits) break;   // one unit past the last is read ahead
                    }
                for (uint32_t c = 0; c < nchunks; ++c)
                    for (uint32_t i = 0; i < kRecChunk; ++i)
                        if (taken[c * kRecChunk + i] != (i < count[c] ? 1u : 0u)) return std::puts("not once"), 1;
            }
    return 0;
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("units")
    (d / "units.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC, str(d / "units.cpp"), "-o", str(d / "units")], check=True)
    return str(d / "units")


def test_units_take_written_records_only(program):
    r = subprocess.run([program], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
