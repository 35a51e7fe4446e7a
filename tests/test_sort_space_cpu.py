"""The segmented sort's work space behind the ids of its scratch: at whatever
id the scratch begins (a plain batch run sorts every tree's results in a piece
of one scratch), the parts lie at a multiple of 16 bytes, nothing overlaps and
nothing passes the scratch's size.  The library's own arithmetic, compiled for
the host."""

import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2309_16913_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "sort_space.h"
using namespace rtk;
int main() {
    const uint64_t caps[] = {0, 1, 2, 3, 5, 16383, 16384, 16385, 32767, 32768, 32769, 49153, 65536, 65537, 65538, 65539,
                             98307, 1000001, 7723880, 1443956528, 40000000003ull};
    for (uint64_t cap : caps)
        for (uint64_t scratch = 1 << 20; scratch < (1 << 20) + 64; scratch += 4) {
            const LongSpace s = long_space(scratch, cap);
            if ((scratch + 4 * s.parts) % 16) return std::printf("parts of %llu ids at %llu\n", (unsigned long long)cap, (unsigned long long)scratch), 1;
            if (s.parts < cap || s.desc < s.parts + 4 * most_parts(cap) || s.sub < s.desc + kDesc * most_long(cap) ||
                s.end < s.sub + kLongDigits * most_long(cap))
                return std::puts("overlap"), 1;
            if (s.end > sort_scratch_words(cap)) return std::printf("past the scratch: %llu ids\n", (unsigned long long)cap), 1;
        }
    return 0;
}
"""


def test_work_space(tmp_path):
    (tmp_path / "space.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", CSRC, str(tmp_path / "space.cpp"), "-o",
                    str(tmp_path / "space")], check=True)
    r = subprocess.run([str(tmp_path / "space")], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
