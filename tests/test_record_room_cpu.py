"""The room that a host or stream-ordered select asks for its records is only
worth having: a call on a card without that much goes on with the rest, and it
stays within a constant of what the call needs, however many windows it has.
The library's own code, compiled for the host."""

import os
import subprocess

import pytest

from test_dev_pool_cpu import CSRC, HEAD

PROGRAMS = {
    # 200M windows need 43 GB; room for their records would not fit the card
    "asked_for": r"""
#include "rec_space.h"
int main() {
    for (bool shared : {false, true})
    for (uint32_t width : {16u, 32u, 64u})
        for (uint64_t nq = 1; nq <= 4000000000ull; nq = nq * 3 + 1)
            for (uint64_t cap : {(uint64_t)0, (uint64_t)1000, (uint64_t)1 << 20, (uint64_t)1 << 34, ~(uint64_t)0}) {
                const uint64_t b = rec_arena_guess(256, width, shared, nq, cap);
                CHECK(b <= (1ull << 30));
                CHECK(rec_chunks_in(b) >= 1);
                // small calls get what cannot run out
                if (cap <= 65536 && nq <= 16384) CHECK(rec_chunks_in(b) >= rec_chunks_sure(nq, cap));
            }
    return 0;
}
""",
    "done_without": r"""
int main() {
    card = 2 * GiB;
    void *rest = nullptr;
    CHECK(dev_malloc(0, &rest, 1 * GiB) == hipSuccess);
    PoolWs *w = nullptr;
    CHECK(pool_acquire(0, 300 * MiB, 800 * MiB, &w) == hipSuccess && w->bytes >= 300 * MiB);
    pool_release(0, w, nullptr);
    CHECK(pool_acquire(0, 300 * MiB, 700 * MiB, &w) == hipSuccess && w->bytes >= 1000 * MiB);
    pool_release(0, w, nullptr);
    CHECK(pool_acquire(0, 1100 * MiB, 0, &w) == hipErrorOutOfMemory);
    CHECK(pool_acquire(0, 1 * GiB, 5 * GiB, &w) == hipSuccess && w->bytes == 1 * GiB);
    return 0;
}
""",
}


@pytest.mark.parametrize("name", sorted(PROGRAMS))
def test_records_are_optional(name, tmp_path):
    src, exe = tmp_path / "room.cpp", tmp_path / "room"
    src.write_text(HEAD + PROGRAMS[name])
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", CSRC,
                    str(src), os.path.join(CSRC, "dev_pool.cpp"), "-o", str(exe), "-pthread"], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
