"""The memory that the library keeps between calls, compiled for the host
against a stand-in for the HIP allocator (a card of a given size, streams whose
work ends when the program says so): what is kept is bounded, never in use by
the device when it is freed or handed out, and back on the device before any
allocation of the library fails."""

import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2309_16913_amd", "csrc")

HEAD = r"""
#include <hip/hip_runtime_api.h>
#include <cstdio>
#include <cstdlib>
#include <map>
#include <set>
#include <vector>
#include "dev_pool.h"
using namespace rtk;
static uint64_t card = 0, used = 0;
static uintptr_t next_at = 1 << 20;
static std::map<void *, uint64_t> mem;          // device allocations
static std::map<void *, uint64_t> busy;         // event -> work it waits for (0: none)
static uint64_t queued = 0, finished = 0;       // one queue of work, in order
static int mallocs = 0;
#define CHECK(c) do { if (!(c)) { std::printf("line %d: %s\n", __LINE__, #c); std::exit(1); } } while (0)
extern "C" {
hipError_t hipMalloc(void **p, size_t n) {
    mallocs += 1;
    if (used + n > card) return hipErrorOutOfMemory;
    *p = reinterpret_cast<void *>(next_at);
    next_at += (n + 4095) / 4096 * 4096 + 4096;
    mem[*p] = n;
    used += n;
    return hipSuccess;
}
hipError_t hipFree(void *p) {
    if (!p) return hipSuccess;
    CHECK(mem.count(p));
    used -= mem[p];
    mem.erase(p);
    return hipSuccess;
}
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = std::malloc(n); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { *e = reinterpret_cast<hipEvent_t>(std::malloc(1)); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) { busy[e] = queued; return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t e) { return busy[e] <= finished ? hipSuccess : hipErrorNotReady; }
hipError_t hipDeviceSynchronize(void) { finished = queued; return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
}
constexpr uint64_t MiB = 1 << 20, GiB = 1 << 30;
static PoolWs *take(uint64_t n) { PoolWs *w = nullptr; CHECK(pool_acquire(0, n, 0, &w) == hipSuccess); CHECK(w->bytes >= n && mem.at(w->d) == w->bytes); return w; }
"""

PROGRAMS = {
    # an allocation that would fit without what is kept succeeds: blocks of
    # freed trees, workspaces of builds and selects
    "given_back": r"""
int main() {
    card = 4 * GiB;
    void *t[4];
    uint64_t got[4];
    for (int i = 0; i < 4; ++i) CHECK(block_alloc(0, 256 * MiB, &t[i], &got[i]) == hipSuccess);
    for (int i = 0; i < 4; ++i) block_free(0, t[i], got[i]);
    PoolWs *a = take(500 * MiB), *b = take(900 * MiB);
    pool_release(0, a, nullptr);
    pool_release(0, b, nullptr);
    CHECK(used > 2 * GiB);
    void *p = nullptr;
    CHECK(dev_malloc(0, &p, 4 * GiB) == hipSuccess && used == 4 * GiB);
    CHECK(hipFree(p) == hipSuccess);
    // and the workspaces still serve
    a = take(10 * MiB), b = take(20 * MiB);
    CHECK(a != b && a->d != b->d);
    // one whose work is under way is not taken back
    queued += 1;
    pool_release(0, a, nullptr);
    void *was = a->d;
    CHECK(dev_malloc(0, &p, 4 * GiB) == hipErrorOutOfMemory);
    CHECK(a->d == was && mem.count(was));
    return 0;
}
""",
    # workspaces that calls of every size leave are bounded together, but the
    # one released last is kept whatever its size: the next call reuses it
    "bounded": r"""
int main() {
    card = 100 * GiB;
    std::vector<PoolWs *> w;
    for (int i = 1; i <= 12; ++i) w.push_back(take(i * GiB));
    for (PoolWs *x : w) pool_release(0, x, nullptr);
    CHECK(used <= kIdleMax || (used == w.back()->bytes));
    PoolWs *big = take(20 * GiB);
    void *d = big->d;
    pool_release(0, big, nullptr);
    for (int i = 0; i < 5; ++i) {
        const int m = mallocs;
        PoolWs *x = take(20 * GiB);
        CHECK(mallocs == m && x->d == d);
        pool_release(0, x, nullptr);
    }
    // those in use by the device stay until it is done with them
    queued += 1;
    PoolWs *x = take(6 * GiB), *y = take(7 * GiB);
    pool_release(0, x, nullptr);
    pool_release(0, y, nullptr);
    CHECK(x->bytes && y->bytes);
    finished = queued;
    PoolWs *z = take(1 * MiB);
    pool_release(0, z, nullptr);
    uint64_t sum = 0;
    for (auto &m : mem) sum += m.second;
    CHECK(sum <= kIdleMax);
    return 0;
}
""",
    # growth takes more than is asked for only where that is little or there
    # is room
    "growth": r"""
int main() {
    card = 10 * GiB;
    PoolWs *a = take(9 * GiB);
    CHECK(a->bytes <= 9 * GiB + 256 * MiB);
    pool_release(0, a, nullptr);
    a = take(10 * GiB);
    CHECK(a->bytes == 10 * GiB);
    PoolWs *b = nullptr;
    CHECK(pool_acquire(0, 1 * MiB, 0, &b) == hipErrorOutOfMemory && !b);
    pool_release(0, a, nullptr);
    b = take(1 * MiB);
    return 0;
}
""",
}


@pytest.mark.parametrize("name", sorted(PROGRAMS))
def test_pool(name, tmp_path):
    src, exe = tmp_path / "pool.cpp", tmp_path / "pool"
    src.write_text(HEAD + PROGRAMS[name])
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include", "-I", CSRC,
                    str(src), os.path.join(CSRC, "dev_pool.cpp"), "-o", str(exe), "-pthread"], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout
