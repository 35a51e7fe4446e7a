"""The device STR build's level sorts at their edges: levels built in one
block, by counting, by buckets and slices, and by radix sorts after skewed
x-centers, each against the STR rules entry by entry (tests/str_shape.py)."""

import numpy as np
import pytest

import rtgen
from str_shape import assert_export_equal, expected_export

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rt():
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    import paper_2309_16913_amd as m
    return m


def _one_column(n):
    """Every x-center alike: one bucket holds all items."""
    r = rtgen.uniform_rects(n, 1e-3, 71)
    r[:, 0], r[:, 2] = 0.25, 0.75
    return r


def _columns(n, k):
    """k distinct x-centers (straddling buckets of n / k items), many equal
    y-centers."""
    g = rtgen.rng(72)
    x = np.floor(g.random(n) * k).astype(np.float32) / np.float32(k)
    y = np.floor(g.random(n) * 50).astype(np.float32) / np.float32(64)
    return np.stack([x, y, x + np.float32(0.125), y + np.float32(0.125)], 1).astype(np.float32)


def _infinite(n):
    """A share of half-infinite and whole-line items (infinite and NaN centers)."""
    r = rtgen.c2_rects(n)
    inf = np.float32(np.inf)
    r[::7, 0] = -inf
    r[::11, 2] = inf
    r[::13, 1], r[::13, 3] = -inf, inf
    return r


CASES = [
    ("top-1024", lambda: rtgen.c2_rects(1024), 2), ("top-1025", lambda: rtgen.c2_rects(1025), 3),
    ("count-16384", lambda: rtgen.c2_rects(16384), 16), ("bucket-16385", lambda: rtgen.c2_rects(16385), 64),
    ("two-bucket-levels", lambda: rtgen.c2_rects(150_001), 5), ("binary", lambda: rtgen.c2_rects(40_000), 2),
    ("one-column", lambda: _one_column(60_000), 32), ("columns", lambda: _columns(70_000, 40), 33),
    ("few-columns", lambda: _columns(70_000, 5), 16), ("infinite", lambda: _infinite(50_000), 20),
    ("wide-grid", lambda: rtgen.c2_rects(2_200_000), 63), ("outlier", lambda: np.concatenate(
        [rtgen.uniform_rects(90_000, 1e-4, 73), np.array([[3e5, 0, 3e5, 0]], np.float32)]), 32),
]


@pytest.mark.parametrize("sort_lx", [False, True])
@pytest.mark.parametrize("name,rects,fanout", CASES, ids=[c[0] for c in CASES])
def test_build_levels(rt, name, rects, fanout, sort_lx):
    r = rects()
    print(f"case build {name} n={r.shape[0]} F={fanout} sort_lx={sort_lx}", flush=True)
    want = expected_export(r, fanout, sort_lx)
    layout = {0: "soa", 1: "aos", 2: "d2"}[fanout % 3]
    for _ in range(2):   # the second build takes over the first one's memory
        t = rt.build_str(r, fanout, layout, sort_lx=sort_lx)
        assert_export_equal(t.export(), want, name)
        q = rtgen.windows_loguniform(50, 1e-4, 1e-1, 74)
        off, ids = rt.range_select(t, np.concatenate([q, np.array([[-np.inf] * 2 + [np.inf] * 2], np.float32)]))
        assert np.array_equal(ids[int(off[-2]):], np.arange(r.shape[0], dtype=np.uint32))
        t.free()
