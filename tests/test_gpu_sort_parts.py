"""Results longer than a block's sort, cut into parts of 16384 ids: lengths at
the edges of one, two, eight and nine parts, several segments sharing one list
of parts, next to skewed segments that the parts are skipped for, with the
capacity (and with it the scratch) exactly the result's, through both ways a
batch is classified and with id ranges per segment (several trees)."""

import numpy as np
import pytest

import oracle
import rtgen
from test_gpu_walk import device_select

pytestmark = pytest.mark.gpu

LENGTHS = [32768, 32769, 49152, 49153, 131072, 131073, 147456, 147457, 700_001]


@pytest.fixture(scope="module")
def rt():
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    import paper_2309_16913_amd as m
    return m


def line(n, seed=None):
    x = np.arange(n, dtype=np.float32)
    r = np.stack([x, np.zeros(n, np.float32), x, np.zeros(n, np.float32)], axis=1)
    return r if seed is None else rtgen.permute(r, seed)


def windows(n, lengths, seed):
    g = np.random.default_rng(seed)
    a = [int(g.integers(0, n - c + 1)) for c in lengths]
    return np.array([[i - 0.5, -1.0, i + c - 0.5, 1.0] for i, c in zip(a, lengths)], np.float32)


@pytest.mark.parametrize("few", [True, False])
@pytest.mark.parametrize("permuted", [True, False])
def test_part_edges(rt, few, permuted):
    n = 700_001
    r = line(n, 5 if permuted else None)
    lengths = LENGTHS + ([] if few else [int(c) for c in np.random.default_rng(6).integers(0, 40, 2100)] + [33_000] * 9)
    q = windows(n, lengths, 7)
    want = oracle.get().select(oracle.get().build_str(r, 32), q)
    assert np.array_equal(np.diff(want[0].astype(np.int64)), lengths)
    print(f"case part edges few={few} permuted={permuted} nq={len(lengths)} ids={want[1].size}", flush=True)
    t = rt.build_str(r, 32, "soa")
    off, ids = device_select(rt, t, q, int(want[1].size))
    assert np.array_equal(off, want[0].astype(np.int64))
    assert np.array_equal(ids, want[1])


def test_parts_of_several_trees(rt):
    sizes = [40_000, 200_000, 70_000]
    rs = [line(n, 11 + i) for i, n in enumerate(sizes)]
    qs = [windows(n, [n, 33_000, 100, 39_000], 21 + i) for i, n in enumerate(sizes)]
    print("case parts of several trees", flush=True)
    trees = [rt.build_str(r, 16, "aos") for r in rs]
    b = rt.Batch(trees, qs)
    b.run()
    for i in range(len(sizes)):
        want = oracle.get().select(oracle.get().build_str(rs[i], 16), qs[i])
        off, ids = b.result(i)
        assert np.array_equal(np.asarray(off).astype(np.int64), want[0].astype(np.int64))
        assert np.array_equal(ids, want[1])


@pytest.mark.parametrize("few", [True, False])
@pytest.mark.parametrize("length", [300, 1000, 1024, 1500, 4096, 12_000, 30_000, 40_000])
def test_bucket_lengths(rt, few, length):
    """Results that are one run of consecutive ids, in random spatial order, of
    1 / ratio of the id range: the sort's buckets then hold 1 to about 260 ids,
    which takes from none to all rounds of the in-bucket merging, and beyond
    its limit the bitonic fallback."""
    for ratio in [1, 2, 3, 5, 8, 16, 40, 63, 64, 65]:
        n = length * ratio
        i = np.arange(n)
        x = (i // length).astype(np.float32)
        y = np.random.default_rng(length + ratio).permutation(n).astype(np.float32)
        r = np.stack([x, y, x, y], axis=1)
        at = sorted({0, ratio // 2, ratio - 1})
        q = [[j - 0.25, -1.0, j + 0.25, float(n)] for j in at]
        if not few:
            q += [[-9.0, -9.0, -8.0, -8.0]] * 2100
        q = np.array(q, np.float32)
        print(f"case bucket lengths few={few} length={length} ratio={ratio}", flush=True)
        t = rt.build_str(r, 64, "soa")
        off, ids = device_select(rt, t, q, length * len(at))
        assert np.array_equal(off[: len(at) + 1], np.arange(len(at) + 1) * length)
        for k, j in enumerate(at):
            assert np.array_equal(ids[k * length:(k + 1) * length], np.arange(j * length, (j + 1) * length)), ratio
        t.free()
