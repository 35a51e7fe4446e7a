"""Repeated joins, whose levels run in one pass each, against the brute-force
oracle: node widths around the packing limits, more hits than a block collects,
pairs that crowd one bucket or sub-bucket of the sort, results that outgrow
what an earlier join left, and capacities below the result."""

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rt():
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    import paper_2309_16913_amd as m
    return m


@pytest.fixture(scope="module")
def ora():
    return oracle.get()


def boxes(n, side, seed):
    g = np.random.default_rng(seed)
    lo = g.random((n, 2), np.float32) - np.float32(0.5)
    return np.concatenate([lo, lo + g.random((n, 2), np.float32) * np.float32(side)], axis=1)


def device_join(rt, a, b, cap):
    import torch
    out = torch.full((2 * cap + 3,), -1, dtype=torch.int32, device="cuda")
    n = rt.spatial_join_device(a, b, out.data_ptr() + 4, cap, stream=torch.cuda.current_stream().cuda_stream)
    return n, out.cpu().numpy().view(np.uint32)


def check(rt, ta, tb, want):
    for _ in range(4):   # level by level, one pass per level, as a graph, again
        got = rt.spatial_join(ta, tb)
        assert np.array_equal(got, want)
    for cap in [want.shape[0], want.shape[0] + 5, max(want.shape[0] - 1, 0)]:
        for _ in range(3):
            n, out = device_join(rt, ta, tb, cap)
            assert n == want.shape[0]
            if n <= cap:   # at a word that is no multiple of the pairs' size
                assert np.array_equal(out[1:1 + 2 * n].reshape(n, 2), want)
                assert (out[1 + 2 * n:] == 0xFFFFFFFF).all() and out[0] == 0xFFFFFFFF
            else:
                assert (out == 0xFFFFFFFF).all()


@pytest.mark.parametrize("sort_lx", [False, True])
@pytest.mark.parametrize("fa,fb", [(2, 2), (3, 64), (16, 16), (31, 32), (32, 32), (32, 33), (33, 20), (63, 64), (64, 64)])
@pytest.mark.parametrize("na,nb,side", [(1, 1, 2.0), (70, 4000, 0.05), (5000, 6000, 0.02)])
def test_node_widths(rt, ora, fa, fb, na, nb, side, sort_lx):
    print(f"case once widths fa={fa} fb={fb} n={na},{nb} side={side} sort_lx={sort_lx}", flush=True)
    A, B = boxes(na, side, na + fa), boxes(nb, side, nb + fb)
    check(rt, rt.build_str(A, fa, "soa", sort_lx=sort_lx), rt.build_str(B, fb, "aos", sort_lx=sort_lx),
          ora.brute_join(A, B))


@pytest.mark.parametrize("fanout", [16, 32, 64])
def test_all_pairs(rt, ora, fanout):
    """Everything meets everything: every node pair keeps all its entries and a
    block's hits outgrow its list."""
    A, B = boxes(1500, 3.0, 1), boxes(900, 3.0, 2)
    A[:, :2], B[:, :2] = A[:, :2] - 3, B[:, :2] - 3
    A[:, 2:], B[:, 2:] = A[:, 2:] + 3, B[:, 2:] + 3
    print(f"case once all pairs F={fanout}", flush=True)
    want = ora.brute_join(A, B)
    assert want.shape[0] == 1500 * 900
    check(rt, rt.build_str(A, fanout, "d2"), rt.build_str(B, fanout, "soa"), want)


@pytest.mark.parametrize("big", [1, 3, 40])
def test_crowded_buckets(rt, ora, big):
    """A few large objects meet all of B, the others hardly any: the sort's
    buckets hold from none to more pairs than its LDS."""
    A, B = boxes(3000, 1e-4, 3), boxes(9000, 1e-4, 4)
    A[100:100 + big] = [-1, -1, 1, 1]
    print(f"case once crowded big={big}", flush=True)
    check(rt, rt.build_str(A, 32, "soa"), rt.build_str(B, 32, "soa"), ora.brute_join(A, B))


def test_growing_results(rt, ora):
    """Joins of the same heights one after the other whose levels and results
    outgrow the sizes that the one before left, and shrink again."""
    trees = []
    for n, side in [(4000, 0.001), (4000, 0.05), (3900, 0.3), (4050, 0.0)]:
        A, B = boxes(n, side, n), boxes(n, side, n + 1)
        trees.append((rt.build_str(A, 16, "soa"), rt.build_str(B, 16, "soa"), ora.brute_join(A, B)))
    for i in [0, 0, 1, 0, 2, 2, 2, 1, 3, 3, 0, 2]:
        a, b, want = trees[i]
        print(f"case once growing {i}", flush=True)
        assert np.array_equal(rt.spatial_join(a, b), want)
