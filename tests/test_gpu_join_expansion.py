"""The expansion that a join is asked for is the one that runs, on the first
call and on repeated ones (which replay their levels, the third from a graph);
only joins that leave it to the library run their levels in one pass.  The
kernels are those that torch's profiler saw.  Pairs against the oracle, with the
edges of the lower bound among the inputs."""

import numpy as np
import pytest

import oracle
import rtgen
from test_gpu_join_prune import _edge_rects

pytestmark = pytest.mark.gpu

TILE, CAND, ONCE = "join_level_kernel", "join_cand_kernel", "join_once_kernel"


@pytest.fixture(scope="module")
def rt():
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    import paper_2309_16913_amd as m
    return m


def kernels(call):
    """The join kernels that a call launched, and its result."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        got = call()
        torch.cuda.synchronize()
    names = [e.name for e in p.events()]
    return {k for k in (TILE, CAND, ONCE) if any(k in n for n in names)}, got


@pytest.mark.parametrize("fanout", [16, 32, 64])
def test_asked_for_expansion_runs(rt, fanout):
    O3, O4, O5, LB = rt.JOIN_O3, rt.JOIN_O4, rt.JOIN_O5, rt.JOIN_LB
    A, B = rtgen.uniform_rects(9_000, 4e-3, 1), rtgen.clustered_rects(8_000, 8, 0.05, 4e-3, 2)
    o = oracle.get()
    want = o.join(o.build_str(A, 32), o.build_str(B, 32))
    import torch
    buf = torch.empty(2 * want.shape[0], dtype=torch.int32, device="cuda")
    a, b = rt.build_str(A, fanout, "soa", sort_lx=True), rt.build_str(B, fanout, "soa", sort_lx=True)
    assert a.info().height == b.info().height
    for flags in (rt.JOIN_TILE, 0, O3, O4, O5, O3 | O4, O3 | O5, O3 | O5 | LB, None):
        print(f"case expansion F={fanout} flags={flags}", flush=True)
        for rep in range(4):
            ran, got = kernels(lambda: rt.spatial_join(a, b, flags))
            assert np.array_equal(got, want), (flags, rep)
            if flags is not None:
                assert ran == {TILE if flags == rt.JOIN_TILE else CAND}, (flags, rep, ran)
            elif rep:   # the sizes of the joins before may not fit the first
                assert ran == {ONCE}, (rep, ran)
        for rep in range(3):
            buf.fill_(7)
            ran, n = kernels(lambda: rt.spatial_join_device(a, b, buf.data_ptr(), want.shape[0], flags))
            assert n == want.shape[0] and np.array_equal(buf.cpu().numpy().view(np.uint32).reshape(-1, 2), want)
            assert ran == {ONCE if flags is None else TILE if flags == rt.JOIN_TILE else CAND}, (flags, rep, ran)


@pytest.mark.parametrize("n,F,seed", [(3_000, 8, 64), (20_000, 32, 65), (9_000, 64, 66)])
def test_lower_bound_edges_repeated(rt, n, F, seed):
    """Infinite extents, widths near the largest float, subnormals and pairs
    that touch exactly, through the first run and the replays of every pruning
    expansion."""
    A, B = _edge_rects(n, seed), _edge_rects(n // 2 + 1, seed + 1000)
    o = oracle.get()
    want = o.join(o.build_str(A, F), o.build_str(B, F))
    a, b = rt.build_str(A, F, "soa", sort_lx=True), rt.build_str(B, F, "aos", sort_lx=True)
    O3, O4, O5, LB = rt.JOIN_O3, rt.JOIN_O4, rt.JOIN_O5, rt.JOIN_LB
    for flags in (O3 | O5 | LB, O3 | O5, O3 | O4, O5, None):
        for rep in range(3):
            assert np.array_equal(rt.spatial_join(a, b, flags), want), (flags, rep)
