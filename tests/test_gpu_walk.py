"""The batched count walk at its edges, against the CPU oracle: trees of every
lane-group width with partly filled groups, grids whose windows are all handed
out by place or several per counter update, large windows that hand their
remaining subtrees to further launches, item lists that fill up, and leaf
ranges deferred by the replay."""

import numpy as np
import pytest

import oracle
import rtgen

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


def device_select(rt, t, q, cap, replay=True):
    import torch
    nq = q.shape[0]
    dq = torch.from_numpy(q).cuda()
    off = torch.empty(nq + 1, dtype=torch.int64, device="cuda")
    ids = torch.full((max(cap, 1),), -1, dtype=torch.int32, device="cuda")
    wb = (rt.select_replay_workspace_bytes if replay else rt.select_workspace_bytes)(nq, cap)
    w = torch.empty(wb, dtype=torch.uint8, device="cuda")
    st = torch.zeros(2, dtype=torch.int64, device="cuda")
    rt.range_select_device(t, dq.data_ptr(), nq, off.data_ptr(), ids.data_ptr(), cap, w.data_ptr(), wb,
                           st.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert st.cpu().tolist() == [cap, 0]
    return off.cpu().numpy(), ids[:cap].cpu().numpy().view(np.uint32)


def check(rt, ora, r, q, want, fanout, layout, split, bulk="auto", replay=True):
    print(f"case walk n={r.shape[0]} nq={q.shape[0]} F={fanout} {layout} split={split} bulk={bulk} replay={replay}",
          flush=True)
    t = rt.build_str(r, fanout, layout)
    t.set_split(split)
    t.set_bulk_copy(bulk)
    off, ids = device_select(rt, t, q, int(want[1].size), replay)
    assert np.array_equal(off, want[0].astype(np.int64))
    assert np.array_equal(ids, want[1])
    t.free()


@pytest.mark.parametrize("fanout,layout", [(2, "soa"), (5, "aos"), (16, "d2"), (17, "soa"), (32, "aos"), (33, "d2"),
                                           (63, "soa"), (64, "d2")])
@pytest.mark.parametrize("nq", [1, 7, 2500, 40_000])
def test_walk_grids(rt, ora, fanout, layout, nq):
    r = rtgen.c2_rects(30_011)
    q = rtgen.windows_loguniform(nq, 1e-5, 1e-2 if nq > 7 else 0.3, 31 + nq)
    want = ora.select(ora.build_str(r, 32), q)
    check(rt, ora, r, q, want, fanout, layout, 0)
    check(rt, ora, r, q, want, fanout, layout, 0, replay=False)
    check(rt, ora, r, q, want, fanout, layout, 1)


@pytest.mark.parametrize("fanout,layout,nq", [(2, "soa", 6000), (16, "aos", 3000), (64, "soa", 600)])
def test_walk_shared_windows(rt, ora, fanout, layout, nq):
    """Windows large enough to be shared (6000 of them on a binary tree fill
    the item lists), whole-space windows among them, with and without the
    replay's deferred ranges."""
    r = rtgen.c2_rects(25_000 if fanout == 2 else 200_000)
    q = rtgen.windows_loguniform(nq, 3e-3, 3e-2, 77)
    q[::97] = (-np.inf, -np.inf, np.inf, np.inf)
    want = ora.select(ora.build_str(r, 32), q)
    for bulk in ("off", "on"):
        check(rt, ora, r, q, want, fanout, layout, 2, bulk)


@pytest.mark.parametrize("nq,big", [(100, 1), (3, 3), (2000, 40)])
def test_two_stage_deferred_ranges(rt, ora, nq, big):
    """Two-stage select whose records (a chunk per lane group) reach past the
    few ids' sort scratch into the fill stage's own layout while the replay
    defers long leaf ranges: the descriptors must not land on the records."""
    import torch
    r = rtgen.c2_rects(200_000)
    q = rtgen.windows_loguniform(nq, 1e-8, 1e-7, 61)
    q[:big] = (-0.5, -0.5, 0.45, 1.5)
    wo, wi = ora.select(ora.build_str(r, 32), q)
    total = int(wo[-1])
    t = rt.build_str(r, 16, "soa")
    t.set_bulk_copy("on")
    wb = rt.select_replay_workspace_bytes(nq, 4 * total)
    work = torch.empty(wb, dtype=torch.uint8, device="cuda")
    dq = torch.from_numpy(q).cuda()
    off = torch.empty(nq + 1, dtype=torch.int64, device="cuda")
    ids = torch.full((total,), -1, dtype=torch.int32, device="cuda")
    st = torch.zeros(2, dtype=torch.int64, device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    rt.range_select_device_count(t, dq.data_ptr(), nq, off.data_ptr(), work.data_ptr(), wb, s)
    rt.range_select_device_fill(t, dq.data_ptr(), nq, off.data_ptr(), ids.data_ptr(), total, work.data_ptr(), wb,
                                st.data_ptr(), s)
    torch.cuda.synchronize()
    assert st.cpu().tolist() == [total, 0]
    chunks, over = rt.select_replay_info(work.data_ptr())
    assert chunks > 0 and not over
    assert np.array_equal(off.cpu().numpy(), wo.astype(np.int64))
    assert np.array_equal(ids.cpu().numpy().view(np.uint32), wi)


@pytest.mark.parametrize("nq", [1, 9, 3000])
def test_library_workspaces(rt, ora, nq):
    """Host and stream-ordered selects whose fill stage outgrows the count
    stage's workspace (whole-space windows) and so moves to another one while
    the records stay, twice on two streams, between selects that do not."""
    import torch
    r = rtgen.c2_rects(300_000)
    t = rt.build_str(r, 32, "soa")
    ot = ora.build_str(r, 32)
    q = rtgen.windows_loguniform(nq, 1e-7, 1e-4, 5)
    small = q.copy()
    q[:9] = (-1.0, -1.0, 2.0, 2.0)
    for w in (small, q, small):
        wo, wi = ora.select(ot, w)
        off, ids = rt.range_select(t, w)
        assert np.array_equal(off, wo) and np.array_equal(ids, wi)
        dq = torch.from_numpy(w).cuda()
        torch.cuda.synchronize()
        outs = []
        for s in (torch.cuda.Stream(), torch.cuda.Stream()):
            d = (torch.empty(nq + 1, dtype=torch.int64, device="cuda"),
                 torch.full((wi.size + 5,), -1, dtype=torch.int32, device="cuda"),
                 torch.zeros(1, dtype=torch.int64, device="cuda"))
            torch.cuda.synchronize()
            assert rt.range_select_async(t, dq.data_ptr(), nq, d[0].data_ptr(), d[1].data_ptr(), wi.size + 5,
                                         d[2].data_ptr(), s.cuda_stream)
            outs.append((d, s))
        torch.cuda.synchronize()
        for (off, ids, total), _ in outs:
            assert int(total.item()) == wi.size
            assert np.array_equal(off.cpu().numpy(), wo.astype(np.int64))
            assert np.array_equal(ids[:wi.size].cpu().numpy().view(np.uint32), wi) and bool((ids[wi.size:] == -1).all())


@pytest.mark.parametrize("fanout,layout", [(64, "soa"), (64, "aos"), (63, "d2"), (32, "soa"), (16, "aos"), (3, "soa")])
def test_runs_of_contained_children(rt, ora, fanout, layout):
    """Windows over the whole space, over its halves and over strips, one
    tree of fanout ** 2 objects (the root's children are full leaves) and one
    of a few more: contained children at the front, in the middle, at the end
    or all of a node's become runs of one leaf up to the whole node, of 3 ids
    up to several rounds of the copy."""
    g = np.random.default_rng(fanout)
    for n in [fanout * fanout, fanout * fanout + 1, 6 * fanout * fanout + 5]:
        r = np.tile(g.random((n, 2), np.float32), (1, 2))
        e = np.linspace(-0.01, 1.01, 9, dtype=np.float32)
        q = [[-1, -1, 2, 2]]
        q += [[-1, lo, 2, hi] for lo in e for hi in e if lo < hi]
        q += [[lo, -1, hi, 2] for lo in e for hi in e if lo < hi]
        q = np.array(q, np.float32)
        want = ora.select(ora.build_str(r, fanout), q)
        check(rt, ora, r, q, want, fanout, layout, 0)
        check(rt, ora, r, q, want, fanout, layout, 2, "on")


@pytest.mark.parametrize("fanout", [16, 32, 64])
@pytest.mark.parametrize("nq", [1, 9, 4095, 16_383, 16_385, 40_000])
def test_chunks_by_place(rt, ora, fanout, nq):
    """Window counts below, at and above the number of lane groups, most of
    the windows empty and one with most of the records, so that groups that own
    a record chunk leave it empty and others need many."""
    r = rtgen.c2_rects(60_000)
    g = np.random.default_rng(nq)
    lo = g.random((nq, 2), np.float32) + 2
    q = np.concatenate([lo, lo + np.float32(0.01)], axis=1)
    some = g.integers(0, nq, max(nq // 50, 1))
    q[some] = np.concatenate([lo[some] - 2, lo[some] - 2 + np.float32(0.03)], axis=1)
    q[nq // 2] = [0.01, 0.01, 0.99, 0.99]
    want = ora.select(ora.build_str(r, fanout), q)
    for split in [0, 2]:
        check(rt, ora, r, q, want, fanout, "soa", split)
    b = rt.Batch([rt.build_str(r, fanout, "soa"), rt.build_str(r, fanout, "aos")], [q, q[: nq // 2 + 1]])
    for _ in range(3):
        b.run()
        for i, n in enumerate([nq, nq // 2 + 1]):
            off, ids = b.result(i)
            assert np.array_equal(np.asarray(off).astype(np.int64), want[0][: n + 1].astype(np.int64))
            assert np.array_equal(ids, want[1][: int(want[0][n])])
