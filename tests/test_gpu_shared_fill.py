"""The walking fill of shared windows (records that do not fit their arena with
the split mapping on) against the oracle: trees of three levels and more with a
short leaf, every lane-group width and layout, windows of one share and of all
of them, whole-space ones among them, empty ones, more windows than lane groups
and fewer, in one call and in two stages."""

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


def windows(nq, hi, seed):
    q = rtgen.windows_loguniform(nq, 1e-6, hi, seed)
    q[nq // 2] = [-np.inf, -np.inf, np.inf, np.inf]
    q[nq // 3] = [-1.0, 0.25, 2.0, 0.5]
    if nq > 8:
        q[1::5] = [3.0, 3.0, 4.0, 4.0]
    return q


def check(rt, ora, r, q, want, fanout, layout, room, stages):
    import torch
    wo, wi = want
    nq, cap = q.shape[0], int(wi.size)
    print(f"case shared fill n={r.shape[0]} nq={nq} F={fanout} {layout} room={room} stages={stages}", flush=True)
    t = rt.build_str(r, fanout, layout)
    assert t.info().height >= 3
    t.set_split(1)
    dq = torch.from_numpy(q).cuda()
    off = torch.empty(nq + 1, dtype=torch.int64, device="cuda")
    ids = torch.full((cap + 64,), -1, dtype=torch.int32, device="cuda")
    st = torch.zeros(2, dtype=torch.int64, device="cuda")
    w0, w1 = rt.select_workspace_bytes(nq, 0), rt.select_workspace_bytes(nq, cap)
    w = torch.empty(max(w0 + room, w1 + room), dtype=torch.uint8, device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    for _ in range(2):   # the second one on what the first left
        if stages == 1:
            rt.range_select_device(t, dq.data_ptr(), nq, off.data_ptr(), ids.data_ptr(), cap, w.data_ptr(), w1 + room,
                                   st.data_ptr(), s)
        else:
            rt.range_select_device_count(t, dq.data_ptr(), nq, off.data_ptr(), w.data_ptr(), w0 + room, s)
            rt.range_select_device_fill(t, dq.data_ptr(), nq, off.data_ptr(), ids.data_ptr(), cap, w.data_ptr(),
                                        w.numel(), st.data_ptr(), s)
        torch.cuda.synchronize()
        assert st.cpu().tolist() == [cap, 0]
        assert rt.select_replay_info(w.data_ptr())[1], "the case is meant to overflow"
        assert np.array_equal(off.cpu().numpy(), wo.astype(np.int64))
        assert np.array_equal(ids[:cap].cpu().numpy().view(np.uint32), wi) and bool((ids[cap:] == -1).all())
    t.free()


@pytest.mark.parametrize("fanout,layout", [(2, "soa"), (5, "aos"), (16, "d2"), (17, "soa"), (32, "aos"), (33, "d2"),
                                           (63, "soa"), (64, "aos")])
@pytest.mark.parametrize("nq,hi", [(3, 0.5), (40, 0.2), (3000, 2e-2)])
def test_fanouts(rt, ora, fanout, layout, nq, hi):
    r = rtgen.c2_rects(30_011 if fanout < 16 else 290_001)
    q = windows(nq, hi, nq + fanout)
    want = ora.select(ora.build_str(r, 32), q)
    for stages in (1, 2):
        check(rt, ora, r, q, want, fanout, layout, 8192, stages)


@pytest.mark.parametrize("less", [1, 2, 1000])
def test_room(rt, ora, less):
    """A chunk or two less than the records need, which the first launch leaves
    to the items, and one chunk."""
    import torch
    r = rtgen.c2_rects(200_003)
    q = windows(30, 0.3, 5)
    want = ora.select(ora.build_str(r, 32), q)
    t = rt.build_str(r, 16, "soa")
    t.set_split(1)
    dq = torch.from_numpy(q).cuda()
    off = torch.empty(31, dtype=torch.int64, device="cuda")
    wb = rt.select_workspace_bytes(30, 0) + (1 << 22)
    w = torch.empty(wb, dtype=torch.uint8, device="cuda")
    rt.range_select_device_count(t, dq.data_ptr(), 30, off.data_ptr(), w.data_ptr(), wb, 0)
    torch.cuda.synchronize()
    chunks, over = rt.select_replay_info(w.data_ptr())
    assert chunks > 4 and not over
    room = max(1, chunks - less) * 4100 + 512
    for stages in (1, 2):
        check(rt, ora, r, q, want, 16, "soa", room, stages)


def test_many_windows(rt, ora):
    """More windows than lane groups, ordered, most of one share."""
    r = rtgen.c2_rects(100_000)
    q = windows(60_000, 1e-3, 6)
    want = ora.select(ora.build_str(r, 32), q)
    check(rt, ora, r, q, want, 32, "soa", 1 << 20, 1)


def test_too_small_output(rt, ora):
    """An overflowed select whose result does not fit writes no ids."""
    import torch
    r = rtgen.c2_rects(50_000)
    q = windows(20, 0.2, 7)
    total = int(ora.select(ora.build_str(r, 32), q)[0][-1])
    t = rt.build_str(r, 16, "soa")
    t.set_split(1)
    dq = torch.from_numpy(q).cuda()
    off = torch.empty(21, dtype=torch.int64, device="cuda")
    ids = torch.full((total,), -1, dtype=torch.int32, device="cuda")
    st = torch.zeros(2, dtype=torch.int64, device="cuda")
    wb = rt.select_workspace_bytes(20, total - 1) + 8192
    w = torch.empty(wb, dtype=torch.uint8, device="cuda")
    rt.range_select_device(t, dq.data_ptr(), 20, off.data_ptr(), ids.data_ptr(), total - 1, w.data_ptr(), wb,
                           st.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert st.cpu().tolist() == [total, 1] and bool((ids == -1).all())
