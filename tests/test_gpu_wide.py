"""Trees whose nodes pass 4 GiB (node offsets of 64 bits in the batched walk) in
every lane-group width and layout, against brute force on the device; and
batches of more windows than the scan's tiles add up themselves."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

N = 216_000_000


@pytest.fixture(scope="module")
def rt():
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    import paper_2309_16913_amd as m
    return m


@pytest.fixture(scope="module")
def wide(rt):
    """Rectangles, windows of 0 to some 20000 ids, and their ids by brute force."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(4)
    lo = torch.rand(N, 2, generator=g, device="cuda")
    r = torch.cat([lo, lo + torch.rand(N, 2, generator=g, device="cuda") * 1e-5], dim=1).contiguous()
    del lo
    c = torch.rand(48, 2, generator=g, device="cuda")
    s = 10.0 ** (torch.rand(48, 1, generator=g, device="cuda") * 2 - 4)
    q = torch.cat([c - s / 2, c + s / 2], dim=1)
    q[5] = torch.tensor([3.0, 3.0, 4.0, 4.0])
    q = q.contiguous()
    want = []
    for w in q.cpu().tolist():
        hit = (r[:, 0] <= w[2]) & (r[:, 2] >= w[0]) & (r[:, 1] <= w[3]) & (r[:, 3] >= w[1])
        want.append(torch.nonzero(hit).flatten().to(torch.int32))
        del hit
    torch.cuda.empty_cache()
    yield r, q, want
    torch.cuda.empty_cache()


@pytest.mark.parametrize("fanout,layout,n", [(2, "soa", 110_000_000), (16, "aos", N), (16, "d2", N), (32, "soa", N),
                                             (32, "aos", N), (32, "d2", N), (64, "soa", N), (64, "aos", N), (64, "d2", N)])
def test_nodes_past_4_gib(rt, wide, fanout, layout, n):
    import torch
    r, q, want = wide
    want = [w[w < n] for w in want]
    ids_want = torch.cat(want)
    off_want = torch.tensor([0] + np.cumsum([w.numel() for w in want]).tolist(), device="cuda")
    nq, cap = q.shape[0], ids_want.numel()
    s = torch.cuda.current_stream().cuda_stream
    t = rt.build_str_device(r.data_ptr(), n, fanout, layout, s)
    assert t.info().device_bytes > 1 << 32
    print(f"case wide F={fanout} {layout} n={n} ids={cap} node bytes={t.info().device_bytes}", flush=True)
    off = torch.empty(nq + 1, dtype=torch.int64, device="cuda")
    ids = torch.empty(cap, dtype=torch.int32, device="cuda")
    st = torch.zeros(2, dtype=torch.int64, device="cuda")
    full = rt.select_replay_workspace_bytes(nq, cap)
    work = torch.empty(full, dtype=torch.uint8, device="cuda")
    for split in (0, 4):
        t.set_split(split)
        for replay in (True, False):
            t.set_replay(replay)
            ids.fill_(-1)
            rt.range_select_device(t, q.data_ptr(), nq, off.data_ptr(), ids.data_ptr(), cap, work.data_ptr(), full,
                                   st.data_ptr(), s)
            torch.cuda.synchronize()
            chunks, over = rt.select_replay_info(work.data_ptr())
            assert (chunks > 0) == replay and not over
            assert st.cpu().tolist() == [cap, 0]
            assert torch.equal(off, off_want) and torch.equal(ids, ids_want), (split, replay)
    t.set_split(0)
    cnt = torch.empty(nq, dtype=torch.int32, device="cuda")
    rt.range_count_device(t, q.data_ptr(), nq, cnt.data_ptr(), work.data_ptr(), full, s)
    torch.cuda.synchronize()
    assert torch.equal(cnt.to(torch.int64), off_want.diff())
    b = rt.Batch([t], [q.cpu().numpy()])
    for replay in (True, False):
        b.set_replay(replay)
        b.run()
        o, i = b.result(0)
        assert np.array_equal(np.asarray(o).astype(np.int64), off_want.cpu().numpy())
        assert np.array_equal(i, ids_want.cpu().numpy().view(np.uint32)), replay
    b.free()
    t.free()


@pytest.mark.parametrize("nq", [4096 * 2048, 4096 * 2048 + 1, 9_000_001])
def test_scan_of_many_tiles(rt, nq):
    """Window i takes i % 4 neighbouring points of a line."""
    import torch
    x = np.arange(1000, dtype=np.float32)
    t = rt.build_str(np.stack([x, x * 0, x, x * 0], axis=1), 16, "soa")
    i = torch.arange(nq, device="cuda")
    c, a = i % 4, (i * 7919) % 990
    q = torch.stack([a - 0.5, torch.full_like(a, -1), a + c - 0.5, torch.full_like(a, 1)], dim=1).to(torch.float32)
    q[:, 2] = torch.maximum(q[:, 2], q[:, 0])
    q = q.contiguous()
    off_want = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), torch.cumsum(c, 0)])
    cap = int(off_want[-1])
    k = torch.repeat_interleave(i, c)
    ids_want = (a[k] + torch.arange(cap, device="cuda") - off_want[k]).to(torch.int32)
    print(f"case scan of many tiles nq={nq} ids={cap}", flush=True)
    off = torch.empty(nq + 1, dtype=torch.int64, device="cuda")
    ids = torch.full((cap,), -1, dtype=torch.int32, device="cuda")
    st = torch.zeros(2, dtype=torch.int64, device="cuda")
    wb = rt.select_replay_workspace_bytes(nq, cap)
    work = torch.empty(wb, dtype=torch.uint8, device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    rt.range_select_device(t, q.data_ptr(), nq, off.data_ptr(), ids.data_ptr(), cap, work.data_ptr(), wb, st.data_ptr(), s)
    torch.cuda.synchronize()
    assert st.cpu().tolist() == [cap, 0]
    assert torch.equal(off, off_want) and torch.equal(ids, ids_want)
    # the total through the library's own workspace, read by the host
    total = torch.zeros(1, dtype=torch.int64, device="cuda")
    ids.fill_(-1)
    assert rt.range_select_async(t, q.data_ptr(), nq, off.data_ptr(), ids.data_ptr(), cap, total.data_ptr(), s)
    torch.cuda.synchronize()
    assert int(total.item()) == cap and torch.equal(off, off_want) and torch.equal(ids, ids_want)
    assert not rt.range_select_async(t, q.data_ptr(), nq, off.data_ptr(), ids.data_ptr(), cap - 1, total.data_ptr(), s)
    assert int(total.item()) == cap
