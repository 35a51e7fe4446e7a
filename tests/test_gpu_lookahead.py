"""Lookahead loads where they are used -- the walking fill, and counts by output
slot -- with selects that do not replay records, for every node layout, lane-group
width and fanout class, against brute force; and that those kernels ran."""

import numpy as np
import pytest

import oracle
import rtgen
from test_gpu_select import FANOUTS, assert_csr_equal

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layout", ["soa", "aos", "d2"])
@pytest.mark.parametrize("fanout", FANOUTS)
def test_walks_with_lookahead(fanout, layout):
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    import paper_2309_16913_amd as rt
    o = oracle.get()
    for s, n in enumerate([0, 1, fanout, fanout + 1, 97, 1500, 6000]):
        print(f"case lookahead walk F={fanout} {layout} n={n}", flush=True)
        r = rtgen.adversarial_rects(n, 1000 * fanout + s) if n else np.zeros((0, 4), np.float32)
        q = rtgen.adversarial_windows(64, 77 * fanout + s)
        want = o.brute_select(r, q)
        t = rt.build_str(r, fanout, layout)
        t.set_replay(False)
        t.set_lookahead(True)
        for split in (0, 1):
            for bulk in ("off", "on"):
                t.set_split(split)
                t.set_bulk_copy(bulk)
                assert_csr_equal(rt.range_select(t, q), want, f"F={fanout} {layout} n={n} split={split} bulk={bulk}")
        t.free()


@pytest.mark.parametrize("split", [0, 2])
def test_lookahead_kernels_run(split):
    import torch
    from torch.profiler import ProfilerActivity, profile
    import paper_2309_16913_amd as rt
    r, q = rtgen.c2_rects(50_000), rtgen.windows_loguniform(300, 1e-4, 1e-2, 8)
    o = oracle.get()
    want = o.select(o.build_str(r, 32), q)
    t = rt.build_str(r, 16, "soa")
    t.set_split(split)
    t.set_replay(False)
    for la in (False, True):
        t.set_lookahead(la)
        torch.cuda.synchronize()
        with profile(activities=[ProfilerActivity.CUDA]) as p:
            got = rt.range_select(t, q)
            torch.cuda.synchronize()
        assert_csr_equal(got, want, f"split={split} lookahead={la}")
        names = [e.name for e in p.events()]
        # <lane group, layout, 0 count or 1 fill, lookahead, deferral>
        assert any(f"select_kernel<16, 1, 1, {int(la)}, 0>" in n for n in names), names
        assert any(f"select_kernel<16, 1, 0, {int(la)}, 0>" in n for n in names) == (split != 0), names
