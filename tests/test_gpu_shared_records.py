"""Windows whose walks are shared by many lane groups keep their records: at the
documented workspace size, and with the room that the library gives its own
selects, the count pass does not run out of it, and the replayed ids are the
walked ones."""

import os
import subprocess

import numpy as np
import pytest

import rtgen

pytestmark = pytest.mark.gpu

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2309_16913_amd", "csrc")


@pytest.fixture(scope="module")
def rects():
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    return torch.from_numpy(rtgen.c2_rects(10_000_000)).cuda()


@pytest.fixture(scope="module")
def guess(tmp_path_factory):
    """Bytes of record room of a library-held workspace."""
    d = tmp_path_factory.mktemp("guess")
    (d / "g.cpp").write_text('#include <cstdio>\n#include <cstdlib>\n#include "rec_space.h"\n'
                             'int main(int, char **v) { std::printf("%llu", (unsigned long long)rtk::rec_arena_guess('
                             '256, std::atoi(v[1]), true, std::atoll(v[2]), std::atoll(v[3]))); }\n')
    subprocess.run(["g++", "-std=c++17", "-I", CSRC, str(d / "g.cpp"), "-o", str(d / "g")], check=True)
    return lambda width, nq, cap: int(subprocess.run([str(d / "g"), str(width), str(nq), str(cap)], capture_output=True,
                                                     text=True, check=True).stdout)


def select(rt, t, q, cap, wb, stages):
    import torch
    nq = q.shape[0]
    off = torch.empty(nq + 1, dtype=torch.int64, device="cuda")
    ids = torch.full((cap,), -1, dtype=torch.int32, device="cuda")
    st = torch.zeros(2, dtype=torch.int64, device="cuda")
    w = torch.empty(max(wb, rt.select_workspace_bytes(nq, cap)), dtype=torch.uint8, device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    if stages == 1:
        rt.range_select_device(t, q.data_ptr(), nq, off.data_ptr(), ids.data_ptr(), cap, w.data_ptr(), wb, st.data_ptr(), s)
    else:
        rt.range_select_device_count(t, q.data_ptr(), nq, off.data_ptr(), w.data_ptr(), wb, s)
        rt.range_select_device_fill(t, q.data_ptr(), nq, off.data_ptr(), ids.data_ptr(), cap, w.data_ptr(), w.numel(),
                                    st.data_ptr(), s)
    torch.cuda.synchronize()
    assert st.cpu().tolist() == [cap, 0]
    return off, ids, rt.select_replay_info(w.data_ptr())


@pytest.mark.parametrize("fanout,layout", [(16, "aos"), (32, "soa"), (64, "d2")])
@pytest.mark.parametrize("nq,hi", [(10, 1e-2), (100, 1e-3), (100, 1e-2), (1000, 1e-4), (1000, 1e-3), (1000, 1e-2), (10_000, 1e-3)])
def test_no_overflow(rects, guess, fanout, layout, nq, hi):
    import torch
    import paper_2309_16913_amd as rt
    q = torch.from_numpy(rtgen.windows_loguniform(nq, 1e-6, hi, nq + 3)).cuda()
    t = rt.build_str_device(rects.data_ptr(), rects.shape[0], fanout, layout, torch.cuda.current_stream().cuda_stream)
    off = torch.empty(nq + 1, dtype=torch.int64, device="cuda")
    w0 = rt.select_workspace_bytes(nq, 0)
    work = torch.empty(w0, dtype=torch.uint8, device="cuda")
    rt.range_select_device_count(t, q.data_ptr(), nq, off.data_ptr(), work.data_ptr(), w0, 0)
    cap = int(off[nq].item())
    print(f"case shared records F={fanout} {layout} nq={nq} hi={hi} ids={cap}", flush=True)
    walked = select(rt, t, q, cap, rt.select_workspace_bytes(nq, cap), 1)
    assert walked[2] == (0, False)
    t.set_split(16)
    width = 16 if fanout <= 16 else 32 if fanout <= 32 else 64
    for wb, stages in ((rt.select_replay_workspace_bytes(nq, cap), 1), (w0 + guess(width, nq, cap + 1000), 2)):
        got = select(rt, t, q, cap, wb, stages)
        chunks, over = got[2]
        assert chunks > 0 and not over, (chunks, stages)
        assert torch.equal(got[0], walked[0]) and torch.equal(got[1], walked[1])
    t.free()
