"""Plain batch runs whose trees' results begin at every remainder of four ids in
the common scratch and hold segments of several parts, against the oracle."""

import numpy as np
import pytest

import oracle
from test_gpu_sort_parts import line, windows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("first", [4, 5, 6, 7])
def test_plain_run_long_segments(first):
    import torch
    assert torch.cuda.is_available(), "GPU test needs a GPU"
    import paper_2309_16913_amd as rt
    sizes = [100, 120_000, 60_001]
    lengths = [[first], [33_000, 120_000, 7], [60_001, 50_000]]
    rs = [line(n, 31 + i) for i, n in enumerate(sizes)]
    qs = [windows(n, c, 41 + i) for i, (n, c) in enumerate(zip(sizes, lengths))]
    print(f"case plain long segments first={first}", flush=True)
    b = rt.Batch([rt.build_str(r, 32, "soa") for r in rs], qs)
    b.run_plain()
    for i in range(len(sizes)):
        want = oracle.get().select(oracle.get().build_str(rs[i], 32), qs[i])
        off, ids = b.result(i)
        assert np.array_equal(np.asarray(off).astype(np.int64), want[0].astype(np.int64))
        assert np.array_equal(ids, want[1])
