"""The workspace a select asks for: callers keep these sizes, and the select with
fixed scratch accepts a size by them, so they do not move with the layout."""

import pytest

import paper_2309_16913_amd as rt


@pytest.mark.parametrize("nq,cap,size", [(1, 0, 1875200),
                                        (1, 1, 1875200),
                                        (1, 8000000, 34689024),
                                        (100, 32769, 2016000),
                                        (8191, 1000000, 6587392),
                                        (8192, 1000000, 6587904),
                                        (262145, 7, 49854208),
                                        (1000000, 1443956528, 6112883968)])
def test_select_workspace_bytes(nq, cap, size):
    assert rt.select_workspace_bytes(nq, cap) == size


def test_fixed_scratch_limit():
    """The largest result of one window that 32 MiB of scratch take."""
    assert rt.select_workspace_bytes(1, 7723880) <= 32 << 20 < rt.select_workspace_bytes(1, 7723880 + 1)
