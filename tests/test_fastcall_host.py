"""csrc/fastcall.cpp without a GPU: whatever it does not handle it leaves to the ctypes path by returning None."""
import os

import torch


def test_leaves_everything_else_to_the_other_path():
    from paper_2512_22036_amd import binding
    from paper_2512_22036_amd.build import FASTCALL, build_fastcall, build_library
    if not os.path.exists(binding.library_path()):
        build_library()
    if not os.path.exists(FASTCALL):
        build_fastcall()
    fast = binding._bind_fastcall(binding.load_library())
    assert fast is not None

    class Plain:
        c, scratch, N, k = binding._CLayout(), torch.zeros(4), 2, 2

    ids, rows = torch.zeros((2, 2), dtype=torch.int32), torch.zeros((4, 8))
    for layout in (Plain(), None, 3):
        assert fast.plan(layout, ids) is None
        assert fast.dispatch(layout, rows, rows, None, None, None, None, 0) is None
        assert fast.plan_dispatch(layout, ids, rows, rows, None, None) is None
        assert fast.combine(layout, rows, rows, rows) is None
        assert fast.combine_two_hop(layout, rows, rows, rows, rows) is None
    assert fast.plan(Plain()) is None and fast.combine(Plain(), 1, "a", None) is None
    assert fast.dispatch(Plain(), rows, rows, None, None, None, None, "flags") is None
