"""Which plans write their arrays indexed by pair through the L2s, as the library's host-only query tells it from the sizes: tiles of whole
64-byte units, enough of them and not too many.  No GPU is needed, nothing is launched."""
import ctypes

import pytest


@pytest.fixture(scope="module")
def through():
    import os

    from paper_2512_22036_amd import binding
    if not os.path.exists(binding.library_path()):
        from paper_2512_22036_amd.build import build_library
        build_library()
    lib = binding.load_library()

    def ask(N, k, E=64, D=8):
        L = binding._CLayout()
        assert lib.fusco_layout_bind(ctypes.byref(L), N, k, E, D, 0x10000000, lib.fusco_layout_bytes(N, k, E, D)) == 0
        return lib.fusco_probe_plan_through(ctypes.byref(L))

    ask.lib = lib
    return ask


@pytest.mark.parametrize("k", [1, 2, 4, 8, 16, 32, 48, 64])
def test_tiles_of_whole_units(through, k):
    tile = 2048 // k
    assert [through(n * tile, k) for n in (1, 100, 199, 200, 512, 1024)] == [0, 0, 0, 1, 1, 1]
    assert through(199 * tile + 1, k) == 1 and through(1024 * tile + 1, k) == through(4096 * tile, k) == 0


@pytest.mark.parametrize("k", [3, 5, 6, 7, 9, 10, 12, 24])
def test_tiles_of_partial_units(through, k):
    tile = 2048 // k   # fewer than 2048 pairs a tile: all but the first start inside a unit
    assert tile * k % 16 != 0
    assert [through(n * tile, k) for n in (199, 200, 500, 1024, 2000)] == [0, 0, 0, 0, 0]


def test_bad_arguments(through):
    assert through.lib.fusco_probe_plan_through(None) < 0
