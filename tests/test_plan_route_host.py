"""Which plans write their arrays indexed by pair through the L2s, and which fused plan + dispatch calls their rows, as the library's host-only
queries tell it from the sizes.  No GPU is needed, nothing is launched."""
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


@pytest.fixture(scope="module")
def fused(through):
    from paper_2512_22036_amd import binding

    def ask(N, k, row, aux=0, at=0x20000000):
        L = binding._CLayout()
        assert through.lib.fusco_layout_bind(ctypes.byref(L), N, k, 64, 8, 0x10000000, through.lib.fusco_layout_bytes(N, k, 64, 8)) == 0
        return through.lib.fusco_probe_plan_dispatch_through(ctypes.byref(L), row, aux, at)

    return ask


def test_rows_of_fused_calls_by_size(fused):
    assert fused(128, 8, 2032) == fused(127, 8, 2048) == 0 and fused(128, 8, 2048) == 1     # 2 MiB
    assert fused(128, 8, 7168, 224) == fused(128, 8, 7168) == 1                              # the decode batch of the benchmark
    assert fused(4, 8, 7168, 224) == fused(1, 64, 1 << 20) == fused(0, 8, 7168) == 0
    assert fused(64, 32, 12288) == 1 and fused(64, 32, 12352) == 0                            # 384 KiB by a workgroup


def test_few_workgroups_that_write_much(fused):
    assert [fused(N, 8, 16384) for N in (16, 18, 32, 47, 48, 64, 256)] == [0, 0, 0, 0, 1, 1, 1]
    assert [fused(N, 16, 10752) for N in (14, 40, 47, 48)] == [0, 0, 0, 1]
    assert [fused(N, 8, 32768) for N in (10, 47, 48)] == [0, 0, 1]                           # two column segments
    assert [fused(N, 8, 12288) for N in (21, 22, 48)] == [0, 1, 1]                           # 96 KiB by a workgroup
    assert [fused(N, 8, 12352) for N in (22, 47, 48)] == [0, 0, 1]


def test_rows_of_partial_units(fused):
    assert [fused(N, 8, 10400) for N in (40, 63, 64, 201, 202)] == [0, 0, 1, 1, 0]           # up to 16 MiB
    assert [fused(N, 8, 8192, at=0x20000010) for N in (40, 63, 64, 255, 256)] == [0, 0, 1, 1, 0]
    assert [fused(N, 8, 8192, at=0x20000040) for N in (40, 63, 64, 255, 256)] == [1, 1, 1, 1, 1]


def test_fused_bad_arguments(fused, through):
    assert fused(128, 8, 0) < 0 and fused(128, 8, 24) < 0 and fused(128, 8, 16, 8) < 0 and fused(128, 8, 1 << 21) < 0
    assert fused(257, 8, 7168) == -3 and through.lib.fusco_probe_plan_dispatch_through(None, 16, 0, None) < 0
