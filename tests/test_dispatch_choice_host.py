"""Which kernel fusco_dispatch takes, as its host-only query tells it: no GPU is needed, nothing is launched."""
import ctypes

import pytest

EXPERT, WIRE, TWO_HOP, STREAMING = 1, 2, 4, 8


@pytest.fixture(scope="module")
def tiled():
    import os

    from paper_2512_22036_amd import binding
    if not os.path.exists(binding.library_path()):
        from paper_2512_22036_amd.build import build_library
        build_library()
    lib = binding.load_library()

    def ask(N, k, E, D, row, aux=0, flags=0):
        L = binding._CLayout()
        # the block is never touched: binding is pointer arithmetic and the query reads the sizes
        assert lib.fusco_layout_bind(ctypes.byref(L), N, k, E, D, 0x10000000, lib.fusco_layout_bytes(N, k, E, D)) == 0
        rc = lib.fusco_dispatch_in_transfer_order(ctypes.byref(L), row, aux, flags)
        assert rc in (0, 1)
        return bool(rc)

    ask.lib = lib
    return ask


def test_query_answers_for_calls_that_write_both_tensors(tiled):
    both = EXPERT | WIRE
    for row, aux in ((14336, 0), (14336, 224), (8448, 0), (16384 + 1040, 0)):
        assert tiled(8192, 8, 256, 8, row, aux) and tiled(8192, 8, 256, 8, row, aux, both)
        assert tiled(8192, 8, 256, 8, row, aux, both | STREAMING)
        assert not tiled(8192, 8, 256, 8, row, aux, WIRE)                 # the receive tensors alone
        assert not tiled(8192, 8, 256, 8, row, aux, both | TWO_HOP) and not tiled(8192, 8, 256, 8, row, aux, TWO_HOP)
    assert not tiled(1000, 8, 256, 8, 14336, 0, both)                     # where the expert tensor alone walks, both do
    knob = tiled.lib.fusco_probe_dispatch_kernel
    for which in (1, 2):                                                  # both tensors: the automatic choice only
        assert knob(which) == 0
        try:
            assert not tiled(8192, 8, 256, 8, 14336, 0, both) and tiled(8192, 8, 256, 8, 14336) == (which == 2)
        finally:
            assert knob(0) == which


def test_launches_that_would_pass_the_thread_limit_walk_the_tokens(tiled):
    # one wave per row: 28128 x 2048 x 64 threads fit a launch, 62504 x 2048 x 64 (1.9 x 2^32) do not
    assert tiled(900_000, 64, 64, 8, 64) and not tiled(2_000_000, 64, 64, 8, 64)
    assert tiled(4_000_000, 16, 64, 8, 16) and not tiled(8_000_000, 16, 64, 8, 16)
    # a source tensor that is taken in chunks has launches of one chunk, however many tokens there are
    assert tiled(2_000_000, 8, 64, 8, 14336)


def test_both_tensors_walk_where_the_tiles_lose(tiled):
    both = EXPERT | WIRE

    def pair(*sizes):
        return tiled(*sizes), tiled(*sizes, 0, both)

    yes, no = (True, True), (True, False)      # the expert tensor alone, both tensors
    # many devices, short rows, few rows per token: measured up to 1.8 times slower than the walk
    assert pair(8192, 16, 256, 16, 14336) == no and pair(4096, 32, 256, 32, 8192) == no and pair(2048, 64, 512, 64, 8192) == no
    assert pair(8192, 8, 256, 16, 14336) == no
    assert pair(8192, 8, 256, 8, 5760) == no and pair(65536, 8, 256, 8, 1024) == no
    assert pair(8192, 4, 64, 4, 14336) == no and pair(8192, 6, 60, 4, 14336) == no and pair(8192, 6, 60, 2, 14336) == no
    # at most 8 devices with long rows and k >= 8, or at most 2 devices with whole rows
    assert pair(8192, 8, 256, 8, 8192) == yes and pair(8192, 8, 256, 8, 8176) == no and pair(8192, 16, 256, 8, 8192) == yes
    assert pair(8192, 10, 160, 5, 10240) == yes and pair(2048, 64, 512, 8, 8192) == yes
    assert pair(8192, 8, 256, 2, 5760) == yes and pair(8192, 8, 256, 4, 5760) == no
    assert pair(8192, 6, 60, 2, 10240) == yes and pair(8192, 6, 60, 1, 10240) == yes
    assert pair(41616, 4, 16, 1, 2320) == no and pair(20000, 4, 16, 1, 4096) == yes and pair(41616, 8, 16, 1, 2320) == yes
