"""How fusco_dispatch moves the rows of a call, as the library's host-only query tells it from sizes, flags and the places of the tensors:
no GPU is needed, nothing is launched, the pointers are never followed."""
import ctypes

import pytest

EXPERT, WIRE, TWO_HOP, STREAMING = 1, 2, 4, 8
TOKENS, TILES, BOTH, SEPARATE = 0, 1, 2, 3
PLAIN, NONTEMPORAL, THROUGH = 0, 16, 32
MIB = 1 << 20


@pytest.fixture(scope="module")
def route():
    import os

    from paper_2512_22036_amd import binding
    if not os.path.exists(binding.library_path()):
        from paper_2512_22036_amd.build import build_library
        build_library()
    lib = binding.load_library()
    assert (binding.ROUTE_TOKENS, binding.ROUTE_TILES, binding.ROUTE_BOTH_BY_TILES, binding.ROUTE_TILES_THEN_TOKENS) == (TOKENS, TILES, BOTH, SEPARATE)
    assert (binding.WALK_PLAIN, binding.WALK_STREAMING, binding.WALK_THROUGH) == (PLAIN, NONTEMPORAL, THROUGH)

    def ask(N, k, E, D, row, aux=0, flags=0, at=0x10000000, wire_at=0x20000000, aux_at=0x30000000):
        L = binding._CLayout()
        assert lib.fusco_layout_bind(ctypes.byref(L), N, k, E, D, 0x10000000, lib.fusco_layout_bytes(N, k, E, D)) == 0
        return lib.fusco_probe_dispatch_route(ctypes.byref(L), row, aux, at, aux_at if aux else None, wire_at, aux_at if aux else None, flags)

    ask.lib = lib
    return ask


def test_route_agrees_with_the_transfer_order_query(route):
    from paper_2512_22036_amd import binding
    lib = route.lib
    for N, k, E, D, row in ((8192, 8, 256, 8, 14336), (1000, 8, 256, 8, 14336), (8192, 4, 64, 8, 8192), (20000, 8, 128, 16, 8192), (32768, 8, 256, 8, 14336)):
        L = binding._CLayout()
        assert lib.fusco_layout_bind(ctypes.byref(L), N, k, E, D, 0x10000000, lib.fusco_layout_bytes(N, k, E, D)) == 0
        for flags in (0, EXPERT, WIRE, EXPERT | WIRE, TWO_HOP, EXPERT | STREAMING, EXPERT | WIRE | STREAMING):
            tiled = lib.fusco_dispatch_in_transfer_order(ctypes.byref(L), row, 0, flags)
            assert (route(N, k, E, D, row, 0, flags) & 15 != TOKENS) == bool(tiled), (N, row, flags)


def test_stores_of_the_token_walk(route):
    assert route(4096, 8, 64, 8, 4096) == TOKENS | PLAIN                      # 128 MiB of rows: they stay for their reader
    assert route(4096, 8, 64, 8, 4096, 0, STREAMING) == TOKENS | NONTEMPORAL
    assert route(40000, 1, 64, 8, 8192) == TOKENS | NONTEMPORAL               # 312 MiB, one entry per token
    assert route(40000, 1, 64, 8, 8192, 0, TWO_HOP) == TOKENS | PLAIN         # the second hop reads the first one's rows
    knob = route.lib.fusco_probe_dispatch_walk
    for setting, stores in ((1, PLAIN), (2, PLAIN), (3, NONTEMPORAL), (4, NONTEMPORAL)):
        assert knob(setting) == 0
        try:
            assert route(40000, 1, 64, 8, 8192) == TOKENS | stores
        finally:
            assert knob(0) == setting


def test_rows_written_through_where_the_l2s_cannot_hold_them(route):
    for k, row in ((1, 2048), (1, 14336), (2, 2048), (2, 7168), (3, 4096)):
        first = -(-(50 * MIB) // ((k + 1) * row))   # source and rows of 50 MiB
        assert route(first, k, 64, 8, row) == TOKENS | THROUGH
        assert route(first - 1, k, 64, 8, row) == TOKENS | PLAIN
        last = 256 * MIB // (k * row)               # what is written fits the memory-side cache
        assert route(last, k, 64, 8, row) == TOKENS | THROUGH and route(last + 1, k, 64, 8, row) != TOKENS | THROUGH
    assert route(4096, 2, 16, 4, 2048) == TOKENS | PLAIN    # the smallest benchmark configuration
    assert route(16384, 4, 64, 8, 2048) == TOKENS | PLAIN


def test_rows_written_through_start_at_whole_units(route):
    for k in (2, 3):
        args = (12288, k, 64, 8, 4096)
        assert route(*args) == route(*args, at=0x10000040) == route(*args, at=0x10000080) == TOKENS | THROUGH
        for shift in (16, 32, 48, 80):   # stores of a wave would cover parts of units
            assert route(*args, at=0x10000000 + shift) == TOKENS | PLAIN
        assert route(12288, k, 64, 8, 4096 + 64) == TOKENS | PLAIN   # not rows of whole lines
    one = (24576, 1, 64, 8, 4096 + 64)
    assert route(*one) == route(*one, at=0x10000040) == TOKENS | THROUGH
    assert route(*one, at=0x10000010) == route(24576, 1, 64, 8, 4096 + 16) == TOKENS | PLAIN


def test_both_tensors_in_two_launches_from_four_devices_on(route):
    flags = EXPERT | WIRE
    for N, row in ((9216, 8256), (9000, 9280), (9300, 14336)):   # 72 to 128 MiB of source
        for D in (1, 2, 3):
            assert route(N, 8, 96, D, row, 0, flags) & 15 != SEPARATE, (N, D)
        assert route(N, 8, 96, 3, row, 0, flags) == BOTH
        for D in (4, 6, 8):   # the send rows go past the memory-side cache, with the flag and without
            assert route(N, 8, 96, D, row, 0, flags) == route(N, 8, 96, D, row, 0, flags | STREAMING) == SEPARATE | NONTEMPORAL
        assert route(N, 8, 96, 8, row + 16, 0, flags) == BOTH                       # rows of partial units
        assert route(N, 8, 96, 8, row, 0, flags, at=0x10000010) == BOTH
        assert route(N, 8, 96, 8, row, 0, flags, wire_at=0x20000020) == BOTH
    assert route(9139, 8, 96, 8, 8256, 0, flags) == BOTH                             # just below 72 MiB
    assert route(16256, 8, 96, 8, 8256, 0, flags) == SEPARATE | NONTEMPORAL          # just below 128 MiB
    assert route(16257, 8, 96, 8, 8256, 0, flags) == BOTH


def test_both_tensors_of_rows_that_fill_their_workgroups_in_two_launches_from_112_mib_on(route):
    flags = EXPERT | WIRE
    for row, devices in ((8192, (4, 5, 6, 8)), (10240, (4, 5)), (11264, (4, 5)), (12288, (4, 5, 6, 8)), (13696, (4, 5)), (14336, (4, 5)), (15360, (4, 5))):
        first = -(-(112 * MIB) // row)
        for D in devices:
            E = D * 16
            assert route(first - 1, 8, E, D, row, 0, flags) == route(73 * MIB // row, 8, E, D, row, 0, flags) == BOTH
            assert route(first, 8, E, D, row, 0, flags) == route(128 * MIB // row, 8, E, D, row, 0, flags) == SEPARATE | NONTEMPORAL
            assert route(first - 1, 8, E, D, row - 64, 64, flags) == BOTH            # both planes together
    for row, devices in ((8256, (4, 8)), (9216, (4, 8)), (10176, (4, 8)), (10240, (6, 8)), (12224, (6, 8)), (12352, (4, 8)), (13632, (4, 8)), (13696, (6, 8)), (14336, (6, 8)), (15424, (4, 8)), (16384, (4, 8))):
        for D in devices:
            assert route(73 * MIB // row, 8, D * 16, D, row, 0, flags) == SEPARATE | NONTEMPORAL


def test_bad_arguments(route):
    assert route(8192, 8, 256, 8, 0) < 0 and route(8192, 8, 256, 8, 24) < 0 and route(8192, 8, 256, 8, 16, 8) < 0
    assert route(8192, 8, 256, 8, 1 << 21) < 0 and route(8192, 8, 256, 8, 16, 0, 16) < 0 and route(8192, 8, 256, 8, 16, 0, TWO_HOP | STREAMING) < 0
    assert route.lib.fusco_probe_dispatch_route(None, 16, 0, None, None, None, None, 0) < 0
