"""Which packs into slices are done by workgroups of twice the width, as the library's host-only query tells it from the sizes: slices in whole
blocks of such workgroups, short ones in long streams only.  No GPU is needed."""
import pytest

KIB, MIB = 1024, 1 << 20


@pytest.fixture(scope="module")
def wide():
    import os

    from paper_2512_22036_amd import binding
    if not os.path.exists(binding.library_path()):
        from paper_2512_22036_amd.build import build_library
        build_library()
    return binding.load_library().fusco_probe_segments_wide


def test_long_slices_from_2_mib_on(wide):
    for slice_bytes in (256 * KIB, 288 * KIB, MIB, 4 * MIB, 1024 * MIB):
        assert [wide(c, slice_bytes) for c in (0, 2 * MIB - 1, 2 * MIB, 18 * MIB, 64 * MIB, 1 << 40)] == [0, 0, 1, 1, 1, 1]


def test_short_slices_from_64_mib_on(wide):
    for slice_bytes in (64 * KIB, 96 * KIB, 128 * KIB, 224 * KIB):
        assert [wide(c, slice_bytes) for c in (2 * MIB, 18 * MIB, 64 * MIB - 1, 64 * MIB, 1 << 40)] == [0, 0, 0, 1, 1]


def test_slices_that_stay_with_narrow_workgroups(wide):
    for slice_bytes in (16 * KIB, 32 * KIB, 48 * KIB, 80 * KIB, 272 * KIB, MIB + 16 * KIB):
        assert [wide(c, slice_bytes) for c in (2 * MIB, 64 * MIB, 1 << 40)] == [0, 0, 0]


def test_bad_slices(wide):
    for slice_bytes in (0, 16, 16 * KIB + 16, (1 << 31) + 16 * KIB):
        assert wide(64 * MIB, slice_bytes) < 0
