"""Pack into slices by workgroups of either width: slices and streams on both sides of the sizes at which the wide ones are taken, streams
that end inside a workgroup, units that cannot be read, a stream longer than its capacity.  Bytes and whole numbers: no tolerance."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

KIB = 1024


def pack(total, slice_bytes, capacity, seed, holes):
    import paper_2512_22036_amd as f
    rng = np.random.default_rng(seed)
    size = []
    left = total
    while left:
        size.append(min(int(rng.choice([16, 48, 4096, 16 * rng.integers(1, 900), 70000 // 16 * 16])), left))
        left -= size[-1]
    size = np.array(size, dtype=np.int64)
    n = len(size)
    order = rng.permutation(n)
    off = np.zeros(n, dtype=np.int64)
    off[order] = np.cumsum(size[order]) - size[order]
    if holes:
        off[rng.choice(n, size=max(1, n // 10), replace=False)] = total   # behind the source: nothing of the segment can be read
    src = rng.integers(0, 256, size=total, dtype=np.uint8)
    ends = np.cumsum(size)
    want, good = np.full(max(total, capacity) + 64 * KIB, 0xEE, dtype=np.uint8), np.zeros(total, dtype=bool)
    for i in range(n):
        if off[i] < total:
            want[ends[i] - size[i]:ends[i]] = src[off[i]:off[i] + size[i]]
            good[ends[i] - size[i]:ends[i]] = True
    end = min(total, -(-capacity // (16 * KIB)) * 16 * KIB)   # whole blocks of 16 KiB
    want[end:] = 0xEE
    slices = -(-capacity // slice_bytes)
    fill_want = np.array([good[s * slice_bytes:min((s + 1) * slice_bytes, end)].sum() for s in range(slices)])
    desc = torch.from_numpy(np.stack([off, size], 1)).cuda()
    cum, status = torch.zeros(n + 1, dtype=torch.int64, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    fill = torch.full((slices,), 7, dtype=torch.int32, device="cuda")
    packed = torch.full((len(want),), 0xEE, dtype=torch.uint8, device="cuda")
    f.fusco_segments_scan(desc, cum, status)
    f.fusco_segments_copy(torch.from_numpy(src).cuda(), desc, packed, None, cum, capacity, status, slice_bytes=slice_bytes, slice_fill=fill)
    assert np.array_equal(packed.cpu().numpy(), want)
    assert np.array_equal(fill.cpu().numpy(), fill_want)
    assert int(status) == np.count_nonzero(~good[:end]) // 16


@pytest.mark.parametrize("holes", [False, True])
@pytest.mark.parametrize("slice_bytes", [16 * KIB, 32 * KIB, 48 * KIB, 64 * KIB, 80 * KIB, 96 * KIB, 1024 * KIB])
@pytest.mark.parametrize("total", [2048 * KIB - 16, 2048 * KIB, 2048 * KIB + 16, 2064 * KIB, 2080 * KIB - 4096, 3000 * KIB + 48])
def test_pack_into_slices(total, slice_bytes, holes):
    pack(total, slice_bytes, -(-total // slice_bytes) * slice_bytes, total + slice_bytes, holes)


# capacities of an odd and an even number of blocks of 16 KiB, below and above the stream's bytes
@pytest.mark.parametrize("capacity", [2048 * KIB, 2064 * KIB, 2064 * KIB - 16, 2070 * KIB, 2400 * KIB])
@pytest.mark.parametrize("slice_bytes", [48 * KIB, 64 * KIB, 1024 * KIB])
def test_streams_and_capacities_that_differ(slice_bytes, capacity):
    pack(2200 * KIB + 16, slice_bytes, capacity, capacity + slice_bytes, True)


# slices of 256 KiB from 2 MiB on, shorter ones from 64 MiB on
@pytest.mark.parametrize("slice_bytes,total", [(224 * KIB, 3000 * KIB + 48), (256 * KIB, 2048 * KIB - 16), (256 * KIB, 2300 * KIB + 16), (64 * KIB, 65536 * KIB - 80 * KIB),
                                               (64 * KIB, 65536 * KIB + 16), (128 * KIB, 65536 * KIB)])
def test_slices_on_both_sides_of_the_wide_workgroups(slice_bytes, total):
    pack(total, slice_bytes, -(-total // slice_bytes) * slice_bytes, total + slice_bytes, True)
