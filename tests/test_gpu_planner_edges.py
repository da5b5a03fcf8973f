"""The planner's kernels at the sizes where their work is split - rounds and waves of the single-tile planner, its
workgroups of eight pairs, tiles, invalid ids and repeated experts anywhere - against the descriptors worked out by
sorting.  All whole numbers: no tolerance."""
import numpy as np
import pytest
import torch

from definitions import random_topk

pytestmark = pytest.mark.gpu


def plan_by_sorting(A, E, D):
    """Every descriptor array; entries that no valid pair assigns are None or cut off."""
    N, k = A.shape
    e = A.reshape(-1).astype(np.int64)
    ok = (e >= 0) & (e < E)
    pair = np.arange(N * k)
    token, dev = pair // k, np.where(ok, e // (E // D), -1)
    order = pair[ok][np.argsort(e[ok], kind="stable")]
    slot = np.full(N * k, -1)
    slot[order] = np.arange(len(order))
    # one row per (device, token), devices first; first: the pair that comes first among those of a (token, device)
    rows, first_at = np.unique(dev[ok] * N + token[ok], return_index=True)
    row = np.full(N * k, -1)
    row[ok] = np.searchsorted(rows, dev[ok] * N + token[ok])
    first = np.zeros(N * k, dtype=np.uint8)
    first[pair[ok][first_at]] = 1
    count = np.bincount(e[ok], minlength=E)
    sends = np.bincount(rows // N, minlength=D) if len(rows) else np.zeros(D, dtype=np.int64)
    return dict(exp_count=count, exp_off=np.concatenate([[0], np.cumsum(count)]), send_count=sends,
                send_off=np.concatenate([[0], np.cumsum(sends)]), pair_slot=slot, pair_send_row=row, pair_first=first,
                slot_pair=order, slot_token=order // k, slot_send_row=row[order], send_src=rows % N,
                status=np.array([np.count_nonzero(~ok)])), ok


def check(L, A, tag):
    want, ok = plan_by_sorting(A, L.E, L.D)
    got = L.to_host()
    for name, w in want.items():
        assert np.array_equal(getattr(got, name)[:len(w)], w), (tag, name)
    cap = L.tile_tokens * L.k
    for i in range(L.tile_count):
        s = want["pair_slot"][i * cap:(i + 1) * cap]
        s = np.sort(s[s >= 0])
        tile = got.tile_slots[i * cap:(i + 1) * cap]
        assert np.array_equal(tile[:len(s)], s) and np.all(tile[len(s):] == -1), (tag, "tile", i)


def routing(seed, N, k, E, distinct, bad):
    rng = np.random.default_rng(seed)
    A = random_topk(rng, N, k, E, distinct)
    if bad:
        flat = A.reshape(-1)
        at = rng.choice(len(flat), size=max(1, len(flat) // 9), replace=False)
        flat[at] = rng.choice([-1, E, np.iinfo(np.int32).max, np.iinfo(np.int32).min], size=len(at))
        A = flat.reshape(N, k)
    return np.ascontiguousarray(A, dtype=np.int32)


SINGLE_TILE = [(N, k, E, D) for k, E, D in [(1, 64, 8), (3, 24, 24), (7, 1024, 64), (8, 256, 8), (33, 96, 4), (64, 1024, 1024)]
               for N in sorted({1, 2, 64 // k, 8 * (64 // k), 8 * (64 // k) + 1, 1024 // k, 2048 // k})]


@pytest.mark.parametrize("bad", [False, True])
@pytest.mark.parametrize("N,k,E,D", SINGLE_TILE)
def test_single_tile_planner(N, k, E, D, bad):
    import paper_2512_22036_amd as f
    distinct = (N + k) % 2 == 0 and k <= E
    A = routing(N * 64 + k, N, k, E, distinct, bad)
    d_A = torch.from_numpy(A).cuda()
    L = f.Layout(N, k, E, D)
    assert L.tile_count == 1
    L.mem.fill_(0x7B)
    f.fusco_plan(L, d_A)
    check(L, A, "plan")
    # in one launch with the dispatch: the same descriptors, and the rows on their slots and nowhere else
    F = f.Layout(N, k, E, D)
    F.mem.fill_(0x7B)
    x = torch.randint(0, 256, (N, 48), dtype=torch.uint8, device="cuda")
    rows = torch.full((N * k, 48), 0xEE, dtype=torch.uint8, device="cuda")
    f.fusco_plan_dispatch(F, d_A, x, rows)
    assert torch.equal(F.mem, L.mem)
    want, ok = plan_by_sorting(A, E, D)
    n = len(want["slot_token"])
    assert torch.equal(rows[:n], x[torch.from_numpy(want["slot_token"]).cuda()])
    assert bool((rows[n:] == 0xEE).all())


# tiles read one by one with the requested rows alone and with more (37 and more), with a chunk level (96 and more) whose
# last chunk is ragged; rounds of whole tokens that fill a wave or not; more columns of counts than threads
SEVERAL_TILES = [(257, 8, 256, 8), (683, 3, 24, 24), (293, 7, 1024, 64), (129, 33, 96, 4), (65, 64, 1024, 1024), (2049, 1, 64, 8),
                 (9500, 8, 256, 8), (3000, 33, 1024, 1024), (24577, 8, 256, 64), (65900, 3, 24, 8), (7000, 33, 640, 640),
                 (220000, 1, 16, 4)]


@pytest.mark.parametrize("bad", [False, True])
@pytest.mark.parametrize("N,k,E,D", SEVERAL_TILES)
def test_several_tiles(N, k, E, D, bad):
    import paper_2512_22036_amd as f
    A = routing(N + k, N, k, E, not bad, bad)
    if bad:
        A[N // 3:N // 3 + 2048 // k + 1] = E - 1   # a tile of one expert: every pair of a wave has the same key
    L = f.Layout(N, k, E, D)
    assert L.tile_count > 1
    L.mem.fill_(0x7B)
    f.fusco_plan(L, torch.from_numpy(A).cuda())
    check(L, A, "plan")


# a few tiles in one launch: every width of the reads (by k and by where the routing lies), both ends of the sizes and one past
# them, ragged last tiles and eighths of tiles, devices in one and in both halves of the mask, one past the mask
@pytest.mark.parametrize("offset", [0, 1, 2])
@pytest.mark.parametrize("N,k,E,D", [(2049, 1, 16, 1), (8192, 1, 64, 32), (8193, 1, 64, 64), (1025, 2, 16, 4), (8192, 2, 128, 64),
                                     (8192, 3, 96, 8), (6144, 4, 60, 4), (6145, 4, 64, 8), (5000, 5, 160, 5), (1537, 6, 160, 5),
                                     (293, 7, 1024, 64), (257, 8, 256, 8), (4096, 8, 256, 64), (4097, 8, 256, 8), (3000, 8, 1023, 33),
                                     (2000, 10, 384, 8), (129, 16, 64, 2), (2048, 16, 1024, 64), (2000, 12, 130, 65), (150, 17, 96, 4),
                                     # the most pairs of one launch and the next size: 20480 (k <= 4), 24576
                                     (6826, 3, 96, 8), (6827, 3, 96, 8), (5120, 4, 60, 4), (5121, 4, 64, 8), (4915, 5, 160, 5), (4916, 5, 160, 5),
                                     (3072, 8, 256, 64), (3073, 8, 256, 8), (1536, 16, 1024, 64), (1537, 16, 1024, 64)])
def test_few_tiles(N, k, E, D, offset):
    import paper_2512_22036_amd as f
    for bad in (False, True):
        A = routing(N + k + offset, N, k, E, not bad, bad)
        if bad:
            A[N // 2:N // 2 + 300] = 0   # one expert many times
        flat = torch.zeros(N * k + 4, dtype=torch.int32, device="cuda")
        d_A = flat[offset:offset + N * k].view(N, k)
        d_A.copy_(torch.from_numpy(A))
        L = f.Layout(N, k, E, D)
        assert L.tile_count > 1
        L.mem.fill_(0x7B)
        f.fusco_plan(L, d_A)
        check(L, A, "plan")


@pytest.mark.parametrize("row_bytes,aux_bytes", [(32768 - 16, 0), (32768, 0), (32768 + 16, 0), (32768, 16), (32752, 48), (65536, 0),
                                                 (65536 + 16, 32), (40960, 32768 + 16), (98304 + 1040, 224)])
@pytest.mark.parametrize("N,k,E,D", [(1, 8, 256, 8), (5, 3, 24, 24), (31, 64, 512, 8), (300, 6, 160, 5)])
def test_single_launch_with_long_rows(N, k, E, D, row_bytes, aux_bytes):
    """Rows around the 32 KiB that a workgroup of the fused call holds, and rows in several column segments, the second
    plane beginning anywhere in a segment."""
    import paper_2512_22036_amd as f
    A = routing(N + row_bytes, N, k, E, False, N > 4)
    d_A = torch.from_numpy(A).cuda()
    F = f.Layout(N, k, E, D)
    F.mem.fill_(0x7B)
    planes = {}
    for name, width in (("x", row_bytes), ("x_aux", aux_bytes)):
        if width:
            planes[name] = torch.randint(0, 256, (N, width), dtype=torch.uint8, device="cuda")
            planes["expert_buf" if name == "x" else "expert_aux"] = torch.full((N * k + 1, width), 0xEE, dtype=torch.uint8, device="cuda")
    f.fusco_plan_dispatch(F, d_A, **planes)
    check(F, A, "fused")
    want, ok = plan_by_sorting(A, E, D)
    token = torch.from_numpy(want["slot_token"]).cuda()
    for src, dst in (("x", "expert_buf"), ("x_aux", "expert_aux")):
        if src in planes:
            assert torch.equal(planes[dst][:len(token)], planes[src][token])
            assert bool((planes[dst][len(token):] == 0xEE).all())


@pytest.mark.parametrize("row_bytes,aux_bytes", [(2048, 0), (8192, 0), (8192, 16), (16384, 0), (16384, 64)])
@pytest.mark.parametrize("N", [613, 614, 818, 819])
def test_single_launch_by_resident_workgroups(N, row_bytes, aux_bytes):
    """768, 769, 1024 and 1025 workgroups of the fused call (the chip holds three or four on a compute unit), with one, two
    and four chunks per thread, a second plane."""
    import paper_2512_22036_amd as f
    k, E, D = 2, 64, 8
    assert 1 + -(-N * k // 8) + N in (768, 769, 1024, 1025)
    A = routing(N + row_bytes, N, k, E, False, True)
    L = f.Layout(N, k, E, D)
    L.mem.fill_(0x7B)
    planes = {}
    for name, width in (("x", row_bytes), ("x_aux", aux_bytes)):
        if width:
            planes[name] = torch.randint(0, 256, (N, width), dtype=torch.uint8, device="cuda")
            planes["expert_buf" if name == "x" else "expert_aux"] = torch.full((N * k, width), 0xEE, dtype=torch.uint8, device="cuda")
    f.fusco_plan_dispatch(L, torch.from_numpy(A).cuda(), **planes)
    check(L, A, "fused")
    token = torch.from_numpy(plan_by_sorting(A, E, D)[0]["slot_token"]).cuda()
    for src, dst in (("x", "expert_buf"), ("x_aux", "expert_aux")):
        if src in planes:
            assert torch.equal(planes[dst][:len(token)], planes[src][token])
            assert bool((planes[dst][len(token):] == 0xEE).all())


def test_calls_without_a_stream_use_the_current_one():
    from paper_2512_22036_amd import binding
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert binding._stream(None) == side.cuda_stream
    assert binding._stream(None) == torch.cuda.current_stream().cuda_stream
    assert binding._stream(side) == side.cuda_stream
