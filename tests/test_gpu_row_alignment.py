"""Rows that do not consist of whole 64-byte units - by their size or by where the tensor starts - take other stores
than rows that do: tiled dispatch (both planes) and combine's output, at the sizes where the choice is made.  Moved
bytes are compared with torch.equal; combine's sums bit for bit with the oracle's (fp32 fused multiply-adds in order,
one rounding), so there is no tolerance."""
import numpy as np
import pytest
import torch

from definitions import random_topk

pytestmark = pytest.mark.gpu


def rows_at(rows, row_bytes, offset):
    """A [rows, row_bytes] byte tensor that starts `offset` bytes into its allocation, filled with 0xEE, and the whole."""
    room = torch.full((rows * row_bytes + 256,), 0xEE, dtype=torch.uint8, device="cuda")
    return room[offset:offset + rows * row_bytes].view(rows, row_bytes), room


@pytest.mark.parametrize("row_bytes,aux_bytes,offset", [(4096, 0, 0), (4096, 0, 16), (4112, 0, 0), (4160, 64, 0), (4160, 224, 0),
                                                        (4096, 128, 32), (5008, 48, 48), (48, 16, 0), (16384 + 16, 0, 16),
                                                        (12288, 0, 0), (12288, 16, 0), (13312, 0, 0), (13312, 0, 16), (13328, 0, 0)])
def test_tiled_dispatch(row_bytes, aux_bytes, offset):
    import paper_2512_22036_amd as f
    N, k, E, D = 4200, 8, 64, 8
    rng = np.random.default_rng(row_bytes + aux_bytes + offset)
    A = torch.from_numpy(random_topk(rng, N, k, E)).cuda()
    L = f.Layout(N, k, E, D)
    f.fusco_plan(L, A)
    x = torch.randint(0, 256, (N, row_bytes), dtype=torch.uint8, device="cuda")
    xa = torch.randint(0, 256, (N, aux_bytes), dtype=torch.uint8, device="cuda") if aux_bytes else None
    eb, room = rows_at(L.P, row_bytes, offset)
    ea, room_a = rows_at(L.P, aux_bytes, offset) if aux_bytes else (None, None)
    assert f.fusco_probe_dispatch_kernel(2) == 0
    try:
        assert f.fusco_dispatch_in_transfer_order(L, row_bytes, aux_bytes)
        f.fusco_dispatch(L, x, eb, x_aux=xa, expert_aux=ea)
    finally:
        f.fusco_probe_dispatch_kernel(0)
    token = L.array("slot_token").long()
    assert torch.equal(eb, x[token])
    assert bool((room[:offset] == 0xEE).all()) and bool((room[offset + eb.numel():] == 0xEE).all())
    if aux_bytes:
        assert torch.equal(ea, xa[token])
        assert bool((room_a[:offset] == 0xEE).all()) and bool((room_a[offset + ea.numel():] == 0xEE).all())


@pytest.mark.parametrize("N", [40, 2500])     # below and above 64 MiB of expert outputs
@pytest.mark.parametrize("H", [4096, 4104])
@pytest.mark.parametrize("offset", [0, 16])
@pytest.mark.parametrize("y_f32,out_f32", [(False, False), (False, True), (True, False), (True, True)])
def test_combine_output(oracle, N, H, offset, y_f32, out_f32):
    import paper_2512_22036_amd as f
    k, E, D = 8, 64, 8
    rng = np.random.default_rng(N + H)
    A = random_topk(rng, N, k, E)
    L = f.Layout(N, k, E, D)
    f.fusco_plan(L, torch.from_numpy(A).cuda())
    y = torch.randn((L.P, H), device="cuda").to(torch.float32 if y_f32 else torch.bfloat16)
    w = torch.rand((N, k), device="cuda")
    kind = torch.float32 if out_f32 else torch.bfloat16
    out, room = rows_at(N, H * (4 if out_f32 else 2), offset)
    out = out.view(kind)
    f.fusco_combine(L, y, w, out)
    slots = L.array("pair_slot").cpu().numpy()
    few = np.unique(rng.integers(0, N, size=64))           # the oracle is slow: some tokens, first and last among them
    few[0], few[-1] = 0, N - 1
    pick = torch.from_numpy(slots.reshape(N, k)[few].reshape(-1)).cuda().long()
    rows = y[pick].cpu()
    rows = rows.numpy() if y_f32 else rows.view(torch.int16).numpy().view(np.uint16)
    want32, want16 = oracle.combine_f32(rows, w[torch.from_numpy(few).cuda()].cpu().numpy(),
                                        np.arange(len(few) * k, dtype=np.int32))
    got = out[torch.from_numpy(few).cuda()].cpu()
    if out_f32:
        assert np.array_equal(got.numpy().view(np.uint32), want32.view(np.uint32))
    else:
        assert np.array_equal(got.view(torch.int16).numpy().view(np.uint16), want16)
    # the others against the same sum in plain torch: k products and sums of one rounding each
    exact = (w[:, :, None].double() * y[torch.from_numpy(slots).cuda().long()].view(N, k, H).double()).sum(1) if N < 100 else None
    if exact is not None:
        size = (w[:, :, None].double() * y[torch.from_numpy(slots).cuda().long()].view(N, k, H).double().abs()).sum(1)
        bound = size * k * 2.0 ** -24 + (0 if out_f32 else exact.abs() * 2.0 ** -8)
        assert bool(((out.double() - exact).abs() <= bound).all())
    assert bool((room[:offset] == 0xEE).all()) and bool((room[offset + out.numel() * out.element_size():] == 0xEE).all())


# rows of more than 256 or 512 chunks of small inputs are cut into segments of 64 or 128 threads, two-hop rows into segments of 256:
# row lengths around their edges, token counts on either side of 512 workgroups, the last and the first size past the limits
# (64 MiB of experts' outputs; 48 MiB two-hop)
@pytest.mark.parametrize("two_hop", [False, True])
@pytest.mark.parametrize("N,k,C", [(1, 8, 513), (1, 1, 512), (3, 6, 575), (7, 8, 577), (63, 8, 1024), (64, 8, 1024), (65, 3, 1025), (102, 2, 640),
                                   (103, 2, 639), (5, 5, 2049), (511, 8, 1024), (512, 8, 1024), (383, 8, 1024), (384, 8, 1024), (1000, 2, 896), (64, 8, 256), (64, 8, 257), (127, 8, 512),
                                   (128, 8, 512), (170, 4, 384), (171, 4, 384)])
@pytest.mark.parametrize("y_f32,out_f32", [(False, False), (False, True), (True, False)])
def test_combine_of_small_inputs_in_column_segments(N, k, C, two_hop, y_f32, out_f32):
    import paper_2512_22036_amd as f
    E, D = 64, 8
    H = C * (4 if y_f32 else 8)
    rng = np.random.default_rng(N + C)
    L = f.Layout(N, k, E, D)
    f.fusco_plan(L, torch.from_numpy(random_topk(rng, N, k, E)).cuda())
    y = torch.randint(-127, 128, (L.P, H), device="cuda").to(torch.float32 if y_f32 else torch.bfloat16)
    w = torch.full((N, k), 0.125, device="cuda")      # whole numbers and a power of two: every sum is exact
    kind = torch.float32 if out_f32 else torch.bfloat16
    out, room = rows_at(N, H * (4 if out_f32 else 2), 0)
    out = out.view(kind)
    if two_hop:
        f.fusco_combine_two_hop(L, y, w, torch.empty((L.send_cap, H), device="cuda"), out)
    else:
        f.fusco_combine(L, y, w, out)
    want = torch.zeros((N, H), dtype=torch.float32, device="cuda")
    for rows in L.array("pair_slot").view(N, k).long().t():
        want += y[rows].float()
    assert torch.equal(out, (want / 8).to(kind))
    assert bool((room[out.numel() * out.element_size():] == 0xEE).all())


# 128 MiB of input and output are the most that leave the output in the memory-side cache (1820 tokens with rows of 8 KiB,
# 1816 with rows of 8208 B, which are not whole 64-byte units)
@pytest.mark.parametrize("N,H", [(1820, 4096), (1821, 4096), (1816, 4104), (1817, 4104), (4097, 4096),
                                 (1023, 7168), (1024, 7168)])
@pytest.mark.parametrize("two_hop", [False, True])
def test_combine_output_around_the_size_that_goes_past_the_cache(N, H, two_hop):
    import paper_2512_22036_amd as f
    k, E, D = 8, 64, 8
    rng = np.random.default_rng(N)
    L = f.Layout(N, k, E, D)
    f.fusco_plan(L, torch.from_numpy(random_topk(rng, N, k, E)).cuda())
    y = torch.randn((L.P, H), device="cuda").to(torch.bfloat16)
    w = torch.full((N, k), 0.125, device="cuda")      # an exact mean of eight: any order of exact sums rounds the same
    y = (y * 16).round().clamp(-127, 127)             # whole numbers: every partial sum is exact
    out, room = rows_at(N, H * 2, 0)
    out = out.view(torch.bfloat16)
    if two_hop:
        f.fusco_combine_two_hop(L, y, w, torch.empty((L.send_cap, H), device="cuda"), out)
    else:
        f.fusco_combine(L, y, w, out)
    want = torch.zeros((N, H), dtype=torch.float32, device="cuda")
    for rows in L.array("pair_slot").view(N, k).long().t():
        want += y[rows].float()
    assert torch.equal(out, (want / 8).to(torch.bfloat16))
    assert bool((room[out.numel() * 2:] == 0xEE).all())


@pytest.mark.parametrize("N,k,E,D,row_bytes,aux_bytes,limit", [
    (4200, 8, 256, 8, 8448, 0, 0),              # 17 tiles, the last one ragged; as many devices as entries
    (4200, 8, 64, 4, 8192 + 16, 64, 0),         # rows that are not whole units, a second plane
    (2300, 16, 64, 2, 8192, 0, 0),              # two devices: nearly every token has a row on both; 128 tokens per tile
    (4200, 8, 64, 1, 8448, 48, 0),              # one device
    (4200, 8, 64, 8, 16384 + 1040, 0, 0),       # two column segments
    (4200, 8, 256, 8, 8448, 0, 16 << 20),       # source rows taken in chunks of 8 tiles
])
def test_both_tensors_tile_by_tile(N, k, E, D, row_bytes, aux_bytes, limit):
    """Expert tensor of more than 256 MB and the receive tensors in one call: large enough for the tiles by itself.
    Invalid ids and repeated experts among the entries; rows past the last send row stay untouched."""
    import paper_2512_22036_amd as f
    rng = np.random.default_rng(N + D)
    A = random_topk(rng, N, k, E, distinct=False)
    A[7, 2], A[N - 1, 0] = -1, E
    L = f.Layout(N, k, E, D)
    f.fusco_plan(L, torch.from_numpy(A).cuda())
    x = torch.randint(0, 256, (N, row_bytes), dtype=torch.uint8, device="cuda")
    xa = torch.randint(0, 256, (N, aux_bytes), dtype=torch.uint8, device="cuda") if aux_bytes else None

    def filled(rows, width):
        return torch.full((rows, width), 0xEE, dtype=torch.uint8, device="cuda") if width else None

    got = dict(expert_buf=filled(L.P, row_bytes), expert_aux=filled(L.P, aux_bytes), send_buf=filled(L.send_cap, row_bytes),
               send_aux=filled(L.send_cap, aux_bytes))
    before = f.fusco_probe_source_chunk_bytes(limit) if limit else 0
    try:
        assert f.fusco_dispatch_in_transfer_order(L, row_bytes, aux_bytes, f.DISPATCH_EXPERT | f.DISPATCH_WIRE)
        f.fusco_dispatch(L, x, x_aux=xa, flags=f.DISPATCH_EXPERT | f.DISPATCH_WIRE, **got)
    finally:
        if limit:
            f.fusco_probe_source_chunk_bytes(before)
    valid = L.P - int(L.array("status").item())
    U = int(L.array("send_off")[D].item())
    token, source = L.array("slot_token")[:valid].long(), L.array("send_src")[:U].long()
    assert torch.equal(got["expert_buf"][:valid], x[token]) and bool((got["expert_buf"][valid:] == 0xEE).all())
    assert torch.equal(got["send_buf"][:U], x[source]) and bool((got["send_buf"][U:] == 0xEE).all())
    if aux_bytes:
        assert torch.equal(got["expert_aux"][:valid], xa[token]) and torch.equal(got["send_aux"][:U], xa[source])
        assert bool((got["expert_aux"][valid:] == 0xEE).all()) and bool((got["send_aux"][U:] == 0xEE).all())


def test_both_tensors_tile_by_tile_over_random_shapes():
    """40 random shapes at which the library itself moves both tensors tile by tile: many or few devices, long and short
    rows, one or several column segments, a second plane, a ragged last tile, invalid ids and repeated experts."""
    import paper_2512_22036_amd as f
    both = f.DISPATCH_EXPERT | f.DISPATCH_WIRE
    rng = np.random.default_rng(31)
    seen, moved = set(), 0
    for case in range(40):
        few = case % 2 == 1                       # at most 2 devices: any k, rows that a workgroup holds whole
        k = int(rng.choice([2, 3, 5, 6, 8, 16] if few else [8, 9, 10, 16, 24, 33, 64]))
        D = int(rng.integers(1, 3)) if few else int(rng.integers(1, 9))
        E = D * int(rng.integers(max(1, 16 // D), 33))
        tokens = 2048 // k                        # per tile
        row = 16 * int(rng.integers(1, 3840 * 64 // tokens + 1) if few else rng.integers(512, 2600))
        aux = 16 * int(rng.choice([0, 0, 1, 3, 14]))
        if few:
            row = max(16 if k >= 8 else 4096, min(row, 16384 - 256) - aux)
        if case == 5:
            k, tokens, row, aux = 8, 256, 64, 0   # one wave per row
        N = max(17 * tokens, (256 << 20) // (k * (row + aux))) + int(rng.integers(1, 2 * tokens))
        tag = "case %d: N=%d k=%d E=%d D=%d row=%d aux=%d" % (case, N, k, E, D, row, aux)
        L = f.Layout(N, k, E, D)
        if not f.fusco_dispatch_in_transfer_order(L, row, aux, both):
            continue                              # a large source tensor of short rows, few entries per token: the walk
        A = torch.randint(0, E, (N, k), dtype=torch.int32, device="cuda")
        A[0, 0], A[N // 2, k - 1], A[N - 1, 1] = -1, E, -7
        f.fusco_plan(L, A)
        x = torch.randint(0, 256, (N, row), dtype=torch.uint8, device="cuda")
        xa = torch.randint(0, 256, (N, aux), dtype=torch.uint8, device="cuda") if aux else None

        def filled(rows, width):
            return torch.full((rows, width), 0xEE, dtype=torch.uint8, device="cuda") if width else None

        eb, ea, sb, sa = filled(L.P, row), filled(L.P, aux), filled(L.send_cap, row), filled(L.send_cap, aux)
        f.fusco_dispatch(L, x, eb, x_aux=xa, expert_aux=ea, send_buf=sb, send_aux=sa, flags=both)
        valid, U = L.P - 3, int(L.array("send_off")[D].item())
        assert int(L.array("status").item()) == 3, tag
        token, source = L.array("slot_token")[:valid].long(), L.array("send_src")[:U].long()
        for src, expert, send in ((x, eb, sb), (xa, ea, sa)):
            if src is not None:
                assert torch.equal(expert[:valid], src[token]) and bool((expert[valid:] == 0xEE).all()), tag
                assert torch.equal(send[:U], src[source]) and bool((send[U:] == 0xEE).all()), tag
        moved += 1
        seen.add((few, -(-(row + aux) // 16) > 1024, aux > 0, (row + aux) // 16 < 512))
    assert moved >= 35 and len(seen) >= 6 and any(s[0] for s in seen) and any(s[1] for s in seen)


# the token walk of few workgroups (up to 1024 of a row's column segments) and the one of many, both ends of the rule; send rows alone go by
# their size and number (8 devices); every pairing of loads and stores
@pytest.mark.parametrize("N,k,row_bytes,aux_bytes", [(1, 1, 16, 0), (7, 64, 48, 16), (300, 8, 4112, 0), (1024, 3, 1040, 224), (1025, 3, 1040, 224),
                                                     (512, 4, 16384 + 16, 0), (513, 4, 16384 + 16, 0), (30, 6, 40000, 32), (90, 8, 16368, 48),
                                                     (1200, 2, 2064, 0), (1201, 2, 1520, 16), (1201, 2, 1520, 32), (1201, 1, 4784, 0), (1201, 1, 4784, 16),
                                                     (1300, 23, 4096, 0), (1300, 24, 4096, 0), (1300, 24, 4112, 0),
                                                     (5999, 2, 2032, 16), (6000, 2, 2032, 16), (3999, 2, 12288, 0), (4000, 2, 12288, 0), (4000, 2, 12256, 16)])
@pytest.mark.parametrize("flags", [1, 2, 3])
def test_token_walk(N, k, row_bytes, aux_bytes, flags):
    import paper_2512_22036_amd as f
    E, D = 128, 8
    rng = np.random.default_rng(N + row_bytes)
    A = random_topk(rng, N, k, E).astype(np.int32)
    if N > 1:
        A[N // 2] = -1                     # a token without a row, and one without its first entry
        A[N // 3, 0] = E
    L = f.Layout(N, k, E, D)
    f.fusco_plan(L, torch.from_numpy(A).cuda())
    x = torch.randint(0, 256, (N, row_bytes), dtype=torch.uint8, device="cuda")
    xa = torch.randint(0, 256, (N, aux_bytes), dtype=torch.uint8, device="cuda") if aux_bytes else None
    rows, sends = int(L.array("exp_off")[E]), int(L.array("send_off")[D])
    token, src = L.array("slot_token")[:rows].long(), L.array("send_src")[:sends].long()
    assert not f.fusco_dispatch_in_transfer_order(L, row_bytes, aux_bytes, flags)
    for mode in range(5):
        eb, room = rows_at(L.P, row_bytes, 0)
        sb, room_s = rows_at(L.send_cap, row_bytes, 16)
        ea, _ = rows_at(L.P, max(aux_bytes, 16), 0)
        sa, _ = rows_at(L.send_cap, max(aux_bytes, 16), 0)
        planes = dict(x_aux=xa, expert_aux=ea, send_aux=sa) if aux_bytes else {}
        assert f.fusco_probe_dispatch_walk(mode) == 0
        try:
            f.fusco_dispatch(L, x, eb, send_buf=sb, flags=flags, **planes)
        finally:
            f.fusco_probe_dispatch_walk(0)
        want = rows if flags & 1 else 0
        assert torch.equal(eb[:want], x[token[:want]]) and bool((room[want * row_bytes:] == 0xEE).all())
        want = sends if flags & 2 else 0
        assert torch.equal(sb[:want], x[src[:want]]) and bool((room_s[16 + want * row_bytes:] == 0xEE).all())
        if aux_bytes:
            assert torch.equal(ea[:rows if flags & 1 else 0], xa[token[:rows if flags & 1 else 0]])
            assert torch.equal(sa[:sends if flags & 2 else 0], xa[src[:sends if flags & 2 else 0]])


# rows in flight by the number of waves (4096 and 32768) and by k, for inputs on either side of 64 MiB; k = 1 and 2 have kernels of their own
@pytest.mark.parametrize("N,k,H", [(1000, 64, 1024), (2047, 32, 1024), (2048, 32, 1024), (1170, 8, 7168), (1171, 8, 7168), (8191, 8, 1024), (8192, 8, 1024),
                                   (4681, 8, 3584), (4682, 8, 3584), (4500, 1, 8192), (4500, 2, 8192), (300, 1, 520), (300, 2, 520), (2100, 3, 4096), (2900, 3, 4096)])
def test_combine_by_waves(N, k, H):
    import paper_2512_22036_amd as f
    E, D = 64, 8
    rng = np.random.default_rng(N + k)
    A = random_topk(rng, N, k, E).astype(np.int32)
    A[1::7, 0] = -1                       # an entry without a row
    L = f.Layout(N, k, E, D)
    f.fusco_plan(L, torch.from_numpy(A).cuda())
    y = torch.randint(-15, 16, (L.P, H), device="cuda").to(torch.bfloat16)
    w = torch.full((N, k), 0.5, device="cuda")        # whole numbers and a power of two: every sum is exact
    out, room = rows_at(N, H * 4, 0)
    out = out.view(torch.float32)
    f.fusco_combine(L, y, w, out)
    want = torch.zeros((N, H), dtype=torch.float32, device="cuda")
    for rows in L.array("pair_slot").view(N, k).long().t():
        want += torch.where((rows >= 0)[:, None], y[rows.clamp_min(0)].float(), 0.0)
    assert torch.equal(out, want / 2)
    assert bool((room[out.numel() * 4:] == 0xEE).all())


# entries taken eight or four at a time with every number of them left over, absent ones among them; below and above 16 and 32 MiB, and below
# and above the 4, 42 and 64 MiB between which fp32 rows are spaced
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 6, 7, 8, 9, 11, 13, 14, 15, 16, 19, 23, 24, 29, 64])
@pytest.mark.parametrize("y_f32", [False, True])
@pytest.mark.parametrize("mib", [1, 4.2, 12, 18, 31, 40, 44, 66])
def test_combine_with_entries_left_over(k, y_f32, mib):
    import paper_2512_22036_amd as f
    E, D, H = 64, 8, 520
    N = max(3, int(mib * 2 ** 20) // (k * H * (4 if y_f32 else 2)))
    rng = np.random.default_rng(k + int(mib))
    A = random_topk(rng, N, k, E).astype(np.int32)
    A[rng.random((N, k)) < 0.2] = -1      # any number of entries with a row, in any place
    L = f.Layout(N, k, E, D)
    f.fusco_plan(L, torch.from_numpy(A).cuda())
    y = torch.randint(-15, 16, (L.P, H), device="cuda").to(torch.float32 if y_f32 else torch.bfloat16)
    w = torch.full((N, k), 0.5, device="cuda")        # whole numbers and a power of two: every sum is exact
    out, room = rows_at(N, H * 4, 0)
    out = out.view(torch.float32)
    f.fusco_combine(L, y, w, out)
    want = torch.zeros((N, H), dtype=torch.float32, device="cuda")
    for rows in L.array("pair_slot").view(N, k).long().t():
        want += torch.where((rows >= 0)[:, None], y[rows.clamp_min(0)].float(), 0.0)
    assert torch.equal(out, want / 2)
    assert bool((room[out.numel() * 4:] == 0xEE).all())


# two-hop combine around its limits: 11, 20, 48, 64 and 96 MiB of input, 3000 tokens, 4500, 7000 and 16384 waves, rows of 144, 352 and 400 chunks; capped workgroups of 1 to 16 waves,
# one and two devices; fp32 rows beside them
@pytest.mark.parametrize("N,k,C,D", [(2250, 4, 80, 4), (2249, 4, 84, 4), (2250, 4, 75, 4), (1000, 4, 327, 4), (1000, 4, 328, 4), (500, 7, 352, 8), (500, 7, 353, 8),
                                     (400, 5, 640, 8), (900, 8, 436, 8), (900, 8, 437, 8), (8191, 6, 79, 4), (8192, 6, 79, 4), (8192, 3, 250, 8), (8195, 3, 256, 8),
                                     (50000, 2, 64, 4), (13000, 2, 256, 4), (13000, 2, 257, 4), (50000, 1, 128, 8), (25000, 4, 64, 1), (25000, 4, 63, 2), (12600, 8, 65, 8),
                                     (4000, 4, 400, 8), (2600, 6, 410, 8), (3200, 4, 520, 4), (2000, 8, 576, 8), (2700, 4, 600, 2), (2000, 5, 670, 2), (1800, 3, 1200, 8),
                                     (9000, 3, 256, 3), (9000, 3, 256, 4), (800, 8, 1040, 8), (2999, 6, 50, 8), (3000, 6, 50, 8),
                                     (1749, 6, 256, 8), (1750, 6, 256, 8), (500, 8, 1000, 8), (550, 8, 1000, 8),
                                     (2500, 5, 143, 8), (2500, 5, 144, 8), (1400, 8, 399, 8), (1400, 8, 400, 8), (600, 4, 546, 2), (600, 4, 547, 2)])
@pytest.mark.parametrize("y_f32,out_f32", [(False, False), (False, True), (True, True)])
def test_two_hop_around_its_limits(N, k, C, D, y_f32, out_f32):
    import paper_2512_22036_amd as f
    E, H = 24, C * (4 if y_f32 else 8)
    rng = np.random.default_rng(N + C)
    A = random_topk(rng, N, k, E).astype(np.int32)
    A[1::5, 0] = -1                       # an entry without a row
    L = f.Layout(N, k, E, D)
    f.fusco_plan(L, torch.from_numpy(A).cuda())
    y = torch.randint(-15, 16, (L.P, H), device="cuda").to(torch.float32 if y_f32 else torch.bfloat16)
    w = torch.full((N, k), 0.5, device="cuda")        # whole numbers and a power of two: every sum is exact
    kind = torch.float32 if out_f32 else torch.bfloat16
    out, room = rows_at(N, H * (4 if out_f32 else 2), 0)
    out = out.view(kind)
    partial = torch.full((L.send_cap, H), -1.0, device="cuda")
    f.fusco_combine_two_hop(L, y, w, partial, out)
    slots, sends = L.array("pair_slot").view(N, k).long(), L.array("pair_send_row").view(N, k).long()
    want, want_partial = torch.zeros((N, H), device="cuda"), torch.zeros((L.send_cap, H), device="cuda")
    for rows, send in zip(slots.t(), sends.t()):
        here = rows >= 0
        term = y[rows[here]].float() / 2
        want[here] += term
        want_partial[send[here]] += term   # a token has one row per device: no index twice
    assert torch.equal(out, want.to(kind))
    U = int(L.array("send_off")[D].item())
    assert torch.equal(partial[:U], want_partial[:U]) and bool((partial[U:] == -1).all())
    assert bool((room[out.numel() * out.element_size():] == 0xEE).all())


# send rows alone on one and two devices: few rows of many entries
@pytest.mark.parametrize("N,k,D,row_bytes", [(1500, 3, 1, 20000), (1499, 3, 1, 20000), (1500, 2, 1, 20000), (1300, 6, 2, 4096), (1300, 6, 2, 4112), (1300, 5, 2, 4096)])
def test_token_walk_of_send_rows_on_few_devices(N, k, D, row_bytes):
    import paper_2512_22036_amd as f
    rng = np.random.default_rng(N + k)
    A = random_topk(rng, N, k, 16).astype(np.int32)
    A[N // 2] = -1
    L = f.Layout(N, k, 16, D)
    f.fusco_plan(L, torch.from_numpy(A).cuda())
    x = torch.randint(0, 256, (N, row_bytes), dtype=torch.uint8, device="cuda")
    sb, room = rows_at(L.send_cap, row_bytes, 16)
    f.fusco_dispatch(L, x, send_buf=sb, flags=2)
    U = int(L.array("send_off")[D])
    assert torch.equal(sb[:U], x[L.array("send_src")[:U].long()])
    assert bool((room[16 + U * row_bytes:] == 0xEE).all())
