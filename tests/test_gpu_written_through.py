"""Dispatches whose rows are written through the L2: both sides of the sizes and row widths at which that is chosen, with and without a
second plane, rows that end anywhere in a workgroup, the memory behind the rows untouched.  Bytes: no tolerance."""
import numpy as np
import pytest
import torch

from definitions import random_topk

pytestmark = pytest.mark.gpu


def setup(N, k, E, D, row_bytes, aux_bytes, shift):
    import paper_2512_22036_amd as f
    rng = np.random.default_rng(N + k + row_bytes)
    A = random_topk(rng, N, k, E)
    A[N // 2, 0] = -1   # an entry without an expert: its slot is nobody's
    planes = {}
    for name, width in (("x", row_bytes), ("x_aux", aux_bytes)):
        if width:
            planes[name] = torch.randint(0, 256, (N, width), dtype=torch.uint8, device="cuda")
            mem = torch.full(((N * k + 1) * width + shift,), 0xEE, dtype=torch.uint8, device="cuda")
            planes["expert_buf" if name == "x" else "expert_aux"] = mem[shift:].view(N * k + 1, width)
    return f, f.Layout(N, k, E, D), torch.from_numpy(A).cuda(), planes


def check(L, planes):
    got = L.to_host()
    n = int(got.exp_off[-1])
    assert n == L.P - 1
    token = torch.from_numpy(got.slot_token[:n].astype(np.int64)).cuda()
    for src, dst in (("x", "expert_buf"), ("x_aux", "expert_aux")):
        if src in planes:
            assert torch.equal(planes[dst][:n], planes[src][token])
            assert bool((planes[dst][n:] == 0xEE).all())


# 2 MiB of rows; up to 384 KiB written by a workgroup; 16 MiB of rows that are no whole 64-byte units; one, two, four chunks a thread and column segments;
# 3 x 256 and 4 x 256 workgroups
@pytest.mark.parametrize("N,k,row_bytes,aux_bytes", [(128, 8, 2032, 0), (128, 8, 2048, 0), (128, 8, 2048, 224), (127, 8, 2064, 48), (100, 4, 16384 + 16, 16),
                                                     (24, 16, 24576, 0), (24, 16, 24576 + 16, 0), (128, 8, 16384, 0), (128, 8, 16400, 0), (127, 8, 16400, 0),
                                                     (64, 8, 40960, 64), (682, 3, 1040, 0), (818, 2, 8192, 16), (2048, 1, 8208, 0)])
@pytest.mark.parametrize("shift", [0, 16])
def test_fused(N, k, row_bytes, aux_bytes, shift):
    f, L, A, planes = setup(N, k, 64, 8, row_bytes, aux_bytes, shift)
    f.fusco_plan_dispatch(L, A, **planes)
    check(L, planes)


# one to four entries, rows of whole lines and others, a few of the calls large enough to be written through; more than 1024 workgroups, rows cut into columns
@pytest.mark.parametrize("N,k,row_bytes", [(4095, 1, 2048), (4096, 1, 2048), (4097, 1, 2064), (8000, 1, 1040), (2100, 1, 20480 + 48), (5120, 2, 1024), (5119, 2, 1024),
                                           (5200, 2, 1040), (3500, 3, 1152), (1100, 2, 17408), (1100, 3, 16384 + 128), (3000, 4, 1024)])
def test_token_walk(N, k, row_bytes):
    f, L, A, planes = setup(N, k, 64, 8, row_bytes, 0, 0)
    f.fusco_plan(L, A)
    assert not f.fusco_dispatch_in_transfer_order(L, row_bytes)
    f.fusco_dispatch(L, planes["x"], planes["expert_buf"])
    check(L, planes)


# only rows of whole 64-byte units, for two and three entries of whole lines
@pytest.mark.parametrize("N,k,row_bytes,shift,through", [(12288, 2, 4096, 16, False), (12288, 2, 4096, 64, True), (9000, 3, 4224, 48, False), (9000, 3, 4224, 0, True),
                                                         (24577, 1, 2048, 16, False),
                                                         (12800, 1, 2048, 0, True), (12799, 1, 2048, 0, False), (8534, 2, 2048, 0, True), (8533, 2, 2048, 0, False),
                                                         (3200, 3, 4096, 0, True), (3199, 3, 4096, 0, False), (1200, 2, 17408, 0, True), (1200, 3, 16384 + 128, 0, True),
                                                         (2100, 1, 20480 + 48, 0, False), (26000, 1, 1088, 0, True)])
def test_token_walk_from_any_place(N, k, row_bytes, shift, through):
    f, L, A, planes = setup(N, k, 64, 8, row_bytes, 0, shift)
    f.fusco_plan(L, A)
    route = f.fusco_probe_dispatch_route(L, row_bytes, expert_buf=planes["expert_buf"])
    assert route == f.ROUTE_TOKENS | (f.WALK_THROUGH if through else f.WALK_PLAIN)
    f.fusco_dispatch(L, planes["x"], planes["expert_buf"])
    check(L, planes)


@pytest.mark.parametrize("N,k,row_bytes,shift,through", [(47, 8, 16384, 0, False), (48, 8, 16384, 0, True), (47, 16, 10752, 0, False), (49, 8, 32768, 0, True),
                                                         (30, 8, 12288, 0, True), (63, 8, 10400, 0, False), (64, 8, 10400, 0, True), (64, 8, 8192, 16, True),
                                                         (40, 8, 8192, 48, False), (40, 8, 8192, 64, True), (64, 32, 12288, 0, True)])
def test_fused_on_both_sides_of_the_rule(N, k, row_bytes, shift, through):
    f, L, A, planes = setup(N, k, 64, 8, row_bytes, 0, shift)
    assert f.fusco_probe_plan_dispatch_through(L, row_bytes, expert_buf=planes["expert_buf"]) == through
    f.fusco_plan_dispatch(L, A, **planes)
    check(L, planes)
