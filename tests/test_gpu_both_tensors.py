"""Expert and receive tensors of one call on both sides of the source size from which they are written by launches of their own, with
and without a second plane, in whole 64-byte units and not.  Bytes: no tolerance."""
import numpy as np
import pytest
import torch

from definitions import random_topk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,D,row_bytes,aux_bytes", [(9215, 8, 8192, 0), (9216, 8, 8192, 0), (9216, 8, 8192 + 16, 0), (9216, 2, 8192, 0), (9145, 4, 8192, 64),
                                                     (9145, 4, 8192, 80), (5000, 8, 16384, 0), (8192, 8, 16384, 0), (8193, 8, 16384, 0),
                                                     (9216, 3, 8192, 0), (9300, 3, 9216, 64), (14335, 8, 8192, 0), (14336, 8, 8192, 0),
                                                     (9216, 4, 8256, 0), (7500, 4, 10240 - 64, 64)])
def test_both_tensors(N, D, row_bytes, aux_bytes):
    import paper_2512_22036_amd as f
    k, E = 8, 64 if D != 3 else 48
    A = random_topk(np.random.default_rng(N + row_bytes), N, k, E)
    A[N // 3, 2] = -1   # an entry without an expert
    L = f.Layout(N, k, E, D)
    f.fusco_plan(L, torch.from_numpy(A).cuda())
    got = L.to_host()
    n, U = int(got.exp_off[-1]), int(got.send_off[-1])
    planes, want = {}, []
    for suffix, width in (("", row_bytes), ("_aux", aux_bytes)):
        if not width:
            continue
        x = torch.randint(0, 256, (N, width), dtype=torch.uint8, device="cuda")
        rows, wire = (torch.full((r, width), 0xEE, dtype=torch.uint8, device="cuda") for r in (L.P, L.send_cap))
        planes.update({"x" + suffix: x, ("expert_buf" if not suffix else "expert_aux"): rows, ("send_buf" if not suffix else "send_aux"): wire})
        want.append((x, rows, wire))
    assert f.fusco_dispatch_in_transfer_order(L, row_bytes, aux_bytes, f.DISPATCH_EXPERT | f.DISPATCH_WIRE)
    f.fusco_dispatch(L, planes.pop("x"), planes.pop("expert_buf"), flags=f.DISPATCH_EXPERT | f.DISPATCH_WIRE, **planes)
    token, sent = (torch.from_numpy(a.astype(np.int64)).cuda() for a in (got.slot_token[:n], got.send_src[:U]))
    for x, rows, wire in want:
        assert torch.equal(rows[:n], x[token]) and bool((rows[n:] == 0xEE).all())
        assert torch.equal(wire[:U], x[sent]) and bool((wire[U:] == 0xEE).all())


@pytest.mark.parametrize("streaming", [False, True])
def test_two_launches_of_one_call(streaming):
    """A call that writes the receive tensors by a launch of their own: armed events span both launches and are used up by the one call, and
    the streaming flag changes no byte."""
    import paper_2512_22036_amd as f
    N, k, E, D, row = 11521, 8, 64, 8, 8192 + 64   # rows of 8 KiB are not taken in two launches at this size
    flags = f.DISPATCH_EXPERT | f.DISPATCH_WIRE | (f.DISPATCH_STREAMING if streaming else 0)
    L = f.Layout(N, k, E, D)
    f.fusco_plan(L, torch.from_numpy(random_topk(np.random.default_rng(5), N, k, E)).cuda())
    got = L.to_host()
    U = int(got.send_off[-1])
    x = torch.randint(0, 256, (N, row), dtype=torch.uint8, device="cuda")
    rows, wire = (torch.full((r, row), 0xEE, dtype=torch.uint8, device="cuda") for r in (L.P, L.send_cap))
    route = f.fusco_probe_dispatch_route(L, row, expert_buf=rows, send_buf=wire, flags=flags)
    assert route == f.ROUTE_TILES_THEN_TOKENS | f.WALK_STREAMING
    ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
    for e in ev:
        e.record()
    torch.cuda.synchronize()
    f.fusco_probe_time_next_call(*ev)
    f.fusco_dispatch(L, x, rows, send_buf=wire, flags=flags)
    torch.cuda.synchronize()
    ms = ev[0].elapsed_time(ev[1])
    # the call writes P + U rows, which take this long at the nominal 8 TB/s; the pairs alone take less than that
    assert (L.P + U) * row / 8e12 * 1e3 < ms < 5.0
    token, sent = (torch.from_numpy(a.astype(np.int64)).cuda() for a in (got.slot_token, got.send_src[:U]))
    assert torch.equal(rows, x[token]) and torch.equal(wire[:U], x[sent]) and bool((wire[U:] == 0xEE).all())
    f.fusco_dispatch(L, x, rows, send_buf=wire, flags=flags)   # not armed any more
    torch.cuda.synchronize()
    assert ev[0].elapsed_time(ev[1]) == ms
