"""Rows of bf16 that become rows of fp32 (combine with fp32 output, partial rows of the two-hop combine): the lanes that read a
chunk are not the ones that store its floats, so rows end in every place of a wave, and the rows behind them stay as they were.
Against the oracle, bit for bit: the sums have a stated order."""
import numpy as np
import pytest
import torch

from definitions import random_topk

pytestmark = pytest.mark.gpu

GUARD = 3   # rows behind the tensors in use


def inputs(oracle, N, k, E, D, H):
    import paper_2512_22036_amd as f
    rng = np.random.default_rng(N * 131 + H + k)
    A = random_topk(rng, N, k, E)
    y = (rng.integers(0x3E00, 0x4100, size=(N * k, H), dtype=np.uint16) | (rng.integers(0, 2, size=(N * k, 1), dtype=np.uint16) << 15)).astype(np.uint16)
    w = rng.standard_normal((N, k)).astype(np.float32)
    L = f.Layout(N, k, E, D)
    f.fusco_plan(L, torch.from_numpy(A).cuda())
    tokens = None if N * k * H < 4e6 else np.unique(np.concatenate([[0, N - 1], rng.integers(0, N, 120)])).astype(np.int32)
    return f, oracle.plan(A, E, D), L, y, torch.from_numpy(y.view(np.int16)).cuda().view(torch.bfloat16), w, torch.from_numpy(w).cuda(), tokens


def guarded(rows, H, dtype, shift=0):
    """`rows` rows with GUARD rows of NaN behind them; shift: elements that the first row lies past a 256-byte boundary."""
    mem = torch.full(((rows + GUARD) * H + shift,), float("nan"), dtype=dtype, device="cuda")
    return mem[shift:].view(rows + GUARD, H)


CHUNKS = [1, 3, 4, 7, 8, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127, 128, 129, 449, 1024, 1025, 2049]


# one entry (in two places), two and more (exchanged), of few workgroups
@pytest.mark.parametrize("k", [1, 2, 3, 8, 9])
@pytest.mark.parametrize("chunks", CHUNKS)
def test_combine_to_fp32(oracle, k, chunks):
    N, H = 5, 8 * chunks
    f, pl, L, y, d_y, w, d_w, tokens = inputs(oracle, N, k, 16, 4, H)
    want = oracle.combine_f32(y, w, pl.pair_slot, tokens)[0]
    for shift in (0, 4):   # rows from a 64-byte boundary on, and not
        out = guarded(N, H, torch.float32, shift)
        f.fusco_combine(L, d_y, d_w, out[:N])
        assert np.array_equal(out[:N].cpu().numpy().view(np.uint32), want.view(np.uint32))
        assert bool(torch.isnan(out[N:]).all())


# inputs bound by memory: one entry at a time, the only two at once, two of several at once; outputs that stay in the cache and that do not
@pytest.mark.parametrize("N,k,H", [(66000, 1, 8 * 65), (33000, 2, 8 * 65), (33000, 2, 8 * 64), (70000, 2, 8 * 33), (22500, 3, 8 * 65), (8200, 8, 8 * 65),
                                   (9000, 8, 8 * 130), (40000, 3, 8 * 66), (40000, 3, 8 * 68)])
def test_large_combine_to_fp32(oracle, N, k, H):
    f, pl, L, y, d_y, w, d_w, tokens = inputs(oracle, N, k, 64, 8, H)
    out = guarded(N, H, torch.float32)
    f.fusco_combine(L, d_y, d_w, out[:N])
    want = oracle.combine_f32(y, w, pl.pair_slot, tokens)[0]
    assert np.array_equal(out[:N].cpu().numpy()[tokens].view(np.uint32), want.view(np.uint32))
    assert bool(torch.isnan(out[N:]).all())


def check_two_hop(oracle, N, k, E, D, H, shift):
    f, pl, L, y, d_y, w, d_w, _ = inputs(oracle, N, k, E, D, H)
    o32, o16, part = oracle.combine_two_hop_f32(pl, y, w, want_partial=True)
    for dtype in (torch.float32, torch.bfloat16):
        partial, out = guarded(L.send_cap, H, torch.float32, shift), guarded(N, H, dtype)
        f.fusco_combine_two_hop(L, d_y, d_w, partial[:L.send_cap], out[:N])
        assert torch.equal(partial[:pl.U].view(torch.int32), torch.from_numpy(part.view(np.int32)).cuda())
        assert bool(torch.isnan(partial[pl.U:]).all()) and bool(torch.isnan(out[N:].float()).all())
        got = out[:N].cpu()
        if dtype == torch.float32:
            assert np.array_equal(got.numpy().view(np.uint32), o32.view(np.uint32))
        else:
            assert np.array_equal(got.view(torch.int16).numpy().view(np.uint16), o16)


@pytest.mark.parametrize("k", [1, 2, 8])
@pytest.mark.parametrize("chunks", CHUNKS)
def test_two_hop(oracle, k, chunks):
    for shift in (0, 4):   # partial rows written through or not, by where they start
        check_two_hop(oracle, 5, k, 16, 4, 8 * chunks, shift)


# the sizes of the launch rules: entries in turn (11 MiB and more), one by one (wide rows from 20 MiB on), at once again (96 MiB); partial rows in
# whole 64-byte units and not, on both sides of 20 MiB, and past the cache (400 MiB)
@pytest.mark.parametrize("N,k,H", [(5000, 4, 8 * 65), (5000, 4, 8 * 66), (2300, 4, 8 * 145), (2300, 4, 8 * 146), (1000, 6, 8 * 217), (12500, 8, 8 * 65),
                                   (12500, 8, 8 * 66), (8192, 8, 3200)])
def test_large_two_hop(oracle, N, k, H):
    check_two_hop(oracle, N, k, 64, 8, H, 0)
