"""Expert tensors from source tensors on both sides of the size up to which they are taken in one piece, in whole 64-byte units and not,
with and without a second plane.  Bytes: no tolerance."""
import numpy as np
import pytest
import torch

from definitions import random_topk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,k,row_bytes,aux_bytes", [(16385, 5, 8192, 0), (28672, 5, 8192, 0), (28673, 5, 8192, 0), (28617, 8, 8192, 16), (14336, 8, 16384, 0),
                                                     (14337, 8, 16384, 0), (18001, 6, 8192 + 64, 64)])
def test_expert_tensor(N, k, row_bytes, aux_bytes):
    import paper_2512_22036_amd as f
    E, D = 64, 8
    A = random_topk(np.random.default_rng(N + row_bytes), N, k, E)
    A[N // 3, 2] = -1   # an entry without an expert
    L = f.Layout(N, k, E, D)
    f.fusco_plan(L, torch.from_numpy(A).cuda())
    got = L.to_host()
    n = int(got.exp_off[-1])
    x = torch.randint(0, 256, (N, row_bytes), dtype=torch.uint8, device="cuda")
    rows = torch.full((L.P, row_bytes), 0xEE, dtype=torch.uint8, device="cuda")
    aux, want = {}, [(x, rows)]
    if aux_bytes:
        aux = dict(x_aux=torch.randint(0, 256, (N, aux_bytes), dtype=torch.uint8, device="cuda"),
                   expert_aux=torch.full((L.P, aux_bytes), 0xEE, dtype=torch.uint8, device="cuda"))
        want.append((aux["x_aux"], aux["expert_aux"]))
    assert f.fusco_dispatch_in_transfer_order(L, row_bytes, aux_bytes)
    f.fusco_dispatch(L, x, rows, **aux)
    token = torch.from_numpy(got.slot_token[:n].astype(np.int64)).cuda()
    for source, moved in want:
        assert torch.equal(moved[:n], source[token]) and bool((moved[n:] == 0xEE).all())
