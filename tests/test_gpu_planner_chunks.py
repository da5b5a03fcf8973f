"""Plans of many tiles: chunks whose tiles a thread of the summing pass holds in registers or walks, ragged last chunks and tiles, one and
several groups of columns, both sides of the tile count from which what pass 2 reads and writes goes through the L2.  All
whole numbers: no tolerance."""
import pytest
import torch

from test_gpu_planner_edges import check, routing

pytestmark = pytest.mark.gpu


# 199, 200 and 201 tiles; 256, 257 (chunks of 16 and 32); 1024, 1025 (32 and 64 tiles a chunk, 4 and 8 rows a thread); waves with idle lanes (k = 6, 10)
@pytest.mark.parametrize("N,k,E,D", [(50944, 8, 256, 8), (51200, 8, 256, 8), (51201, 8, 119, 7), (65536, 8, 64, 8), (65537, 8, 64, 8), (262144, 8, 64, 4),
                                     (262145, 8, 64, 4), (70000, 6, 120, 8), (45000, 10, 60, 4), (6500, 64, 1024, 1024), (420000, 1, 127, 1)])
@pytest.mark.parametrize("bad", [False, True])
def test_many_tiles(N, k, E, D, bad):
    import paper_2512_22036_amd as f
    A = routing(N + k, N, k, E, not bad, bad)
    if bad:
        A[N // 3:N // 3 + 2048 // k + 1] = E - 1   # a tile of one expert
    L = f.Layout(N, k, E, D)
    assert L.tile_count >= 199
    L.mem.fill_(0x7B)
    L.scratch.fill_(0x7B)
    f.fusco_plan(L, torch.from_numpy(A).cuda())
    check(L, A, "plan")
