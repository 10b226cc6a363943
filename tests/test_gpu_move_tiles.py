"""In-place move of K and V at the edges of its 32 KB tiles (128 rows of 256 bytes, 512 of 64): budgets one below, at
and above a tile, evicted slots that shift every row by one, by a tile less one and by more than a tile, rows that
stay; bit-exact."""
import pytest
import torch

from test_gpu_evict import run_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,dtype,rows", [(128, torch.bfloat16, 128), (16, torch.float32, 512), (64, torch.bfloat16, 256)])
@pytest.mark.parametrize("tiles", [1, 2, 5])
@pytest.mark.parametrize("extra", [-1, 0, 1])
def test_tile_edges(d, dtype, rows, tiles, extra):
    B = rows * tiles + extra
    for gone in (1, rows - 1, rows + 1, 3 * rows):
        n = B + gone
        for first in (0, rows // 2, B - 1):               # the evicted slots lie together, from here on
            score = torch.ones((2, n + 3))
            score[:, first:first + gone] = 0.5
            score[1] = score[1].flip(0)                   # the other head: the same from the end
            run_case(2, d, n, B, n + 3, dtype, score, seed=gone)
