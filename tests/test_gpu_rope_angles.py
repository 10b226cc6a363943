"""reform_rerotate_keys on chosen displacements: every quadrant, small and large angles, and rotary
dimensions on both sides of the kernel's frequency table, against the fp64 oracle.

Bound in fp32: sine and cosine are within 1e-7 of the true ones (polynomials of an argument reduced
in fp64) and the rotation adds three roundings, so an output is within 3e-7 of the pair's size."""
import numpy as np
import pytest
import torch

import oracle
from helpers import to_np
from paper_2506_01215_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("d,rot", [(8, 8), (128, 96), (2056, 2048), (2112, 2112), (4096, 4096)])
def test_displacements_match_oracle(d, rot):
    g = torch.Generator().manual_seed(d)
    rows = 61
    k = torch.randn((2, rows, d), generator=g)
    step = torch.arange(rows, dtype=torch.int64)
    kept = torch.stack([step + step // 3, step + (step ** 4) * 120]).to(torch.int32)   # up to 1.6e9 positions
    kd = k.to(DEV)
    binding.reform_rerotate_keys(kd, kept.to(DEV), rows, 10000.0, rot)
    torch.cuda.synchronize()
    got = to_np(kd).astype(np.float64)
    for h in range(2):
        x = to_np(k[h]).astype(np.float64)
        want = oracle.rerotate_keys(x, kept[h].numpy(), 10000.0, rot)
        size = np.ones_like(x)
        half = rot // 2
        pair = np.hypot(x[:, :half], x[:, half:rot])
        size[:, :half] = size[:, half:rot] = pair
        # the angle itself: fp64 roundings of a few 1e-16 of up to 1.6e9 radians
        bound = (3e-7 + 2e-15 * np.abs(kept[h].numpy() - np.arange(rows))[:, None]) * size
        assert (np.abs(got[h] - want) <= bound).all(), np.max(np.abs(got[h] - want) / bound)
