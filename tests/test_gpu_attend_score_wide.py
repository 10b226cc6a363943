"""Score pass, tiled, with 64 keys to a wave: eight waves uncut (passes that fill the chip evenly) and four waves in slices (long
passes).  Key counts that end inside a workgroup and a wave, last query tiles that are not full, with and without a window;
against the fp64 oracle."""
import math

import pytest
import torch

from helpers import assert_scores_close, oracle_kv_heads_dense, to_np
from paper_2506_01215_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# Which form a shape takes is checked on the CPU (test_attend_plan.py).
EIGHT = [
    (32, 8, 64, 15924, 100, 0),       # 16024 keys: the last workgroup has 152; a second tile of 36 rows
    (32, 8, 64, 15525, 140, 100),     # the window begins in the first tile of rows; 15665 keys
    (8, 8, 128, 12639, 36, 0),        # 12675: a wave with three
    (8, 8, 128, 12747, 136, 100),
]
FOUR = [
    (32, 32, 128, 12001, 3001, 2833), # 15002 keys, 45 tiles, the last of 17 rows
    (32, 16, 128, 12007, 3009, 0),    # two heads, 15016 keys, 48 tiles, the last of one row
]


def inputs(Hq, Hkv, d, M, Ct, W):
    g = torch.Generator().manual_seed(Hq + M + Ct + W)
    n = M + Ct
    q = torch.randn((Hq, Ct, d), generator=g).to(torch.bfloat16)
    k = (1.5 * torch.randn((Hkv, n + 1, d), generator=g)).to(torch.bfloat16)
    v = torch.randn((Hkv, n + 1, d), generator=g).to(torch.bfloat16)
    k[:, M - 1] = k[:, 2]
    k[:, n:] = float("nan")
    return q, k, v


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("Hq,Hkv,d,M,Ct,W", EIGHT + FOUR)
def test_score_matches_oracle(Hq, Hkv, d, M, Ct, W, accumulate):
    n, W = M + Ct, W or Ct
    q, k, v = inputs(Hq, Hkv, d, M, Ct, W)
    scale = 1.0 / math.sqrt(d)
    before = 0.25 if accumulate else 7.0
    score = torch.full((Hkv, n + 1), before, device=DEV)
    binding.reform_chunk_attend_score(q.to(DEV), k.to(DEV), v.to(DEV), M, scale, obs_window=W, accumulate=accumulate, score=score)
    torch.cuda.synchronize()
    # a window of W rows scores as a chunk of those rows alone does, behind M + Ct - W keys; some KV heads are checked
    heads = [0, Hkv - 1] if Hkv * Ct < 5000 else [Hkv - 1]
    _, _, s_ref = oracle_kv_heads_dense(to_np(q[:, Ct - W:]), to_np(k), to_np(v), n - W, scale, heads)
    # bound of the other attention tests: fp32 sums of fp32 probabilities
    assert_scores_close(to_np(score)[heads, :n], s_ref[:, :n] + (before if accumulate else 0.0), 1e-5, "score")
    assert (score[:, n:] == before).all()
    assert (score[:, M - 1] == score[:, 2]).all()
