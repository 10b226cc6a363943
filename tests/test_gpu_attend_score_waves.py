"""Score pass whose four waves share 32 keys and divide the row blocks: block counts that do and do not divide by four
waves and two blocks in flight, key counts around a workgroup's 32, windows that begin inside a block, keys that only
the last rows see, accumulated scores; against the fp64 oracle, and identical cache keys get identical scores."""
import math

import pytest
import torch

import oracle
from helpers import assert_scores_close, to_np
from paper_2506_01215_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# Which form a shape takes is checked on the CPU (test_attend_plan.py).
FOUR_WAVES = [
    (9, 1, 128, 15, 16, 16),          # nine blocks, 31 keys
    (4, 1, 64, 0, 33, 33),            # twelve, 33 keys, diagonal
    (2, 2, 128, 1000, 150, 150),      # ten, from one head each
    (14, 2, 64, 500, 40, 25),         # the window begins inside a block
    (8, 1, 64, 64, 192, 192),         # 96, the most
    (8, 1, 128, 5300, 192, 192),      # the same at head_dim 128, 172 workgroups
    (4, 1, 128, 0, 256, 256),         # 64
    (3, 1, 64, 2047, 65, 65),
    (11, 1, 128, 96, 1, 1),           # one row, a block per head
]
TILED = [(8, 2, 64, 21000, 200, W) for W in (63, 64, 65, 129, 193)] + [(8, 1, 128, 64, 192, 192)]


@pytest.mark.parametrize("Hq,Hkv,d,M,Ct,W", FOUR_WAVES)
@pytest.mark.parametrize("accumulate", [False, True])
def test_score_matches_oracle(Hq, Hkv, d, M, Ct, W, accumulate):
    g = torch.Generator().manual_seed(Hq + M + Ct + W)
    n = M + Ct
    q = torch.randn((Hq, Ct, d), generator=g).to(torch.bfloat16)
    k = (1.5 * torch.randn((Hkv, n + 1, d), generator=g)).to(torch.bfloat16)
    v = torch.randn((Hkv, n + 1, d), generator=g).to(torch.bfloat16)
    if M > 40:
        k[:, M - 1] = k[:, 2]
    k[:, n:] = float("nan")
    scale = 1.0 / math.sqrt(d)
    _, _, s_ref = oracle.attend_score(to_np(q), to_np(k), to_np(v), M, scale, W)
    score = torch.full((Hkv, n + 1), 0.25 if accumulate else 7.0, device=DEV)
    _, _, score = binding.reform_chunk_attend_score(q.to(DEV), k.to(DEV), v.to(DEV), M, scale, obs_window=W,
                                                    accumulate=accumulate, score=score)
    torch.cuda.synchronize()
    # bound of the other attention tests: fp32 sums of fp32 probabilities
    assert_scores_close(to_np(score)[:, :n], s_ref[:, :n] + (0.25 if accumulate else 0.0), 1e-5, "score")
    assert (score[:, n:] == (0.25 if accumulate else 7.0)).all()
    if M > 40:
        assert (score[:, M - 1] == score[:, 2]).all()


@pytest.mark.parametrize("Hq,Hkv,d,M,Ct,W", TILED)
def test_tiles_begin_with_the_window(Hq, Hkv, d, M, Ct, W):
    """Too many keys for the form above, or too few for that many blocks: query tiles of 64, counted from the first observing row."""
    g = torch.Generator().manual_seed(W)
    q = torch.randn((Hq, Ct, d), generator=g).to(torch.bfloat16)
    k = (1.5 * torch.randn((Hkv, M + Ct, d), generator=g)).to(torch.bfloat16)
    v = torch.randn((Hkv, M + Ct, d), generator=g).to(torch.bfloat16)
    _, _, s_ref = oracle.attend_score(to_np(q), to_np(k), to_np(v), M, 0.125, W)
    _, _, score = binding.reform_chunk_attend_score(q.to(DEV), k.to(DEV), v.to(DEV), M, 0.125, obs_window=W)
    torch.cuda.synchronize()
    assert_scores_close(to_np(score), s_ref, 1e-5, "score")
