"""Score pass of eight waves at head_dim 128 with query tiles of 192 rows (uncut passes of 512 rows and more): last tiles whose
rows end in their first, second and third group of 64, diagonals that begin inside a tile; against the fp64 oracle."""
import math

import pytest
import torch

import helpers
from helpers import assert_scores_close, oracle_kv_heads_dense, to_np
from paper_2506_01215_amd import binding

DEV = "cuda:0"
SHAPES = [
    (64, 64, 3488, 512),              # the fewest rows of this form, the last tile has two full groups
    (64, 64, 3425, 575),              # 2 * 192 + 191
    (64, 64, 3424, 576),              # full tiles alone
    (64, 64, 3423, 577),              # a last tile of one row
    (64, 64, 3359, 641),              # one row in the second group
    (64, 64, 3296, 704),              # one group and a full second one; the diagonal of the first keys is in the third tile
    (16, 8, 14831, 705),              # one row in the third group, two heads to a group
]


@pytest.mark.parametrize("Hq,Hkv,M,Ct", SHAPES)
def test_shapes_take_the_form(Hq, Hkv, M, Ct, tmp_path_factory):
    plan = helpers.load_attend_plan(tmp_path_factory)
    assert plan.score_form(Hkv, Hq // Hkv, 128, M, Ct, 0, 256) == 8001        # eight waves, uncut


@pytest.mark.gpu
@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("Hq,Hkv,M,Ct", SHAPES)
def test_score_matches_oracle(Hq, Hkv, M, Ct, accumulate):
    d, n = 128, M + Ct
    g = torch.Generator().manual_seed(M + Ct)
    q = torch.randn((Hq, Ct, d), generator=g).to(torch.bfloat16)
    k = (1.5 * torch.randn((Hkv, n + 1, d), generator=g)).to(torch.bfloat16)
    v = torch.randn((Hkv, n + 1, d), generator=g).to(torch.bfloat16)
    k[:, M - 1] = k[:, 2]
    k[:, n:] = float("nan")
    scale = 1.0 / math.sqrt(d)
    before = 0.25 if accumulate else 7.0
    score = torch.full((Hkv, n + 1), before, device=DEV)
    binding.reform_chunk_attend_score(q.to(DEV), k.to(DEV), v.to(DEV), M, scale, accumulate=accumulate, score=score)
    torch.cuda.synchronize()
    heads = [0, Hkv - 1]
    _, _, s_ref = oracle_kv_heads_dense(to_np(q), to_np(k), to_np(v), M, scale, heads)
    # bound of the other attention tests: fp32 sums of fp32 probabilities
    assert_scores_close(to_np(score)[heads, :n], s_ref[:, :n] + (before if accumulate else 0.0), 1e-5, "score")
    assert (score[:, n:] == before).all()
    assert (score[:, M - 1] == score[:, 2]).all()
