"""Forward pass of few rows by workgroups of 32, whose waves divide the keys (attn_fwd_short): last row blocks of one row and of
all, tiles that end with the keys and do not, rows that see none of a wave's keys, odd numbers of heads to a group, four and eight
waves; against the fp64 oracle.  And shapes beyond it for the forms that small problems used to take."""
import math

import pytest
import torch

import helpers
import oracle
import test_gpu_attend_fwd_narrow
import test_gpu_attend_merge_score
import test_gpu_attend_split
from helpers import assert_close, assert_scores_close, oracle_kv_heads_dense, to_np
from paper_2506_01215_amd import binding

DEV = "cuda:0"
# Hq, Hkv, d, cache, chunk and the waves of a workgroup, checked on the CPU below
SHORT = [
    (8, 8, 128, 0, 33, 8),            # no cache: keys of the last tile that the first rows do not see
    (10, 2, 64, 31, 40, 8),           # 200 rows, 71 keys
    (14, 2, 128, 95, 45, 8),          # the first row block's keys end with a tile
    (3, 1, 64, 640, 700, 8),          # 2100 rows, the last block of 20, tiles that some of a block's rows do not see
    (4, 2, 128, 1, 95, 8),            # 96 keys: whole tiles
    (17, 1, 64, 500, 33, 8),          # 561 rows: a block of 17
    (32, 1, 128, 0, 64, 8),           # a block is one chunk row of every head
    (1, 1, 64, 900, 257, 8),          # a last block of one row
    (32, 8, 64, 0, 601, 4),
    (32, 8, 128, 63, 257, 4),
    (32, 32, 128, 44, 301, 4),        # one head to a group: blocks of 32 chunk rows, the last of 13
]
LONGER = [
    (14, 2, 64, 3600, 201, 128, 3),
    (1, 1, 64, 1720, 268, 0, 2),
    (3, 1, 64, 1918, 86, 0, 2),
    (2, 1, 64, 1857, 129, 128, 2),
    (24, 8, 64, 0, 1366, 0, 1),
    (32, 8, 128, 0, 1025, 0, 1),
    (1, 1, 128, 508, 135, 0, 3),
    (4, 1, 64, 3703, 66, 0, 3),
    (2, 2, 64, 875, 131, 128, 6),
    (14, 2, 64, 927, 16, 16, 6),
    (3, 1, 64, 848, 31, 5, 6),
]


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    return helpers.load_attend_plan(tmp_path_factory)


@pytest.mark.parametrize("Hq,Hkv,d,M,Ct,waves", SHORT)
def test_the_short_shapes_take_the_form(plan, Hq, Hkv, d, M, Ct, waves):
    assert plan.short_waves(Hkv, Hq // Hkv, d, M, Ct, 0, 1, 256) == waves


@pytest.mark.parametrize("Hq,Hkv,d,M,Ct,W,form", LONGER)
def test_the_longer_shapes_take_the_other_forms(plan, Hq, Hkv, d, M, Ct, W, form):
    assert plan.short_waves(Hkv, Hq // Hkv, d, M, Ct, W, 1, 256) == 0
    assert plan.form(Hkv, Hq // Hkv, d, M, Ct, W, 1, 256) == form


@pytest.mark.parametrize("Hq,Hkv,d,M,Ct,taken", [
    # attention alone, us, plan / short (best number of waves)
    (32, 8, 64, 1000, 60, True),      # 15.4, 9.2
    (4, 4, 64, 74, 767, True),        # 14.5, 7.6
    (32, 8, 128, 1000, 130, True),    # 19.9, 13.6
    (32, 8, 64, 2976, 102, True),     # 17.9, 14.6
    (32, 32, 128, 44, 302, True),     # 12.5, 10.1
    (8, 8, 128, 952, 739, True),      # 21.8, 18.4
    (8, 8, 128, 3000, 100, False),    # 16.3, 33
    (8, 8, 64, 3592, 109, False),     # 12.5, 17.5
    (32, 8, 128, 3063, 958, False),   # 69, 110
    (24, 8, 128, 2182, 85, False),    # 21.5, 22
    (16, 4, 128, 3720, 67, False),    # 18.6, 30
    (8, 8, 128, 4096, 17, False),
    (32, 8, 128, 16640, 1, False),    # a token
])
def test_the_faster_form_is_taken(plan, Hq, Hkv, d, M, Ct, taken):
    assert (plan.short_waves(Hkv, Hq // Hkv, d, M, Ct, 0, 0, 256) != 0) == taken


@pytest.mark.gpu
@pytest.mark.parametrize("Hq,Hkv,d,M,Ct,waves", SHORT)
def test_matches_oracle(Hq, Hkv, d, M, Ct, waves):
    g = torch.Generator().manual_seed(M + Ct)
    n = M + Ct
    q = (torch.randn((Hq, Ct, d), generator=g) * 1.5).to(torch.bfloat16)
    k = (torch.randn((Hkv, n + 3, d), generator=g) * 1.5).to(torch.bfloat16)   # logits of +-10: rows rescale
    v = torch.randn((Hkv, n + 3, d), generator=g).to(torch.bfloat16)
    k[:, n:] = float("nan")           # behind the last key
    v[:, n:] = float("nan")
    scale = 1.0 / math.sqrt(d)
    heads = range(Hkv) if Hkv <= 3 else [0, Hkv - 1]
    G = Hq // Hkv
    mine = [h * G + i for h in heads for i in range(G)]
    o_ref, l_ref, s_ref = oracle_kv_heads_dense(to_np(q), to_np(k), to_np(v), M, scale, heads)
    for score in (True, False):
        out, lse, s = binding.reform_chunk_attend_score(q.to(DEV), k.to(DEV), v.to(DEV), M, scale, want_score=score)
        torch.cuda.synchronize()
        # the bounds of the other attention tests: bf16 rounding of P and of the output
        assert_close(to_np(out)[mine], o_ref, 2e-2, "out", row_floor=True)
        assert_close(to_np(lse)[mine], l_ref, 1e-5, "lse")
        if score:
            assert_scores_close(to_np(s)[list(heads), :n], s_ref[:, :n], 2e-2, "score")


@pytest.mark.gpu
def test_strides_and_logits_that_are_nan():
    """Rows of a tensor of tokens by heads (q and out), and NaN keys: rows that see one are NaN, the others are not touched."""
    Hq, Hkv, d, M, Ct = 6, 2, 128, 40, 50
    g = torch.Generator().manual_seed(5)
    n = M + Ct
    q = torch.randn((Ct, Hq, d), generator=g).to(torch.bfloat16).to(DEV).transpose(0, 1)
    k = torch.randn((Hkv, n, d), generator=g).to(torch.bfloat16).to(DEV)
    v = torch.randn((Hkv, n, d), generator=g).to(torch.bfloat16).to(DEV)
    store = torch.full((Ct, Hq + 1, d), 3.0, dtype=torch.bfloat16, device=DEV)
    out = store[:, :Hq].transpose(0, 1)
    k[1, M + 20] = float("nan")
    binding.reform_chunk_attend_score(q, k, v, M, 0.1, out=out, want_score=False)
    torch.cuda.synchronize()
    dense = binding.reform_chunk_attend_score(q.contiguous(), k, v, M, 0.1, want_score=False)[0]
    torch.cuda.synchronize()
    assert (store[:, Hq:] == 3.0).all()
    assert torch.equal(torch.nan_to_num(out.float(), nan=77.0), torch.nan_to_num(dense.float(), nan=77.0))
    nan = torch.isnan(out.float()).all(dim=-1)
    assert nan[3:, 20:].all() and not torch.isnan(out[:3].float()).any() and not torch.isnan(out[3:, :20].float()).any()


@pytest.mark.gpu
@pytest.mark.parametrize("shape", LONGER, ids=lambda s: "x".join(map(str, s)))
def test_the_other_forms_match_oracle(shape):
    test_gpu_attend_split.test_split_forward_matches_oracle(shape)
