"""Merge of a shared-out forward pass with two rows to a thread (more than 16384 rows in all): row blocks whose last rows
leave a thread with one or none, several pieces to a row, KV heads that do and do not divide by the chip's XCDs; against the
fp64 oracle."""
import math

import pytest
import torch

import helpers
from helpers import assert_close, assert_scores_close, oracle_kv_heads_dense, to_np
from paper_2506_01215_amd import binding

DEV = "cuda:0"
SHAPES = [
    (33, 33, 128, 3210, 257),         # last row block of one row
    (24, 8, 64, 3041, 683),           # of one, three heads to a group
    (28, 4, 128, 857, 599),           # of 97, seven heads to a group
    (28, 4, 128, 949, 586),           # of six
    (24, 8, 64, 3225, 684),           # of four
    (40, 8, 64, 3051, 410),           # of two
    (12, 4, 64, 300, 3001),           # of 43
    (6, 3, 64, 2500, 3001),           # three KV heads
    (4, 2, 64, 129, 4099),            # two
]
# As many rows, which attn_fwd_short takes whole.
BY_THE_SHORT_FORM = [
    (8, 8, 128, 300, 2049),
    (12, 4, 64, 100, 1500),
    (14, 2, 128, 333, 1301),
    (10, 2, 64, 2000, 1700),
    (6, 3, 64, 500, 3001),
]


@pytest.mark.parametrize("Hq,Hkv,d,M,Ct", SHAPES)
def test_shapes_take_the_form(Hq, Hkv, d, M, Ct, tmp_path_factory):
    plan = helpers.load_attend_plan(tmp_path_factory)
    assert plan.form(Hkv, Hq // Hkv, d, M, Ct, 0, 1, 256) == 2           # eight waves, shared out, merged by itself
    assert Hkv * (-(-(Hq // Hkv * Ct) // 256)) * 256 > 16384


@pytest.mark.gpu
@pytest.mark.parametrize("Hq,Hkv,d,M,Ct", SHAPES + BY_THE_SHORT_FORM)
def test_matches_oracle(Hq, Hkv, d, M, Ct):
    n, G = M + Ct, Hq // Hkv
    g = torch.Generator().manual_seed(M + Ct)
    q = (torch.randn((Hq, Ct, d), generator=g) * 1.5).to(torch.bfloat16)
    k = (torch.randn((Hkv, n + 3, d), generator=g) * 1.5).to(torch.bfloat16)
    v = torch.randn((Hkv, n + 3, d), generator=g).to(torch.bfloat16)
    scale, head = 1.0 / math.sqrt(d), Hkv - 1
    out, lse, score = binding.reform_chunk_attend_score(q.to(DEV), k.to(DEV), v.to(DEV), M, scale)
    torch.cuda.synchronize()
    o_ref, l_ref, s_ref = oracle_kv_heads_dense(to_np(q), to_np(k), to_np(v), M, scale, [head])
    mine = slice(head * G, (head + 1) * G)
    # the bounds of the other attention tests: bf16 rounding of P and of the output
    assert_close(to_np(out)[mine], o_ref, 2e-2, "out", row_floor=True)
    assert_close(to_np(lse)[mine], l_ref, 1e-5, "lse")
    assert_scores_close(to_np(score)[[head], :n], s_ref[:, :n], 2e-2, "score")
