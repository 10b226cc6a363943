"""Split attention whose pieces are merged by the launch that also forms the score of few rows: observing rows
in one row block and across two, windows that end inside a 16-row block, row blocks with few pieces and with many,
waves behind the last key, accumulated scores, against the fp64 oracle and the two calls by themselves."""
import math

import pytest
import torch

import oracle
from helpers import assert_close, assert_scores_close, to_np
from paper_2506_01215_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# The last entry of a shape is the form of the forward pass, which is checked on the CPU (test_attend_fwd_choice.py): 6 shared
# out and merged by the score's launch, 7 the same with row blocks of 128, 14 the same by attn_fwd_short; 1 whole row blocks of
# 128, 8 of 32.
MERGED = [
    (1, 1, 128, 0, 129, 100, 7),      # rows 29..128: two row blocks
    (2, 2, 128, 1000, 300, 100, 14),
    (1, 1, 64, 0, 1153, 32, 6),       # no cache: row blocks of few pieces
    (4, 1, 128, 3000, 20, 20, 6),     # eight blocks of rows, half of each empty
    (14, 2, 64, 900, 16, 16, 14),
    (7, 1, 64, 1365, 5, 1, 6),
    (8, 1, 128, 700, 1, 1, 6),        # one token
    (1, 1, 128, 5000, 260, 1, 14),    # only the last row observes
    (1, 1, 128, 0, 129, 1, 7),
    (8, 8, 128, 4096, 17, 17, 6),
    (3, 1, 64, 196, 5, 5, 6),
    (14, 2, 128, 9000, 1, 1, 6),      # seven rows of many pieces, 32 lanes each
    (1, 1, 64, 3000, 40, 3, 6),       # three rows, 64 lanes each
    (1, 1, 64, 443, 809, 128, 6),     # the observing rows end a row block and are the last
    (4, 4, 128, 8351, 397, 128, 14),
    (3, 3, 128, 11034, 387, 128, 6),
    (8, 2, 128, 300, 40, 16, 7),
]
# chunks that are not split
WHOLE = [(1, 1, 64, 0, 17, 5, 1), (3, 1, 64, 0, 6, 6, 1), (2, 2, 64, 0, 200, 128, 8), (3, 1, 64, 130, 31, 5, 8), (3, 1, 64, 200, 31, 5, 8),
         (2, 2, 64, 0, 500, 128, 8), (3, 1, 64, 400, 31, 5, 8), (2, 2, 64, 0, 300, 128, 8)]


@pytest.mark.parametrize("Hq,Hkv,d,M,Ct,W,form", MERGED + WHOLE)
@pytest.mark.parametrize("accumulate", [False, True])
def test_one_call_matches_oracle(Hq, Hkv, d, M, Ct, W, form, accumulate):
    g = torch.Generator().manual_seed(Hq + M + Ct + W)
    n = M + Ct
    q = torch.randn((Hq, Ct, d), generator=g).to(torch.bfloat16)
    k = (1.5 * torch.randn((Hkv, n + 1, d), generator=g)).to(torch.bfloat16)
    v = torch.randn((Hkv, n + 1, d), generator=g).to(torch.bfloat16)
    k[:, n:] = float("nan")
    v[:, n:] = float("nan")
    scale = 1.0 / math.sqrt(d)
    o_ref, l_ref, s_ref = oracle.attend_score(to_np(q), to_np(k), to_np(v), M, scale, W)
    qd, kd, vd = q.to(DEV), k.to(DEV), v.to(DEV)
    need = binding.attend_workspace_bytes(binding.attn_desc(qd, kd, qd, M, scale, W))
    ws = torch.full((need + 256,), 0xff, dtype=torch.uint8, device=DEV)
    before = torch.full((Hkv, n + 1), 0.25 if accumulate else 7.0, device=DEV)
    score = before.clone()
    out, lse, score = binding.reform_chunk_attend_score(qd, kd, vd, M, scale, obs_window=W, accumulate=accumulate,
                                                        score=score, workspace=ws)
    two = before.clone()
    out2, lse2, _ = binding.reform_chunk_attend_score(qd, kd, vd, M, scale, obs_window=W, workspace=ws, phases=1)
    binding.reform_chunk_attend_score(qd, kd, vd, M, scale, obs_window=W, accumulate=accumulate, out=out2, lse=lse2,
                                      score=two, workspace=ws, phases=2)
    torch.cuda.synchronize()
    # bounds of the other attention tests: bf16 rounding of P and of the output; fp32 for lse and score
    assert_close(to_np(out), o_ref, 2e-2, "out", row_floor=True)
    assert_close(to_np(lse), l_ref, 1e-5, "lse")
    assert_scores_close(to_np(score)[:, :n], s_ref[:, :n] + (0.25 if accumulate else 0.0), 1e-5, "score")
    # the same pieces in another order: an lse of at most 20 within a few ulp (2e-6 each), exp of it likewise
    assert_close(to_np(lse), to_np(lse2), 1e-6, "lse, two calls")
    assert_scores_close(to_np(score)[:, :n], to_np(two)[:, :n], 1e-5, "score, two calls")
    assert (score[:, n:] == before[:, n:]).all()
