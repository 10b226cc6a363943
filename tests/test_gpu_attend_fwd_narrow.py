"""Forward pass by workgroups of four waves and 128 query rows: row counts around a row block's 128 and a wave's 32, heads that
do and do not divide the waves, key counts around a tile's 64, row blocks taken whole and shared out, with and without the
score's launch merging the shares, and the uncut form of a workspace without room for shares; against the fp64 oracle."""
import math

import pytest
import torch

import oracle
from helpers import assert_close, assert_scores_close, to_np
from paper_2506_01215_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# Which form a shape takes with a workspace that holds all pieces is checked on the CPU (test_attend_fwd_choice.py).  The last
# entry of a shape: 1 whole row blocks, 3 shared out, 7 merged by the score's launch.
NARROW = [
    (176, 44, 128, 0, 64, 0, 1),      # 256 rows: two full row blocks, four heads to a workgroup
    (308, 44, 128, 0, 23, 0, 1),      # seven heads: rows of a wave from several
    (3, 1, 64, 0, 20, 0, 1),          # 60 rows of one block, 20 keys
    (3, 1, 64, 0, 43, 0, 1),          # 129 rows: one in the last block
    (4, 1, 64, 14, 20, 0, 1),
    (1, 1, 128, 513, 129, 0, 3),      # one row over; 642 keys
    (12, 3, 64, 15362, 82, 0, 3),     # heads divide the waves, the chunk rows do not fill the third block
    (5, 1, 128, 633, 26, 0, 3),
    (1, 1, 128, 0, 129, 128, 7),      # 128 observing rows in two row blocks
    (8, 2, 128, 776, 41, 17, 7),
    (1, 1, 64, 342, 1540, 128, 7),
    (1, 1, 128, 0, 131, 1, 7),
]
# Row counts around the same edges that attn_fwd_short takes where all its pieces have room: 8, 10 with keys shared out, 14
# merged by the score's launch.  Without room some of them run by four waves.
BY_THE_SHORT_FORM = [
    (32, 8, 128, 0, 96, 0, 8),
    (14, 2, 128, 0, 164, 0, 8),
    (24, 8, 64, 0, 266, 0, 8),
    (8, 2, 64, 0, 400, 0, 8),
    (1, 1, 128, 500, 129, 0, 8),
    (4, 1, 64, 427, 54, 0, 8),
    (5, 1, 128, 1000, 200, 0, 10),
    (2, 2, 128, 1000, 300, 128, 14),
    (1, 1, 64, 3000, 300, 128, 14),
    (1, 1, 128, 5000, 260, 128, 14),
]


@pytest.mark.parametrize("Hq,Hkv,d,M,Ct,W,form", NARROW + BY_THE_SHORT_FORM)
@pytest.mark.parametrize("room", [True, False])
def test_one_call_matches_oracle(Hq, Hkv, d, M, Ct, W, form, room):
    g = torch.Generator().manual_seed(Hq + M + Ct + W)
    n = M + Ct
    q = torch.randn((Hq, Ct, d), generator=g).to(torch.bfloat16)
    k = (1.5 * torch.randn((Hkv, n + 1, d), generator=g)).to(torch.bfloat16)
    v = torch.randn((Hkv, n + 1, d), generator=g).to(torch.bfloat16)
    k[:, n:] = float("nan")
    v[:, n:] = float("nan")
    scale = 1.0 / math.sqrt(d)
    o_ref, l_ref, s_ref = oracle.attend_score(to_np(q), to_np(k), to_np(v), M, scale, W or Ct)
    need = binding.attend_workspace_bytes(binding.attn_desc(q, k, q, M, scale, W))
    ws = torch.empty(need if room else (Hq * Ct * 4 + 255) // 256 * 256, dtype=torch.uint8, device=DEV)
    qd, kd, vd = q.to(DEV), k.to(DEV), v.to(DEV)
    for want_score in (True, False):
        ws.fill_(255)
        out, lse, score = binding.reform_chunk_attend_score(qd, kd, vd, M, scale, obs_window=W, want_score=want_score,
                                                            workspace=ws)
        torch.cuda.synchronize()
        # bounds of the other attention tests: bf16 probabilities in P.V, fp32 sums elsewhere
        assert_close(to_np(out), o_ref, 2e-2, "out", row_floor=True)
        assert_close(to_np(lse), l_ref, 1e-5, "lse")
        if want_score:
            assert_scores_close(to_np(score)[:, :n], s_ref[:, :n], 1e-5, "score")
