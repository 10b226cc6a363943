"""fp32 attention whose key blocks are shared by several workgroups: shares without a visible key, rows that end
inside a block, windows, accumulated scores, with the score (merged by its launch) and without, and with a
workspace that has no room for the shares' sums; against the fp64 oracle."""
import math

import pytest
import torch

import oracle
from helpers import assert_close, assert_scores_close, to_np
from paper_2506_01215_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("Hq,Hkv,d,M,Ct,W", [
    (4, 4, 64, 256, 128, 0),          # workload 1
    (8, 2, 64, 1024, 16, 0),
    (8, 2, 64, 1024, 1, 0),
    (4, 4, 32, 0, 300, 0),            # early row blocks leave shares without a key
    (4, 2, 128, 500, 33, 20),
    (2, 1, 128, 1500, 7, 7),
    (1, 1, 32, 127, 2, 1),            # two steps, two shares
    (1, 1, 64, 111, 16, 16),          # one step: whole
])
def test_matches_oracle(Hq, Hkv, d, M, Ct, W):
    g = torch.Generator().manual_seed(Hq + M + Ct)
    n = M + Ct
    q = torch.randn((Hq, Ct, d), generator=g)
    k = 1.5 * torch.randn((Hkv, n + 1, d), generator=g)
    v = torch.randn((Hkv, n + 1, d), generator=g)
    k[:, n:] = float("nan")
    v[:, n:] = float("nan")
    scale = 1.0 / math.sqrt(d)
    o_ref, l_ref, s_ref = oracle.attend_score(to_np(q), to_np(k), to_np(v), M, scale, W)
    qd, kd, vd = q.to(DEV), k.to(DEV), v.to(DEV)
    need = binding.attend_workspace_bytes(binding.attn_desc(qd, kd, qd, M, scale, W))
    for nbytes in (need, (Hq * Ct * 4 + 255) // 256 * 256):
        for want_score in (True, False):
            ws = torch.full((nbytes + 256,), 0xff, dtype=torch.uint8, device=DEV)
            before = torch.full((Hkv, n + 1), 0.25, device=DEV)
            out, lse, score = binding.reform_chunk_attend_score(
                qd, kd, vd, M, scale, obs_window=W, accumulate=True, score=before.clone() if want_score else None,
                want_score=want_score, workspace=ws)
            torch.cuda.synchronize()
            # the bound of the fp32 attention tests
            assert_close(to_np(out), o_ref, 1e-5, "out", row_floor=True)
            assert_close(to_np(lse), l_ref, 1e-5, "lse")
            if want_score:
                assert_scores_close(to_np(score)[:, :n], s_ref[:, :n] + 0.25, 1e-5, "score")
                assert (score[:, n:] == 0.25).all()
