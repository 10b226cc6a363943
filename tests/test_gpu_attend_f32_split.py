"""fp32 attention whose key blocks are shared by several workgroups: shares without a visible key, rows that end
inside a block, windows, accumulated scores, with the score (merged by its launch) and without, and with a
workspace that has no room for the shares' sums; against the fp64 oracle.  And shares all of whose logits are NaN."""
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
    (1, 1, 32, 127, 2, 1),            # nine key blocks: whole
    (1, 1, 32, 191, 2, 1),            # thirteen, two shares
    (1, 1, 128, 176, 20, 20),
    (16, 1, 32, 303, 32, 20),         # 32 row blocks: from 21 key blocks on
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


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("M,Ct,lo,hi", [
    (0, 193, 128, 193),               # all that the last rows see of the second share
    (600, 1, 384, 512),               # the fourth share's keys; split without the score too
])
def test_nan_logits_of_a_whole_share_reach_the_row(M, Ct, lo, hi, d):
    """A row that sees a NaN key is NaN in out and lse, and so is the score of every key it sees, however the keys are
    shared; the rows before it are the rows of the same call without the NaN."""
    g = torch.Generator().manual_seed(d + M)
    n = M + Ct
    q, k, v = (torch.randn((1, r, d), generator=g).to(DEV) for r in (Ct, n, n))
    bad = k.clone()
    bad[:, lo:hi] = float("nan")
    need = binding.attend_workspace_bytes(binding.attn_desc(q, k, q, M, 0.1))
    whole = (Ct * 4 + 255) // 256 * 256
    first = max(lo - M, 0)            # the first row that sees one
    assert need > whole
    for nbytes in (need, whole):
        for want_score in (True, False):
            ws = torch.full((nbytes + 256,), 0xff, dtype=torch.uint8, device=DEV)
            ref = binding.reform_chunk_attend_score(q, k, v, M, 0.1, want_score=want_score, workspace=ws)
            out, lse, score = binding.reform_chunk_attend_score(q, bad, v, M, 0.1, want_score=want_score, workspace=ws)
            torch.cuda.synchronize()
            assert out[:, first:].isnan().all() and lse[:, first:].isnan().all()
            assert torch.equal(out[:, :first], ref[0][:, :first]) and torch.equal(lse[:, :first], ref[1][:, :first])
            if want_score:
                assert score.isnan().all()
