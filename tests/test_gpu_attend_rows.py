"""Query rows of a KV head counted over its heads and chunk rows together: group sizes that do and do
not divide a workgroup's waves, chunks that end inside a wave, a 16-row block or a row block, key tiles
cut between the rows of one token's heads, with the key range split and whole (a workspace without room
for partial results), and strided q and out, against the fp64 oracle."""
import math

import pytest
import torch

import oracle
from helpers import assert_close, assert_scores_close, to_np
from paper_2506_01215_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("Hq,Hkv,d,M,Ct", [
    (7, 1, 64, 100, 1),           # one token, one wave
    (14, 2, 128, 300, 37),        # 259 rows: a second row block of three
    (5, 1, 64, 63, 52),           # 260 rows
    (3, 1, 128, 0, 90),           # diagonal, rows of one token in two row blocks (256 = 85 * 3 + 1)
    (16, 1, 64, 500, 33),         # more heads than waves
    (8, 1, 128, 250, 32),         # as many heads as waves, one slab each
    (8, 2, 64, 1000, 31),         # just below the slabs by head
    (8, 2, 128, 1, 97),           # slabs by head, the last one of a row
    (24, 8, 64, 700, 130),
    (6, 3, 128, 130, 500),
])
def test_rows_match_oracle(Hq, Hkv, d, M, Ct):
    g = torch.Generator().manual_seed(Hq + M + Ct)
    n = M + Ct
    # [row][head][d] storage, as a QKV projection leaves it
    q = torch.randn((Ct, Hq, d), generator=g).to(torch.bfloat16).permute(1, 0, 2)
    k = (1.5 * torch.randn((Hkv, n + 1, d), generator=g)).to(torch.bfloat16)
    v = torch.randn((Hkv, n + 1, d), generator=g).to(torch.bfloat16)
    k[:, n:] = float("nan")
    v[:, n:] = float("nan")
    scale = 1.0 / math.sqrt(d)
    o_ref, l_ref, s_ref = oracle.attend_score(to_np(q), to_np(k), to_np(v), M, scale)
    qd, kd, vd = q.to(DEV), k.to(DEV), v.to(DEV)
    need = binding.attend_workspace_bytes(binding.attn_desc(qd, kd, qd, M, scale))
    for nbytes in (need, (Hq * Ct * 4 + 255) // 256 * 256):
        ws = torch.full((nbytes + 256,), 0xff, dtype=torch.uint8, device=DEV)
        out = torch.empty((Ct, Hq, d), dtype=torch.bfloat16, device=DEV).permute(1, 0, 2)
        out, lse, score = binding.reform_chunk_attend_score(qd, kd, vd, M, scale, out=out, workspace=ws)
        torch.cuda.synchronize()
        # bounds of the other attention tests: bf16 rounding of P and of the output; fp32 for lse and score
        assert_close(to_np(out), o_ref, 2e-2, "out", row_floor=True)
        assert_close(to_np(lse), l_ref, 1e-5, "lse")
        assert_scores_close(to_np(score)[:, :n], s_ref[:, :n], 1e-5, "score")


@pytest.mark.parametrize("sign", [-1.0, 1.0])
@pytest.mark.parametrize("Hq,Hkv,d,M,Ct", [(4, 1, 128, 5000, 1), (2, 2, 64, 700, 16), (3, 1, 64, 300, 6)])
def test_few_rows_far_from_zero(Hq, Hkv, d, M, Ct, sign):
    """All logits of a row near +-1400 (natural units): a sum that begins relative to zero overflows."""
    g = torch.Generator().manual_seed(M)
    q = torch.ones((Hq, Ct, d)).to(torch.bfloat16)
    k = (sign * 40.0 + 0.25 * torch.randn((Hkv, M + Ct, d), generator=g)).to(torch.bfloat16)
    v = torch.randn((Hkv, M + Ct, d), generator=g).to(torch.bfloat16)
    scale = 35.0 / d
    out, lse, _ = binding.reform_chunk_attend_score(q.to(DEV), k.to(DEV), v.to(DEV), M, scale, want_score=False)
    torch.cuda.synchronize()
    o_ref, l_ref, _ = oracle.attend_score(to_np(q), to_np(k), to_np(v), M, scale)
    # fp32 logits of size 1400 carry an error of 1e-4: exp() of them 1e-4, within the bf16 bound
    assert_close(to_np(out), o_ref, 2e-2, "out", row_floor=True)
    assert_close(to_np(lse), l_ref, 1e-5, "lse")
