"""Score pass, tiled, the narrow form: four waves of 32 keys each.  Key counts around a workgroup's 128 and a wave's 32, row
counts around a query tile's 64, windows, many slices, and the uncut form of a workspace without room for slices; against
the fp64 oracle, and identical cache keys get identical scores."""
import math

import pytest
import torch

import oracle
from helpers import assert_scores_close, to_np
from paper_2506_01215_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# Which form a shape takes is checked on the CPU (test_attend_plan.py).
NARROW = [
    (16, 1, 64, 31, 97, 97),          # 128 keys: one workgroup, a second tile of 33 rows
    (16, 1, 64, 32, 97, 97),          # 129
    (7, 1, 64, 159, 289, 289),        # 448 keys: half of the last workgroup's waves have some
    (4, 1, 64, 127, 400, 400),        # 527: a wave with 15 keys
    (2, 2, 64, 0, 2113, 2113),        # every workgroup on the diagonal, one key over, 34 tiles
    (8, 1, 64, 1000, 300, 201),       # a window that is no multiple of a tile
    (4, 4, 64, 9000, 2048, 2048),     # full tiles only
]
NARROW += [(Hq, Hkv, 128, M, Ct, W) for Hq, Hkv, _, M, Ct, W in NARROW]


@pytest.mark.parametrize("Hq,Hkv,d,M,Ct,W", NARROW)
@pytest.mark.parametrize("accumulate,room", [(False, True), (True, True), (False, False)])
def test_score_matches_oracle(Hq, Hkv, d, M, Ct, W, accumulate, room):
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
    need = binding.attend_workspace_bytes(binding.attn_desc(q, k, q, M, scale, W))
    ws = torch.empty(need if room else (Hq * Ct * 4 + 255) // 256 * 256, dtype=torch.uint8, device=DEV)
    score = torch.full((Hkv, n + 1), 0.25 if accumulate else 7.0, device=DEV)
    _, _, score = binding.reform_chunk_attend_score(q.to(DEV), k.to(DEV), v.to(DEV), M, scale, obs_window=W,
                                                    accumulate=accumulate, score=score, workspace=ws)
    torch.cuda.synchronize()
    # bound of the other attention tests: fp32 sums of fp32 probabilities
    assert_scores_close(to_np(score)[:, :n], s_ref[:, :n] + (0.25 if accumulate else 0.0), 1e-5, "score")
    assert (score[:, n:] == (0.25 if accumulate else 7.0)).all()
    if M > 40:
        assert (score[:, M - 1] == score[:, 2]).all()
