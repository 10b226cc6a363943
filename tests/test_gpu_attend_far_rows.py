"""Query rows far apart in memory: a whole query tile of the score pass spans more than 4 GiB, with tiles of 64 rows and of 192, by
eight waves and by four; the scores are those of the same rows side by side."""
import pytest
import torch

import helpers
from paper_2506_01215_amd import binding

DEV = "cuda:0"
SHAPES = [
    # Hq, Hkv, d, cache, chunk, row stride, form of the score pass
    (64, 64, 128, 3488, 512, 11_250_048, 8),   # 191 rows reach over 4 GiB, 190 do not
    (64, 64, 128, 3423, 577, 12_000_000, 8),
    (8, 8, 128, 8686, 141, 34_200_064, 2),     # 63 rows
    (8, 8, 64, 8686, 141, 70_000_000, 2),      # so far that half of them do
]


@pytest.mark.parametrize("Hq,Hkv,d,M,Ct,stride,form", SHAPES)
def test_shapes_take_the_form_and_reach_beyond_32_bits(Hq, Hkv, d, M, Ct, stride, form, tmp_path_factory):
    plan = helpers.load_attend_plan(tmp_path_factory)
    assert plan.score_form(Hkv, Hq // Hkv, d, M, Ct, 0, 256) // 1000 == form
    tile = 192 if form == 8 else 64
    assert Ct >= tile and 2 * (tile - 1) * stride >= 1 << 32


@pytest.mark.gpu
@pytest.mark.parametrize("Hq,Hkv,d,M,Ct,stride,form", SHAPES)
def test_scores_are_those_of_rows_side_by_side(Hq, Hkv, d, M, Ct, stride, form):
    g = torch.Generator(device=DEV).manual_seed(M + Ct)
    q = torch.randn((Hq, Ct, d), generator=g, device=DEV).bfloat16()
    k = (1.5 * torch.randn((Hkv, M + Ct, d), generator=g, device=DEV)).bfloat16()
    v = torch.randn((Hkv, M + Ct, d), generator=g, device=DEV).bfloat16()
    room = torch.empty((Ct - 1) * stride + Hq * d, dtype=torch.bfloat16, device=DEV)
    far = torch.as_strided(room, (Hq, Ct, d), (d, stride, 1))
    far.copy_(q)
    near = binding.reform_chunk_attend_score(q, k, v, M, d ** -0.5)
    got = binding.reform_chunk_attend_score(far, k, v, M, d ** -0.5)
    torch.cuda.synchronize()
    for a, b in zip(near, got):
        assert torch.equal(a, b)
