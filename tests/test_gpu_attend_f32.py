"""The fp32 attention kernels at the edges of their 16-row and 16-key blocks, for the head_dims on
the matrix cores and one that is not, against the fp64 oracle; and infinities in rows of V that
earlier rows of the chunk do not see."""
import math

import pytest
import torch

import oracle
from helpers import assert_close, assert_scores_close, to_np
from paper_2506_01215_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def inputs(Hq, Hkv, d, M, Ct, seed):
    g = torch.Generator().manual_seed(seed)
    q, k, v = (torch.randn((h, r, d), generator=g) for h, r in ((Hq, Ct), (Hkv, M + Ct + 2), (Hkv, M + Ct + 2)))
    k[:, M + Ct:] = float("nan")                       # rows past n are never read into a result
    v[:, M + Ct:] = float("nan")
    return q, k, v


@pytest.mark.parametrize("Hq,Hkv,d,M,Ct,W", [
    (1, 1, 32, 0, 1, 0),
    (2, 2, 64, 15, 1, 0),         # exactly one key block
    (2, 1, 64, 16, 17, 0),        # second row block of one row, chunk begins on a block boundary
    (4, 2, 128, 121, 16, 5),      # window inside a row block, diagonal inside a key block
    (8, 2, 32, 130, 33, 33),      # more key blocks than waves, ragged
    (3, 3, 128, 0, 129, 100),     # no cache
    (4, 4, 64, 1024, 50, 0),      # many key blocks per wave
    (2, 1, 48, 40, 19, 0),        # a head_dim without a matrix-core form
])
def test_block_edges_match_oracle(Hq, Hkv, d, M, Ct, W):
    q, k, v = inputs(Hq, Hkv, d, M, Ct, 7 + M + Ct)
    scale = 1.0 / math.sqrt(d)
    out, lse, score = binding.reform_chunk_attend_score(q.to(DEV), k.to(DEV), v.to(DEV), M, scale, obs_window=W)
    torch.cuda.synchronize()
    o_ref, l_ref, s_ref = oracle.attend_score(to_np(q), to_np(k), to_np(v), M, scale, W=W)
    n = M + Ct
    assert_close(to_np(out), o_ref, 1e-5, "out")
    assert_close(to_np(lse), l_ref, 1e-5, "lse")
    assert_scores_close(to_np(score)[:, :n], s_ref[:, :n], 1e-5, "score")


@pytest.mark.parametrize("d", [32, 64, 128])
def test_infinite_values_stay_with_the_rows_that_see_them(d):
    Hq, M, Ct, at = 2, 20, 30, 9
    q, k, v = inputs(Hq, Hq, d, M, Ct, 3)
    scale = 1.0 / math.sqrt(d)
    want, _, _ = oracle.attend_score(to_np(q), to_np(k), to_np(v), M, scale)
    v[:, M + at, 3] = float("inf")
    out, _, _ = binding.reform_chunk_attend_score(q.to(DEV), k.to(DEV), v.to(DEV), M, scale)
    out = to_np(out)
    assert (out[:, at:, 3] == float("inf")).all()
    out[:, at:, 3] = want[:, at:, 3]
    assert_close(out, want, 1e-5, "rows and dims without the infinity")
