"""fp32 similarities on the matrix cores: dims that leave waves or chunks empty or half full, rows that end inside a
group of 16, several passes of queries, and the maximum over the queries; both sides of the size from which this
form is taken; against the fp64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from helpers import assert_close, to_np
from paper_2506_01215_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("N,D,nq", [
    (2048, 256, 1), (2049, 256, 1), (33000, 16, 1), (273, 32, 15), (1025, 48, 4), (300, 80, 17), (511, 256, 16), (4113, 272, 1),
    (257, 512, 33), (130, 1040, 40), (400, 2000, 16), (300, 2208, 14), (300, 2400, 14),
    (8209, 64, 3), (9000, 1200, 2),          # a second and a third round of workgroups
])
def test_similarities_and_their_maximum(N, D, nq):
    g = torch.Generator().manual_seed(N + D + nq)
    emb = torch.randn((N, D), generator=g).to(DEV)
    qry = torch.randn((nq, D), generator=g).to(DEV)
    emb[N // 2] = 0
    sim = binding.reform_gather_similarity(emb, qry)
    _, pooled = binding.reform_gather_pooled(emb, qry, 10, 1)
    torch.cuda.synchronize()
    # fp32 sums of D products on both sides of the rounding: a few 1e-7 of the root mean square
    assert_close(to_np(sim), oracle.cosine(to_np(emb), to_np(qry)), 1e-5, "sim")
    np.testing.assert_array_equal(to_np(pooled), to_np(sim).max(axis=0))
