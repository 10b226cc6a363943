"""Similarity kernel: queries whose rows end on either side of a staging step (64 lanes x 16 bytes x loads in
flight), blocks of 16 queries that are nearly empty or full, stores that leave most waves without a row
group, against the fp64 oracle."""
import pytest
import torch

import oracle
from helpers import assert_close, to_np
from paper_2506_01215_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("N,D,nq", [
    (1, 32, 1), (17, 256, 1), (300, 512, 8), (129, 544, 9), (4097, 1024, 16), (70, 1056, 20),
    (65, 2016, 16), (260, 2048, 31), (33, 2080, 16), (40, 4096, 5), (4200, 512, 48), (97, 1024, 64),
])
def test_similarities_at_staging_edges(N, D, nq):
    g = torch.Generator().manual_seed(N + D + nq)
    emb = torch.randn((N, D), generator=g).bfloat16().to(DEV)
    qry = torch.randn((nq, D), generator=g).bfloat16().to(DEV)
    # fp32 sums of D products of the same 16-bit values: an error of up to D eps / 2 relative to sum |x y|,
    # 4e-7 in practice
    assert_close(to_np(binding.reform_gather_similarity(emb, qry)), oracle.cosine(to_np(emb), to_np(qry)), 1e-5, "sim")
