"""Similarity passes that take several blocks of 16 queries over the store at once: every number of
blocks, queries that fill the last block partly, several passes, dims that end inside a prefetch
chunk, against the fp64 oracle; and the maximum over the queries that the pooled gather forms in the
same pass, which has to be the maximum of exactly these similarities."""
import numpy as np
import pytest
import torch

import oracle
from helpers import assert_close, to_np
from paper_2506_01215_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("N,D,nq,dtype", [
    (1000, 256, 17, torch.bfloat16),
    (333, 96, 48, torch.bfloat16),        # three full blocks, dim not a multiple of a chunk
    (2049, 512, 64, torch.bfloat16),
    (515, 1024, 65, torch.bfloat16),      # two passes
    (700, 2048, 37, torch.bfloat16),      # two blocks at most fit: two passes
    (16, 2080, 33, torch.bfloat16),       # one group of rows
    (301, 64, 130, torch.bfloat16),       # three passes
    (200, 40, 19, torch.bfloat16),        # dim without a matrix-core form
    (450, 128, 40, torch.float32),
])
def test_similarities_and_their_maximum(N, D, nq, dtype):
    g = torch.Generator().manual_seed(N + nq)
    emb = torch.randn((N, D), generator=g).to(dtype).to(DEV)
    qry = torch.randn((nq, D), generator=g).to(dtype).to(DEV)
    sim = binding.reform_gather_similarity(emb, qry)
    sel, pooled = binding.reform_gather_pooled(emb, qry, 10, 1)
    torch.cuda.synchronize()
    # inputs are the same 16-bit values on both sides: what differs are fp32 sums of D products
    assert_close(to_np(sim), oracle.cosine(to_np(emb), to_np(qry)), 1e-5, "sim")
    np.testing.assert_array_equal(to_np(pooled), to_np(sim).max(axis=0))
