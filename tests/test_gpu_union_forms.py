"""The gather's union: written by the selection itself (one query, no neighbours, nothing forced) by one workgroup,
several, or the launches for a row too long for these, with and without scores; and emitted by workgroups that
count the words before their own, on both sides of the number of them up to which they do."""
import ctypes

import numpy as np
import pytest
import torch

from helpers import numpy_union
from paper_2506_01215_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def gather(N, nq, k, radius, head, tail):
    g = torch.Generator().manual_seed(N + k)
    emb = torch.randn((N, 32), generator=g).bfloat16().to(DEV)
    qry = torch.randn((nq, 32), generator=g).bfloat16().to(DEV)
    union = torch.full((N,), -7, dtype=torch.int32, device=DEV)
    ws = torch.full((binding.gather_workspace_bytes(binding.gather_desc(emb, qry, k, radius, head, tail)) + 256,), 0xff,
                    dtype=torch.uint8, device=DEV)
    idx, _, union, count = binding.reform_gather_topk(emb, qry, k, radius, head, tail, union_idx=union, workspace=ws)
    torch.cuda.synchronize()
    return idx.cpu().numpy(), union.cpu().numpy(), int(count.item())


@pytest.mark.parametrize("N,k", [(1, 1), (300, 299), (4097, 64), (8192, 8192), (8193, 1), (40000, 30001), (131075, 4096)])
def test_union_of_one_query_is_its_selection(N, k):
    idx, union, count = gather(N, 1, k, 0, 0, 0)
    assert count == k
    np.testing.assert_array_equal(union[:k], idx[0])
    assert (union[k:] == -7).all()


@pytest.mark.parametrize("N,k", [(300, 299), (40000, 30001), (64 * 32768 + 1, 300), (64 * 32768 + 1, 500000)])
def test_union_of_one_query_without_scores(N, k):
    """topk_score = NULL at the C entry (the binding always passes one); the last two rows are longer than
    64 workgroups hold."""
    g = torch.Generator().manual_seed(k)
    emb = torch.randn((N, 32), generator=g).bfloat16().to(DEV)
    qry = torch.randn((1, 32), generator=g).bfloat16().to(DEV)
    sim = binding.reform_gather_similarity(emb, qry)[0].cpu().numpy()
    want = np.sort(np.lexsort((np.arange(N), -sim))[:k])
    desc = binding.gather_desc(emb, qry, k, 0, 0, 0)
    nbytes = binding.gather_workspace_bytes(desc)
    ws = torch.full((nbytes + 256,), 0xff, dtype=torch.uint8, device=DEV)
    idx, union, count = (torch.full((n,), -7, dtype=torch.int32, device=DEV) for n in (k, N, 1))
    base = (ws.data_ptr() + 255) // 256 * 256
    rc = binding.load_library().reform_gather_topk(
        ctypes.byref(desc), emb.data_ptr(), qry.data_ptr(), idx.data_ptr(), None, union.data_ptr(), count.data_ptr(),
        base, nbytes, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert rc == 0 and int(count.item()) == k
    np.testing.assert_array_equal(idx.cpu().numpy(), want)
    np.testing.assert_array_equal(union[:k].cpu().numpy(), want)
    assert (union[k:] == -7).all()


@pytest.mark.parametrize("N", [8192, 8193, 16 * 8192, 16 * 8192 + 1, 17 * 8192 + 33])
@pytest.mark.parametrize("nq,radius,head,tail", [(1, 0, 0, 5), (1, 0, 70, 0), (2, 40, 33, 64), (3, 0, 0, 0)])
def test_union_counts(N, nq, radius, head, tail):
    idx, union, count = gather(N, nq, 200, radius, head, tail)
    want = numpy_union(idx, N, radius, head, tail)
    assert count == len(want)
    np.testing.assert_array_equal(union[:count], want)
