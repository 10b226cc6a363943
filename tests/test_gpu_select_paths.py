"""The selection at the sizes where its route changes and with rows that decide how it ends: few or many
candidates equal to the threshold (a list of at most 256, or another digit), all equal, only the
highest or only the lowest digits differing, negative rows, forced slots, rows whose pitch or start
does not allow 16-byte loads.  Bit-exact against the oracle, through the eviction (with the row move that
depends on the ranks) and through the gather (whose union is marked by the same kernels)."""
import numpy as np
import pytest
import torch

import oracle
from helpers import numpy_union
from paper_2506_01215_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def rows(kind, n, g):
    """Two score rows; positive and negative values, ties as the name says."""
    if kind == "spread":
        x = torch.exp(3 * torch.randn((2, n), generator=g))
    elif kind == "mixed":
        x = torch.randn((2, n), generator=g)
    elif kind == "negative":
        x = -torch.exp(torch.randn((2, n), generator=g))
    elif kind == "equal":
        x = torch.full((2, n), 0.25)
    elif kind == "zeros":                      # +0 and -0 compare equal
        x = torch.zeros((2, n)) * (1 - 2 * (torch.arange(n) % 2))
    elif kind == "low_digit":                  # all share their upper 22 bits
        x = (0x3F800000 + torch.randint(0, 1024, (2, n), generator=g)).to(torch.int32).view(torch.float32)
    elif kind == "two_values":
        x = torch.randint(0, 2, (2, n), generator=g).float()
    else:                                      # plateaus of ~250: the list just fits or just does not
        x = torch.randn((2, n // 250 + 1), generator=g).repeat_interleave(250, dim=1)[:, :n]
        x = x[:, torch.randperm(n, generator=g)]
    return x.contiguous()


@pytest.mark.parametrize("n,extra", [(300, 0), (4096, 1), (4097, 3), (8192, 0), (8193, 3), (32769, 0), (70001, 2)])
@pytest.mark.parametrize("kind", ["spread", "mixed", "negative", "equal", "zeros", "low_digit", "two_values", "plateaus"])
def test_eviction_is_exact(n, extra, kind):
    g = torch.Generator().manual_seed(n)
    x = torch.zeros((2, n + extra))
    x[:, :n] = rows(kind, n, g)
    k = torch.randint(-9, 9, (2, n + extra, 8), generator=g).to(torch.bfloat16).to(DEV)
    for B, sink, recent in ((n // 2, 0, 0), (n - 1, 3, 5), (7, 4, 3), (n // 3, n // 5, 1)):
        kd, vd, sd = k.clone(), k.neg(), x.to(DEV)
        kept = torch.full((2, B), -1, dtype=torch.int32, device=DEV)
        pos = torch.arange(n + extra, dtype=torch.int32, device=DEV).repeat(2, 1)
        binding.reform_evict_topk_compact(kd, vd, sd, n, B, sink, recent, pos=pos, kept_idx=kept)
        torch.cuda.synchronize()
        for h in range(2):
            want = oracle.evict_select(x[h, :n].numpy().astype(np.float64), n, B, sink, recent)
            np.testing.assert_array_equal(kept[h].cpu().numpy(), want, err_msg=f"{kind} n={n} B={B}")
            src = torch.from_numpy(want).long()
            assert torch.equal(kd[h, :B].cpu(), k[h].cpu()[src]) and torch.equal(vd[h, :B].cpu(), -k[h].cpu()[src])
            assert torch.equal(pos[h, :B].cpu(), src.int())
            np.testing.assert_array_equal(sd[h, :B].cpu().numpy(), x[h].numpy()[want])


@pytest.mark.parametrize("N,nq,radius,head,tail", [
    (2000, 1, 0, 0, 0), (8192, 3, 1, 5, 0), (8200, 16, 33, 0, 40), (40001, 2, 8, 256, 256), (70000, 16, 3, 1, 1),
    (130000, 1, 64, 0, 31), (300000, 16, 0, 32, 64),      # the last by the multi-launch route
])
def test_gather_is_exact_and_its_union_complete(N, nq, radius, head, tail):
    g = torch.Generator().manual_seed(N)
    emb = torch.randint(-2, 3, (N, 32), generator=g).to(torch.bfloat16).to(DEV)    # many equal rows: ties
    qry = torch.randint(-2, 3, (nq, 32), generator=g).to(torch.bfloat16).to(DEV)
    emb[:, 0] = 3                                          # no zero rows
    sim = binding.reform_gather_similarity(emb, qry).cpu().numpy()
    for k in (1, N // 50, N // 3):
        idx, val, union, count = binding.reform_gather_topk(emb, qry, k, radius, head, tail)
        torch.cuda.synchronize()
        idx = idx.cpu().numpy()
        for q in range(nq):
            want = np.sort(np.lexsort((np.arange(N), -sim[q].astype(np.float64)))[:k])
            np.testing.assert_array_equal(idx[q], want)
            np.testing.assert_array_equal(val[q].cpu().numpy(), sim[q][want])
        got = union.cpu().numpy()[:int(count.item())]
        np.testing.assert_array_equal(got, numpy_union(idx, N, radius, head, tail))


@pytest.mark.parametrize("N", [8193, 16385, 32768, 32769])
def test_many_long_rows_are_exact(N):
    """More rows than workgroups may wait for each other: one workgroup per row up to 32768 candidates, several
    launches above."""
    g = torch.Generator().manual_seed(N)
    rows_e, B = 129, N // 3
    x = torch.randint(0, 4000, (rows_e, N), generator=g).float()                    # ties
    k = torch.randint(-9, 9, (rows_e, N, 8), generator=g).to(torch.bfloat16)
    kd, vd, sd = k.to(DEV), k.neg().to(DEV), x.to(DEV)
    kept = torch.full((rows_e, B), -1, dtype=torch.int32, device=DEV)
    binding.reform_evict_topk_compact(kd, vd, sd, N, B, 3, 5, kept_idx=kept)
    torch.cuda.synchronize()
    for h in range(0, rows_e, 16):
        want = oracle.evict_select(x[h].numpy().astype(np.float64), N, B, 3, 5)
        np.testing.assert_array_equal(kept[h].cpu().numpy(), want)
        src = torch.from_numpy(want).long()
        assert torch.equal(kd[h, :B].cpu(), k[h][src]) and torch.equal(vd[h, :B].cpu(), -k[h][src])
    emb = torch.randint(-2, 3, (N, 32), generator=g).to(torch.bfloat16).to(DEV)
    qry = torch.randint(-2, 3, (65, 32), generator=g).to(torch.bfloat16).to(DEV)
    emb[:, 0] = 3
    sim = binding.reform_gather_similarity(emb, qry).cpu().numpy()
    idx, val, union, count = binding.reform_gather_topk(emb, qry, 60, 2, 1, 9)
    torch.cuda.synchronize()
    idx = idx.cpu().numpy()
    for q in range(65):
        want = np.sort(np.lexsort((np.arange(N), -sim[q].astype(np.float64)))[:60])
        np.testing.assert_array_equal(idx[q], want)
        np.testing.assert_array_equal(val[q].cpu().numpy(), sim[q][want])
    np.testing.assert_array_equal(union.cpu().numpy()[:int(count.item())], numpy_union(idx, N, 2, 1, 9))
