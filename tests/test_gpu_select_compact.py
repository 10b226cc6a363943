"""Gather over rows too many for the waiting selection: blocks of candidates that keep a few, up to a quarter, more, all
or none after the first digit, ties that fill whole blocks, rows that end inside a block, selections on both
sides of a sixteenth of the row, one block at a time and four; exact on the call's own similarities, union included."""
import numpy as np
import pytest
import torch

from helpers import numpy_union
from paper_2506_01215_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
D = 32


def store(kind, N, g):
    if kind == "spread":
        return torch.randn((N, D), generator=g)
    if kind == "ties":
        return torch.randn((5, D), generator=g)[torch.randint(0, 5, (N,), generator=g)]
    if kind == "equal":
        return torch.randn((1, D), generator=g).repeat(N, 1)
    if kind == "near":                # every similarity to the first query within one first digit, 0.5 to 0.625
        e = torch.randn((N, D), generator=g)
        e[:, 0] = 0
        e = 0.83 * e / e.norm(dim=1, keepdim=True)
        e[:, 0] = 0.56
        return e
    if kind == "clumps":              # runs of 3000 rows alike, so that a block keeps anything from none to all
        c = torch.rand((N // 3000 + 1, 1), generator=g).repeat(1, 3000).view(-1)[:N]
        e = torch.randn((N, D), generator=g)
        e = e / e.norm(dim=1, keepdim=True)
        e[:, 0] += 2 * c
        return e
    # sorted by angle: some blocks keep everything, most nothing
    a = torch.linspace(0.0, 3.0, N)
    e = torch.zeros((N, D))
    e[:, 0], e[:, 1] = torch.cos(a), torch.sin(a)
    return e


@pytest.mark.parametrize("kind", ["spread", "ties", "equal", "sorted", "near", "clumps"])
@pytest.mark.parametrize("N,nq,k,radius", [
    (32769, 33, 1, 0),               # one candidate in the last block
    (40000, 33, 2500, 3),            # exactly a sixteenth
    (40000, 33, 2501, 0),            # above it: the passes over whole rows
    (36863, 40, 500, 70),            # the last block lacks one
    (98309, 23, 3000, 8),
    (53250, 150, 1800, 1),           # 14 blocks a row, more than 2048 in all: four blocks to a workgroup, the last with two
])
def test_exact_on_own_similarities(kind, N, nq, k, radius):
    g = torch.Generator().manual_seed(N + k)
    emb = store(kind, N, g).bfloat16().to(DEV)
    qry = torch.randn((nq, D), generator=g).bfloat16().to(DEV)
    qry[0] = 0
    qry[0, 0] = 1
    sim = binding.reform_gather_similarity(emb, qry).cpu().numpy()
    ws = torch.full((binding.gather_workspace_bytes(binding.gather_desc(emb, qry, k, radius, 2, 3)) + 256,), 0xff,
                    dtype=torch.uint8, device=DEV)
    idx, val, union, count = binding.reform_gather_topk(emb, qry, k, radius, 2, 3, workspace=ws)
    torch.cuda.synchronize()
    idx, val = idx.cpu().numpy(), val.cpu().numpy()
    for q in range(nq):
        want = np.sort(np.lexsort((np.arange(N), -sim[q]))[:k])
        np.testing.assert_array_equal(idx[q], want)
        np.testing.assert_array_equal(val[q], sim[q][want])
    want = numpy_union(idx, N, radius, 2, 3)
    assert int(count.item()) == len(want)
    np.testing.assert_array_equal(union.cpu().numpy()[:len(want)], want)
