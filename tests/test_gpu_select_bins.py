"""Selection of similarities, whose first pass bins them by 1/64 of an octave: thresholds below the bins, not positive, in the
first and the last ones, in bins that a list holds, just does not hold and that hold thousands, exact ties in them; one and
several workgroups to a row.  Exact on the similarities that came out."""
import numpy as np
import pytest
import torch

from paper_2506_01215_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def cosines(kind, n, g):
    u = torch.rand(n, generator=g)
    if kind == "spread":
        return 2 * u - 1
    if kind == "negative":
        return -u
    if kind == "tiny":                # below 2^-15, where the bins begin
        return 1e-6 * (u + 0.1)
    if kind == "around the first bin":
        return 2.0 ** -15 * (0.9 + 0.2 * u)
    if kind == "ones":                # the last octave's first bin, ties
        return torch.where(u < 0.5, torch.ones(n), u)
    if kind == "one bin":             # all within 1/64 octave: 11 more bits
        return 0.25 * (1.0 + u / 80)
    if kind == "one key":             # ... and within 2^-17 of it: 6 more
        return 0.25 * (1.0 + u * 2.0 ** -18)
    if kind == "lists":               # bins of 450 to 560
        return 2.0 ** -(6.0 * u) if n < 60000 else 2.0 ** -(14.0 * u)
    return torch.where(u < 0.3, torch.full((n,), 0.375), 0.5 * u)       # ties: thousands equal to one value


@pytest.mark.parametrize("kind", ["spread", "negative", "tiny", "around the first bin", "ones", "one bin", "one key", "lists", "ties"])
@pytest.mark.parametrize("n", [700, 5000, 9000, 40000, 140000])
def test_selection_is_exact(kind, n):
    g = torch.Generator().manual_seed(n)
    c = cosines(kind, n, g)
    emb = torch.zeros((n, 32))
    emb[:, 0], emb[:, 1] = c, torch.sqrt(1 - c.double() ** 2).float()
    qry = torch.zeros((2, 32))
    qry[0, 0] = qry[1, 1] = 1.0
    for k in (1, n // 50, n // 3, n - 1):
        idx, val, union, count = binding.reform_gather_topk(emb.to(DEV), qry.to(DEV), k, 0, 0, 0)
        sim = binding.reform_gather_similarity(emb.to(DEV), qry.to(DEV))
        torch.cuda.synchronize()
        for q in range(2):
            x = sim[q].cpu().numpy()
            want = np.sort(np.lexsort((np.arange(n), -x.astype(np.float64)))[:k])
            np.testing.assert_array_equal(idx[q].cpu().numpy(), want, err_msg=f"{kind} k={k} query {q}")
            np.testing.assert_array_equal(val[q].cpu().numpy(), x[want])


@pytest.mark.parametrize("n", [701, 5000, 9001, 40000, 140001])
def test_half_of_the_rows_and_one_more(n):
    """Up to half of the rows goes by bins, more by digits alone; cosines of both signs."""
    g = torch.Generator().manual_seed(n)
    emb, qry = torch.randn((n, 32), generator=g).to(DEV), torch.randn((2, 32), generator=g).to(DEV)
    sim = binding.reform_gather_similarity(emb, qry)
    for k in (n // 2, n // 2 + 1):
        idx, val, _, _ = binding.reform_gather_topk(emb, qry, k, 0, 0, 0)
        torch.cuda.synchronize()
        for q in range(2):
            x = sim[q].cpu().numpy()
            want = np.sort(np.lexsort((np.arange(n), -x.astype(np.float64)))[:k])
            np.testing.assert_array_equal(idx[q].cpu().numpy(), want)
            np.testing.assert_array_equal(val[q].cpu().numpy(), x[want])
