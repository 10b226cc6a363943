"""Max-pooling inside the selection's launch and in one of its own: windows that end inside and with a group of four tokens,
contexts that end inside one, a workgroup and the waiting form, against torch's pooling of the same similarities; the
selection against a sort of what came out."""
import numpy as np
import pytest
import torch
import torch.nn.functional as F

from paper_2506_01215_amd import binding
from test_gpu_gather_pooled import exact_on_own_scores

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def store(N, kind):
    g = torch.Generator(device="cpu").manual_seed(N)
    emb = torch.randn((N, 32), generator=g)
    if kind == "ends":                # the largest similarities are the first and the last tokens'
        emb[0] = emb[N - 1] = torch.ones(32)
    return emb.to(DEV), torch.ones((1, 32), device=DEV)


@pytest.mark.parametrize("N", [1, 3, 127, 4095, 4096, 4097, 8190, 8192, 8193, 12289, 40003])
@pytest.mark.parametrize("window", [1, 3, 5, 7, 9, 11, 13, 15, 17, 33, 129, 135, 1023, 1025])
def test_windows(N, window):
    emb, qry = store(N, "ends")
    budget = max(1, N // 7)
    _, best = binding.reform_gather_pooled(emb, qry, budget, 1)
    sel, pooled = binding.reform_gather_pooled(emb, qry, budget, window)
    torch.cuda.synchronize()
    want = F.max_pool1d(best.cpu()[None, None], window, stride=1, padding=window // 2)[0, 0]
    assert torch.equal(pooled.cpu(), want)
    np.testing.assert_array_equal(sel.cpu().numpy(), exact_on_own_scores(pooled.cpu().numpy(), budget, 0, 0))


@pytest.mark.parametrize("N", [9001, 600011, 1100003])
def test_an_output_at_an_odd_address_and_long_rows(N):
    """Up to 8192 tokens a workgroup pooled with the selection, more by a launch of their own."""
    emb, qry = store(N, "")
    budget = N // 20
    _, best = binding.reform_gather_pooled(emb, qry, budget, 1, 64, 64)
    out = torch.full((N + 9,), 7.0, device=DEV)
    sel, pooled = binding.reform_gather_pooled(emb, qry, budget, 129, 64, 64, pooled=out[3:3 + N])
    torch.cuda.synchronize()
    want = F.max_pool1d(best.cpu()[None, None], 129, stride=1, padding=64)[0, 0]
    assert torch.equal(pooled.cpu(), want) and (out[:3] == 7.0).all() and (out[3 + N:] == 7.0).all()
    np.testing.assert_array_equal(sel.cpu().numpy(), exact_on_own_scores(pooled.cpu().numpy(), budget, 64, 64))
