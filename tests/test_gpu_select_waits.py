"""The selection by several workgroups per row that wait for each other, where the waits expire.  The poll
limit is set from the host: 0 ends every wait at once, small limits end them at whatever step the workgroups
have reached.  Each workgroup then selects by itself, so the results stay bit-exact; the word that tells
of it is set in the gathers, and clear again with the default limit, also for calls that overlap."""
import numpy as np
import pytest
import torch

import oracle
from helpers import numpy_union
from paper_2506_01215_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
LIMITS = [0, 1, 4, 30, -1]


@pytest.fixture(autouse=True)
def restore_limit():
    yield
    binding.debug_set_move_spin_limit(-1)


def filled(nbytes):
    return torch.full((nbytes + 256,), 0x5a, dtype=torch.uint8, device=DEV)


def scores(kind, rows, n, g):
    if kind == "spread":                       # ends in a short list after two digits
        return torch.exp(2 * torch.randn((rows, n), generator=g))
    return torch.randint(0, 5, (rows, n), generator=g).float()       # ties: a third digit, and counts


@pytest.mark.parametrize("kind", ["spread", "ties"])
@pytest.mark.parametrize("Hkv,n,B,sink,recent", [(2, 8193, 4000, 0, 0), (3, 10000, 9999, 5, 6), (8, 40001, 13000, 0, 300),
                                                 (1, 600001, 250000, 1, 0)])
def test_staged_eviction_is_exact_whatever_expires(Hkv, n, B, sink, recent, kind):
    """head_dim 12 in fp32: 48-byte rows take the staged move, which has no wait of its own."""
    g = torch.Generator().manual_seed(n)
    s = scores(kind, Hkv, n, g)
    k = torch.randn((Hkv, n, 12), generator=g)
    want = [oracle.evict_select(s[h].numpy().astype(np.float64), n, B, sink, recent) for h in range(Hkv)]
    for limit in LIMITS:
        print(f"[waits] eviction {Hkv} x {n} {kind} limit {limit}", flush=True)
        binding.debug_set_move_spin_limit(limit)
        kd, vd, sd = k.to(DEV), -k.to(DEV), s.to(DEV)
        kept = torch.full((Hkv, B), -1, dtype=torch.int32, device=DEV)
        ws = filled(binding.evict_workspace_bytes(binding.evict_desc(kd, n, B, sink, recent)))
        binding.reform_evict_topk_compact(kd, vd, sd, n, B, sink, recent, kept_idx=kept, workspace=ws)
        torch.cuda.synchronize()
        assert binding.evict_status_word(ws) == 0
        for h in range(Hkv):
            np.testing.assert_array_equal(kept[h].cpu().numpy(), want[h])
            src = torch.from_numpy(want[h]).long()
            assert torch.equal(kd[h, :B].cpu(), k[h][src]) and torch.equal(vd[h, :B].cpu(), -k[h][src])
            assert torch.equal(sd[h, :B].cpu(), s[h][src])


def test_status_word_of_the_staged_eviction_of_short_rows():
    g = torch.Generator().manual_seed(3)
    k = torch.randn((2, 500, 12), generator=g).to(DEV)
    ws = filled(binding.evict_workspace_bytes(binding.evict_desc(k, 500, 200)))
    binding.reform_evict_topk_compact(k, k.clone(), torch.rand((2, 500), device=DEV), 500, 200, workspace=ws)
    assert binding.evict_status_word(ws) == 0


def test_in_place_eviction_keeps_the_right_slots():
    """There the move gives up too and says so; the kept slots are right all the same."""
    g = torch.Generator().manual_seed(8)
    Hkv, n, B = 2, 20000, 9000
    s = scores("spread", Hkv, n, g)
    k = torch.randn((Hkv, n, 64), generator=g).bfloat16().to(DEV)
    kept = torch.full((Hkv, B), -1, dtype=torch.int32, device=DEV)
    ws = filled(binding.evict_workspace_bytes(binding.evict_desc(k, n, B)))
    binding.debug_set_move_spin_limit(0)
    binding.reform_evict_topk_compact(k, k.clone(), s.to(DEV), n, B, kept_idx=kept, workspace=ws)
    torch.cuda.synchronize()
    assert binding.evict_status_word(ws) == 1
    for h in range(Hkv):
        np.testing.assert_array_equal(kept[h].cpu().numpy(), oracle.evict_select(s[h].numpy().astype(np.float64), n, B))


def store(N, nq, kind, seed):
    g = torch.Generator().manual_seed(seed)
    if kind == "ties":
        emb = torch.randint(-2, 3, (N, 32), generator=g)
        emb[:, 0] = 3
    else:
        emb = torch.randn((N, 32), generator=g)
    return emb.to(torch.bfloat16).to(DEV), torch.randint(-2, 3, (nq, 32), generator=g).to(torch.bfloat16).to(DEV)


def top(x, k):
    return np.sort(np.lexsort((np.arange(x.shape[0]), -x.astype(np.float64)))[:k])


@pytest.mark.parametrize("kind", ["spread", "ties"])
@pytest.mark.parametrize("N,nq,radius,tail", [(8193, 1, 0, 9), (40001, 3, 8, 9), (131000, 2, 1, 9),
                                              (131000, 1, 0, 0)])       # the union written by the selection
def test_gather_is_exact_whatever_expires(N, nq, radius, tail, kind):
    emb, qry = store(N, nq, kind, N)
    k = N // 20
    sim = binding.reform_gather_similarity(emb, qry).cpu().numpy()
    want = np.stack([top(sim[q], k) for q in range(nq)])
    union_ref = numpy_union(want, N, radius, 0, tail)
    for limit in LIMITS:
        print(f"[waits] gather {N} {kind} limit {limit}", flush=True)
        binding.debug_set_move_spin_limit(limit)
        ws = filled(binding.gather_workspace_bytes(binding.gather_desc(emb, qry, k, radius, 0, tail)))
        idx, val, union, count = binding.reform_gather_topk(emb, qry, k, radius, 0, tail, workspace=ws)
        torch.cuda.synchronize()
        np.testing.assert_array_equal(idx.cpu().numpy(), want)
        np.testing.assert_array_equal(val.cpu().numpy(), np.take_along_axis(sim, want, 1))
        np.testing.assert_array_equal(union.cpu().numpy()[:int(count.item())], union_ref)
        if limit <= 0:
            assert binding.evict_status_word(ws) == (limit == 0)     # the word lies where the eviction's does


@pytest.mark.parametrize("window", [1, 129])
def test_pooled_gather_is_exact_whatever_expires(window):
    emb, qry = store(50000, 3, "spread", 4)
    for limit in LIMITS:
        binding.debug_set_move_spin_limit(limit)
        ws = filled(binding.pooled_workspace_bytes(binding.pooled_desc(emb, qry, 5000, window, 7, 8)))
        sel, pooled = binding.reform_gather_pooled(emb, qry, 5000, window, 7, 8, workspace=ws)
        torch.cuda.synchronize()
        x = pooled.cpu().numpy().copy()
        x[:7] = np.inf
        x[-8:] = np.inf
        np.testing.assert_array_equal(sel.cpu().numpy(), top(x, 5000))
        if limit <= 0:
            assert binding.evict_status_word(ws) == (limit == 0)


def test_calls_on_several_streams_do_not_give_up():
    """Gathers, pooled gathers and evictions at once, whose waiting workgroups fit the chip together."""
    N, k, n, B = 200000, 9000, 30000, 14000
    g = torch.Generator().manual_seed(5)
    emb, qry = store(N, 2, "spread", 6)
    s = scores("spread", 4, n, g)
    cache = torch.randn((4, n, 64), generator=g).bfloat16().to(DEV)
    sim = binding.reform_gather_similarity(emb, qry).cpu().numpy()
    want_g = np.stack([top(sim[q], k) for q in range(2)])
    want_p, _ = binding.reform_gather_pooled(emb, qry, k, 129)
    want_e = np.stack([oracle.evict_select(s[h].numpy().astype(np.float64), n, B) for h in range(4)])
    ws = [filled(x) for x in (binding.gather_workspace_bytes(binding.gather_desc(emb, qry, k)),
                              binding.gather_workspace_bytes(binding.gather_desc(emb, qry, k)),
                              binding.pooled_workspace_bytes(binding.pooled_desc(emb, qry, k)),
                              binding.evict_workspace_bytes(binding.evict_desc(cache, n, B)))]
    streams = [torch.cuda.Stream() for _ in range(4)]
    idx = [torch.zeros((2, k), dtype=torch.int32, device=DEV) for _ in range(2)]
    sel = torch.zeros(k, dtype=torch.int32, device=DEV)
    kept = torch.zeros((4, B), dtype=torch.int32, device=DEV)
    kd, vd, sd, s0 = cache.clone(), cache.clone(), s.to(DEV), s.to(DEV)
    torch.cuda.synchronize()
    for _ in range(20):
        for i in range(2):
            with torch.cuda.stream(streams[i]):
                binding.reform_gather_topk(emb, qry, k, topk_idx=idx[i], want_union=False, workspace=ws[i])
        with torch.cuda.stream(streams[2]):
            binding.reform_gather_pooled(emb, qry, k, 129, sel_idx=sel, workspace=ws[2])
        with torch.cuda.stream(streams[3]):
            sd.copy_(s0)
            binding.reform_evict_topk_compact(kd, vd, sd, n, B, kept_idx=kept, workspace=ws[3])
    torch.cuda.synchronize()
    assert [binding.evict_status_word(w) for w in ws] == [0, 0, 0, 0]
    for i in range(2):
        np.testing.assert_array_equal(idx[i].cpu().numpy(), want_g)
    assert torch.equal(sel, want_p)
    np.testing.assert_array_equal(kept.cpu().numpy(), want_e)
