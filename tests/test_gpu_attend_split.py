"""Attention of problems too small or too uneven for one workgroup per row block or key block.

Forward attention with the key range split over workgroups (few row blocks, or a last round of
workgroups that would be nearly empty), against the fp64 oracle: ranges cut inside the causal
diagonal, row blocks shared by many workgroups or by two, heads and chunk ends that leave a
workgroup partly idle; keys with NaN logits; and the same call with a workspace too small for the partial results.

The eviction score with the observing rows cut into slices, and its form for few rows: windows that
begin inside a query tile, key blocks on the diagonal, accumulation, identical keys."""
import math

import pytest
import torch

import oracle
from helpers import assert_close, assert_scores_close, oracle_kv_heads_dense, to_np
from paper_2506_01215_amd import binding

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# Hq, Hkv, d, cache, chunk, window and the form of the forward pass, which is checked on the CPU (test_attend_fwd_choice.py):
# 1 four waves (else eight), 8 attn_fwd_short, 2 shared out, 4 merged by the score's launch.
SHAPES = [
    (8, 2, 128, 1000, 1, 0, 6),       # one token: every workgroup holds a few tiles of one row block
    (8, 2, 64, 127, 1, 0, 0),         # two tiles a head: one workgroup, nothing to merge
    (8, 8, 128, 4096, 17, 0, 6),
    (14, 2, 64, 2000, 300, 128, 8),   # seven query heads per KV head
    (21, 3, 64, 15224, 46, 46, 3),
    (1, 1, 128, 0, 1500, 0, 3),       # no cache: ranges begin on tiles that rows do not see
    (1, 1, 64, 900, 257, 0, 8),       # last row block of one row
    (1, 1, 64, 13827, 1025, 0, 2),
    (4, 1, 128, 900, 65, 0, 3),
    (6, 3, 128, 2003, 513, 77, 10),   # two heads of a group in one workgroup
    (2, 1, 128, 583, 79, 77, 3),
    (2, 1, 128, 6001, 40, 40, 6),
    (3, 3, 128, 8845, 385, 0, 2),     # eight waves, two row blocks and more
    (12, 3, 128, 9117, 100, 100, 2),
    (9, 3, 128, 9117, 132, 128, 2),
    (3, 1, 64, 15189, 353, 0, 2),
    (2, 1, 64, 14917, 518, 128, 2),
    (2, 2, 128, 12747, 386, 0, 10),   # keys shared out by attn_fwd_short, and not
    (32, 8, 128, 3199, 99, 99, 10),
    (6, 2, 128, 12738, 131, 128, 10),
    (3, 1, 64, 366, 90, 0, 8),
    (2, 1, 64, 351, 132, 128, 8),
]


def inputs(Hq, Hkv, d, M, Ct, seed):
    g = torch.Generator().manual_seed(seed)
    n = M + Ct
    q = (torch.randn((Hq, Ct, d), generator=g) * 1.5).to(torch.bfloat16)
    k = (torch.randn((Hkv, n + 3, d), generator=g) * 1.5).to(torch.bfloat16)   # logits of +-10: rows rescale
    v = torch.randn((Hkv, n + 3, d), generator=g).to(torch.bfloat16)
    return q.to(DEV), k.to(DEV), v.to(DEV)


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_split_forward_matches_oracle(shape):
    Hq, Hkv, d, M, Ct, W, _ = shape
    q, k, v = inputs(Hq, Hkv, d, M, Ct, seed=M + Ct)
    scale = 1.0 / math.sqrt(d)
    desc = binding.attn_desc(q, k, q, M, scale, W)
    lse_bytes = (Hq * Ct * 4 + 255) // 256 * 256
    full = torch.full((binding.attend_workspace_bytes(desc) + 256,), 0xff, dtype=torch.uint8, device=DEV)
    small = torch.full((lse_bytes + 512,), 0xff, dtype=torch.uint8, device=DEV)
    o_ref, l_ref, s_ref = oracle.attend_score(to_np(q), to_np(k), to_np(v), M, scale, W=W)
    results = []
    for ws in (full, full, small):
        out, lse, score = binding.reform_chunk_attend_score(q, k, v, M, scale, obs_window=W, workspace=ws)
        torch.cuda.synchronize()
        # the bounds of the other attention tests: bf16 rounding of P and of the output
        assert_close(to_np(out), o_ref, 2e-2, "out", row_floor=True)
        assert_close(to_np(lse), l_ref, 1e-5, "lse")
        assert_scores_close(to_np(score)[:, :M + Ct], s_ref[:, :M + Ct], 2e-2, "score")
        results.append((out, lse))
    assert torch.equal(results[0][0], results[1][0]) and torch.equal(results[0][1], results[1][1])


# More than four rounds of row blocks: eight waves, whole.
MANY = [
    (136, 136, 64, 100, 2001),      # 1088 row blocks, a wave to a head, the last block of 209 rows
    (132, 44, 64, 0, 2001),         # 1056, three heads
    (132, 44, 128, 100, 2001),
]


@pytest.mark.parametrize("shape", MANY, ids=lambda s: "x".join(map(str, s)))
def test_many_row_blocks_match_oracle(shape):
    Hq, Hkv, d, M, Ct = shape
    G = Hq // Hkv
    q, k, v = inputs(Hq, Hkv, d, M, Ct, seed=7 + M + Ct)
    scale = 1.0 / math.sqrt(d)
    out, lse, _ = binding.reform_chunk_attend_score(q, k, v, M, scale, want_score=False)
    torch.cuda.synchronize()
    for g in (0, Hkv - 1):
        o_ref, l_ref, _ = oracle_kv_heads_dense(to_np(q), to_np(k), to_np(v), M, scale, [g])
        # the bounds of the other attention tests
        assert_close(to_np(out)[g * G:(g + 1) * G], o_ref, 2e-2, "out", row_floor=True)
        assert_close(to_np(lse)[g * G:(g + 1) * G], l_ref, 1e-5, "lse")


# With the form of the forward pass where all its pieces have room, as above; what it is where they do not is checked on the CPU.
PARTS = (0.9, 0.5, 0.2, 0.05)
PARTLY = [
    (8, 2, 128, 1000, 1, 0, 6),
    (14, 2, 64, 2000, 300, 128, 8),
    (6, 3, 128, 2003, 513, 77, 10),
    (2, 1, 128, 6001, 40, 40, 6),
    (16, 2, 128, 1000, 600, 301, 8),
    (2, 2, 64, 0, 1600, 0, 8),
    (1, 1, 128, 0, 1500, 0, 3),
    (5, 1, 128, 633, 26, 26, 3),
    (1, 1, 64, 310, 1561, 128, 7),
    (9, 3, 128, 9117, 132, 128, 2),
    (7, 1, 64, 3441, 31, 17, 10),
    (1, 1, 128, 485, 120, 120, 14),
]


@pytest.mark.parametrize("shape", PARTLY, ids=lambda s: "x".join(map(str, s)))
def test_a_workspace_between_none_and_all(shape):
    """Room for some of the shares and slices: a cut that fits, and nothing behind its end is touched."""
    Hq, Hkv, d, M, Ct, W, _ = shape
    q, k, v = inputs(Hq, Hkv, d, M, Ct, seed=5 + M + Ct)
    scale = 1.0 / math.sqrt(d)
    o_ref, l_ref, s_ref = oracle.attend_score(to_np(q), to_np(k), to_np(v), M, scale, W=W)
    lse_bytes = (Hq * Ct * 4 + 255) // 256 * 256
    need = binding.attend_workspace_bytes(binding.attn_desc(q, k, q, M, scale, W)) - lse_bytes
    for part in PARTS:
        nbytes = lse_bytes + int(part * need)
        ws = torch.full((nbytes + 4096,), 0xa5, dtype=torch.uint8, device=DEV)
        out, lse, score = binding.reform_chunk_attend_score(q, k, v, M, scale, obs_window=W, workspace=ws[:nbytes])
        torch.cuda.synchronize()
        # the bounds of the other attention tests
        assert_close(to_np(out), o_ref, 2e-2, "out", row_floor=True)
        assert_close(to_np(lse), l_ref, 1e-5, "lse")
        assert_scores_close(to_np(score)[:, :M + Ct], s_ref[:, :M + Ct], 1e-5, "score")
        assert (ws[nbytes:] == 0xa5).all()


# Which form a shape takes is checked on the CPU (test_attend_plan.py).
SLICED = [
    (16, 4, 128, 100, 700, 0),      # slices of one tile, the last of 60 rows
    (2, 2, 64, 0, 1600, 0),         # every key block on the diagonal
    (16, 2, 128, 1000, 600, 301),   # window ends inside a tile
    (4, 4, 128, 515, 2048, 2048),
]
FEW_ROWS = [
    (8, 8, 128, 300, 17, 0),        # two row blocks, the second of one row
    (3, 1, 64, 5, 20, 9),           # fewer keys than a workgroup holds
    (16, 2, 64, 700, 1, 0),         # eight row blocks of one row
]


@pytest.mark.parametrize("shape", SLICED + FEW_ROWS + [
    (2, 2, 64, 0, 1500, 0),         # four waves share their keys: every one on the diagonal
    (8, 2, 128, 1000, 600, 301),    # window begins inside a row block
], ids=lambda s: "x".join(map(str, s)))
def test_score_slices_match_oracle(shape):
    Hq, Hkv, d, M, Ct, W = shape
    q, k, v = inputs(Hq, Hkv, d, M, Ct, seed=3 + M + Ct)
    if M > 10:
        k[:, 9] = k[:, 2]
        k[:, M - 1] = k[:, 2]
    scale = 1.0 / math.sqrt(d)
    n = M + Ct
    _, _, s_ref = oracle.attend_score(to_np(q), to_np(k), to_np(v), M, scale, W=W)
    need = binding.attend_workspace_bytes(binding.attn_desc(q, k, q, M, scale, W))
    for nbytes in (need, (Hq * Ct * 4 + 255) // 256 * 256):
        ws = torch.full((nbytes + 256,), 0xff, dtype=torch.uint8, device=DEV)
        _, _, score = binding.reform_chunk_attend_score(q, k, v, M, scale, obs_window=W, workspace=ws)
        twice = score.clone()
        binding.reform_chunk_attend_score(q, k, v, M, scale, obs_window=W, workspace=ws, score=twice, accumulate=True)
        torch.cuda.synchronize()
        # rtol 1e-5: logits and sums are fp32 (the wider bf16 bound concerns P and the output)
        assert_scores_close(to_np(score)[:, :n], s_ref[:, :n], 1e-5, "score")
        assert torch.equal(twice[:, :n], 2 * score[:, :n])
        assert not score[:, n:].any()
        if M > 10:
            assert torch.equal(score[:, 2], score[:, 9]) and torch.equal(score[:, 2], score[:, M - 1])


def test_the_shapes_split():
    """Every shape but the two-tile one asks for more workspace than the lse rows."""
    for Hq, Hkv, d, M, Ct, W, _ in SHAPES:
        q, k, _ = inputs(Hq, Hkv, d, M, Ct, seed=1)
        need = binding.attend_workspace_bytes(binding.attn_desc(q, k, q, M, 0.1, W))
        whole = (Hq * Ct * 4 + 255) // 256 * 256
        assert (need > whole) == (M + Ct > 128), (Hq, Hkv, d, M, Ct, need, whole)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Ct", [1, 40])
@pytest.mark.parametrize("lo,hi", [(64, 96), (0, 128)])
def test_nan_logits_reach_every_output(d, Ct, lo, hi):
    """Keys whose logits are NaN, all that one wave or one share of the keys sees: rows are NaN in out and lse and the
    score of every key is NaN, as with a workspace that has no room to split."""
    Hq, Hkv, M = 8, 2, 1000
    q, k, v = inputs(Hq, Hkv, d, M, Ct, seed=d + Ct)
    k[:, lo:hi] = float("nan")
    need = binding.attend_workspace_bytes(binding.attn_desc(q, k, q, M, 0.1))
    whole = (Hq * Ct * 4 + 255) // 256 * 256
    assert need > whole
    for nbytes in (need, whole):
        ws = torch.full((nbytes + 256,), 0xff, dtype=torch.uint8, device=DEV)
        out, lse, score = binding.reform_chunk_attend_score(q, k, v, M, 0.1, workspace=ws)
        torch.cuda.synchronize()
        assert out.isnan().all() and lse.isnan().all() and score[:, :M + Ct].isnan().all()
        out, lse, _ = binding.reform_chunk_attend_score(q, k, v, M, 0.1, want_score=False, workspace=ws)
        torch.cuda.synchronize()
        assert out.isnan().all() and lse.isnan().all()
