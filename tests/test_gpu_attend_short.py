"""Forward pass of few rows by workgroups of 32, whose waves divide the keys (attn_fwd_short): last row blocks of one row and of
all, tiles that end with the keys and do not, rows that see none of a wave's keys, odd numbers of heads to a group, four and eight
waves; keys shared out over several workgroups, merged by a launch of its own and by the score's; against the fp64 oracle.  And
shapes beyond it for the forms that small problems used to take."""
import ctypes
import math
import random

import pytest
import torch

import helpers
import test_gpu_attend_split
from helpers import assert_close, assert_scores_close, oracle_kv_heads_dense, to_np
from paper_2506_01215_amd import binding

DEV = "cuda:0"
# Hq, Hkv, d, cache, chunk and the waves of a workgroup, checked on the CPU below
SHORT = [
    (8, 8, 128, 0, 97, 8),            # no cache: keys of the last tile that the first rows do not see
    (10, 2, 64, 31, 40, 8),           # 200 rows, 71 keys
    (14, 2, 128, 95, 45, 8),          # the first row block's keys end with a tile
    (3, 1, 64, 340, 700, 8),          # 2100 rows, the last block of 20, tiles that some of a block's rows do not see
    (4, 2, 128, 1, 95, 8),            # 96 keys: whole tiles
    (17, 1, 64, 500, 33, 8),          # 561 rows: a block of 17
    (32, 1, 128, 0, 64, 8),           # a block is one chunk row of every head
    (1, 1, 64, 400, 257, 8),          # a last block of one row
    (32, 8, 64, 0, 601, 4),
    (32, 8, 128, 63, 257, 4),
    (32, 32, 128, 44, 301, 4),        # one head to a group: blocks of 32 chunk rows, the last of 13
]
# ... and, with their windows, 100 times the workgroups to a row block's keys, 10000 more where the score's launch merges them
SHARED = [
    (1, 1, 64, 1533, 185, 0, 308),    # a last block of 25 rows
    (8, 1, 64, 1647, 20, 0, 308),
    (3, 3, 128, 834, 129, 0, 308),    # a last block of one row, three KV heads
    (3, 1, 128, 771, 40, 0, 308),
    (1, 1, 64, 3365, 212, 0, 608),    # so many pieces that a workgroup merges one row
    (7, 1, 64, 3441, 31, 17, 608),
    (7, 1, 128, 1561, 18, 18, 608),
    (1, 1, 64, 607, 37, 17, 10208),
    (3, 1, 64, 610, 15, 1, 10208),
    (1, 1, 128, 485, 120, 120, 10208),   # observing rows in four row blocks
    (4, 1, 128, 505, 15, 10, 10208),
]
LONGER = [
    (1, 1, 64, 0, 33, 33, 1),
    (32, 32, 128, 0, 1030, 0, 1),
    (256, 32, 128, 0, 33, 0, 1),
    (12, 2, 128, 2508, 375, 0, 2),    # eight waves, several row blocks, by rows, with a wave to a head, and of one head
    (12, 3, 128, 2674, 372, 0, 2),
    (4, 4, 128, 2135, 1215, 0, 2),
    (3, 1, 64, 3720, 1445, 0, 2),
    (2, 1, 64, 3014, 2157, 0, 2),
    (2, 2, 64, 3108, 2231, 0, 2),
    (5, 1, 64, 1661, 18, 0, 2),       # and one
    (5, 1, 128, 939, 24, 17, 2),
    (1, 1, 64, 0, 2913, 0, 3),
    (5, 1, 64, 29936, 109, 0, 3),
    (1, 1, 128, 487, 157, 0, 3),
    (8, 1, 128, 623, 28, 0, 3),
    (1, 1, 64, 1399, 17, 5, 6),
    (8, 1, 128, 334, 5, 0, 6),
    (1, 1, 64, 0, 1549, 5, 7),
    (1, 1, 128, 0, 131, 1, 7),
    (2, 1, 128, 39, 66, 5, 7),
]


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    return helpers.load_attend_plan(tmp_path_factory)


@pytest.mark.parametrize("Hq,Hkv,d,M,Ct,waves", SHORT)
def test_the_short_shapes_take_the_form(plan, Hq, Hkv, d, M, Ct, waves):
    assert plan.short_form(Hkv, Hq // Hkv, d, M, Ct, 0, 1, 256) == 100 + waves


@pytest.mark.parametrize("Hq,Hkv,d,M,Ct,W,form", SHARED)
def test_the_shared_shapes_take_the_form(plan, Hq, Hkv, d, M, Ct, W, form):
    assert plan.short_form(Hkv, Hq // Hkv, d, M, Ct, W, 1, 256) == form


@pytest.mark.parametrize("Hq,Hkv,d,M,Ct,W,form", LONGER)
def test_the_longer_shapes_take_the_other_forms(plan, Hq, Hkv, d, M, Ct, W, form):
    assert plan.short_form(Hkv, Hq // Hkv, d, M, Ct, W, 1, 256) == 0
    assert plan.form(Hkv, Hq // Hkv, d, M, Ct, W, 1, 256) == form


def test_pieces_fit_the_room_there_is(plan):
    rng = random.Random(3)
    plan.short_bytes.restype = ctypes.c_long
    less = 0
    for _ in range(3000):
        Hkv, G, d = rng.choice([1, 2, 4, 8]), rng.choice([1, 2, 4, 7]), rng.choice([64, 128])
        M, Ct, scored = rng.randint(500, 20000), rng.randint(9, 200), rng.randint(0, 1)
        want = plan.short_bytes(Hkv, G, d, M, Ct, scored, 256, ctypes.c_long(-1))
        room = rng.randint(0, max(1, 2 * want))
        got = plan.short_bytes(Hkv, G, d, M, Ct, scored, 256, ctypes.c_long(room))
        assert got <= room and (want > room or got == want), (Hkv, G, d, M, Ct, scored, want, room, got)
        less += 0 < got < want
    assert less > 50


@pytest.mark.parametrize("G", [1, 2, 3, 4, 7, 8, 16, 71])
def test_every_tile_of_the_shares_has_one_workgroup_and_its_piece_a_slot(plan, G):
    rng = random.Random(G)
    shared = cut = 0
    for _ in range(1500):
        Hkv, d, cus = rng.choice([1, 2, 3, 4, 8, 32]), rng.choice([64, 128]), rng.choice([256, 256, 32, 304])
        M, Ct, scored = rng.randint(100, 30000), int(2 ** rng.uniform(0, 9)), rng.randint(0, 1)
        plan.short_bytes.restype = ctypes.c_long
        want = plan.short_bytes(Hkv, G, d, M, Ct, scored, cus, ctypes.c_long(-1))
        for room in (-1, want, rng.randint(0, want)):
            rc = plan.replay_short(Hkv, G, d, M, Ct, scored, cus, ctypes.c_long(room))
            assert rc in (0, 1), (Hkv, G, d, M, Ct, scored, cus, room, rc)
            shared += rc == 0
            cut += rc == 0 and 0 <= room < want
    assert shared > 30 and cut > 3


@pytest.mark.parametrize("Hq,Hkv,d,M,Ct,taken", [
    # attention alone, us, plan / short (best number of waves)
    (32, 8, 64, 1000, 60, True),      # 15.4, 9.2
    (4, 4, 64, 74, 767, True),        # 14.5, 7.6
    (32, 8, 128, 1000, 130, True),    # 19.9, 13.6
    (32, 8, 64, 2976, 102, True),     # 17.9, 14.6
    (32, 32, 128, 44, 302, True),     # 12.5, 10.1
    (8, 8, 128, 952, 739, True),      # 21.8, 18.4
    (32, 8, 128, 3063, 958, False),   # 69, 110
    # a little more than one, two or three workgroups to a compute unit
    (40, 8, 64, 5509, 206, False),    # 29.1, 38.5
    (6, 3, 64, 3451, 1569, False),    # 28.1, 34.4
    (71, 1, 128, 143, 350, False),    # 17.0, 21.1
    (16, 16, 64, 5973, 556, False),   # 34.8, 43.0
    (4, 4, 64, 2464, 2669, False),    # 29.3, 34.6
    (40, 8, 128, 1483, 418, False),   # 34.2, 39.7
    (64, 8, 128, 0, 293, False),      # 12.4, 14.7
    (24, 8, 128, 1408, 685, False),   # 33.7, 40.2
    (8, 1, 64, 0, 1134, True),        # 19.9, 10.2
    (10, 2, 64, 0, 1721, True),       # 24.8, 14.5
    (32, 8, 64, 551, 281, True),      # 15.2, 9.7
    (16, 4, 128, 0, 601, True),       # 17.7, 11.9
    (14, 2, 128, 67, 1144, True),     # 30.0, 18.7
    # more K and V than the L2s hold, for few row blocks
    (40, 40, 64, 7597, 76, False),    # 26.2, 35.2
    (40, 40, 64, 11681, 148, False),  # 45.3, 56.1
    (32, 32, 64, 3482, 77, False),    # 16.1, 17.3
    (32, 32, 64, 3182, 167, True),    # 21.1, 16.9
    (40, 40, 128, 1273, 157, True),   # 22.0, 17.5
    # heads that do not divide by the XCDs, each longer than an L2 holds
    (9, 3, 128, 24136, 109, False),   # 34.6, 53.0 with seven shares
    (10, 5, 128, 11981, 130, False),
    (10, 5, 64, 15229, 237, False),   # 46.0, 47.9 with the score
    (6, 3, 128, 29745, 152, True),    # 38.4, 37.5 with eight
    # more K and V than shares gain anything on
    (5, 1, 64, 320666, 52, False),    # 49.7, 51.7
    (2, 2, 64, 171038, 288, False),   # 52.4, 54.4
    (3, 1, 64, 82197, 83, True),      # 32.6, 27.8 with the score
    # a key tile or two of the plans and few rows
    (32, 8, 128, 0, 8, False),        # 5.6, 6.6
    (24, 8, 128, 0, 20, False),       # 6.0, 6.6
    (32, 8, 128, 90, 8, False),       # 6.5, 7.0
    (32, 8, 64, 40, 8, False),        # 4.9, 4.9
    (14, 2, 64, 0, 8, False),         # 4.4, 4.6
    (14, 2, 128, 0, 20, True),        # 7.0, 6.6
    (14, 2, 128, 90, 8, True),        # 6.5, 6.3
    (32, 8, 64, 90, 8, True),         # 5.6, 5.2
    # keys shared out
    (14, 2, 128, 2150, 137, True),    # 19.2, 14.7
    (16, 4, 64, 8964, 90, True),      # 19.7, 15.0
    (8, 8, 64, 6187, 161, True),      # 16.6, 13.2
    (24, 8, 128, 3858, 150, True),    # 26.7, 22.9
    (24, 8, 128, 26775, 23, False),   # 30.1, 35.3
    (32, 8, 128, 18728, 10, False),   # 20.9, 21.8
    (4, 4, 64, 10640, 35, False),     # 11.5, 12.2
    (8, 8, 128, 4096, 17, False),
    (32, 8, 128, 16640, 1, False),    # a token
])
def test_the_faster_form_is_taken(plan, Hq, Hkv, d, M, Ct, taken):
    assert (plan.short_form(Hkv, Hq // Hkv, d, M, Ct, 0, 0, 256) != 0) == taken


@pytest.mark.parametrize("Hq,Hkv,M,Ct,W,taken", [
    # whole calls at head_dim 128 whose score's launch merges the plan's pieces, us, plan / short
    (20, 5, 2519, 20, 20, False),     # 18.2, 19.1
    (64, 8, 585, 8, 4, False),        # 14.8, 15.6
    (20, 5, 1380, 21, 3, False),      # 15.4, 16.1
    (16, 4, 317, 10, 10, False),      # 13.2, 14.0
    (32, 8, 2175, 43, 6, True),       # 21.7, 17.2
    (4, 4, 7859, 224, 4, True),       # 26.9, 21.8
    (12, 4, 66, 66, 27, True),        # 16.7, 13.6
])
def test_the_faster_form_of_a_call_with_few_observing_rows_is_taken(plan, Hq, Hkv, M, Ct, W, taken):
    assert (plan.short_form(Hkv, Hq // Hkv, 128, M, Ct, W, 1, 256) != 0) == taken


@pytest.mark.gpu
@pytest.mark.parametrize("Hq,Hkv,d,M,Ct,waves", SHORT)
def test_matches_oracle(Hq, Hkv, d, M, Ct, waves):
    g = torch.Generator().manual_seed(M + Ct)
    n = M + Ct
    q = (torch.randn((Hq, Ct, d), generator=g) * 1.5).to(torch.bfloat16)
    k = (torch.randn((Hkv, n + 3, d), generator=g) * 1.5).to(torch.bfloat16)   # logits of +-10: rows rescale
    v = torch.randn((Hkv, n + 3, d), generator=g).to(torch.bfloat16)
    k[:, n:] = float("nan")           # behind the last key
    v[:, n:] = float("nan")
    scale = 1.0 / math.sqrt(d)
    heads = range(Hkv) if Hkv <= 3 else [0, Hkv - 1]
    G = Hq // Hkv
    mine = [h * G + i for h in heads for i in range(G)]
    o_ref, l_ref, s_ref = oracle_kv_heads_dense(to_np(q), to_np(k), to_np(v), M, scale, heads)
    for score in (True, False):
        out, lse, s = binding.reform_chunk_attend_score(q.to(DEV), k.to(DEV), v.to(DEV), M, scale, want_score=score)
        torch.cuda.synchronize()
        # the bounds of the other attention tests: bf16 rounding of P and of the output
        assert_close(to_np(out)[mine], o_ref, 2e-2, "out", row_floor=True)
        assert_close(to_np(lse)[mine], l_ref, 1e-5, "lse")
        if score:
            assert_scores_close(to_np(s)[list(heads), :n], s_ref[:, :n], 2e-2, "score")


@pytest.mark.gpu
def test_strides_and_logits_that_are_nan():
    """Rows of a tensor of tokens by heads (q and out), and NaN keys: rows that see one are NaN, the others are not touched."""
    Hq, Hkv, d, M, Ct = 6, 2, 128, 40, 50
    g = torch.Generator().manual_seed(5)
    n = M + Ct
    q = torch.randn((Ct, Hq, d), generator=g).to(torch.bfloat16).to(DEV).transpose(0, 1)
    k = torch.randn((Hkv, n, d), generator=g).to(torch.bfloat16).to(DEV)
    v = torch.randn((Hkv, n, d), generator=g).to(torch.bfloat16).to(DEV)
    store = torch.full((Ct, Hq + 1, d), 3.0, dtype=torch.bfloat16, device=DEV)
    out = store[:, :Hq].transpose(0, 1)
    k[1, M + 20] = float("nan")
    binding.reform_chunk_attend_score(q, k, v, M, 0.1, out=out, want_score=False)
    torch.cuda.synchronize()
    dense = binding.reform_chunk_attend_score(q.contiguous(), k, v, M, 0.1, want_score=False)[0]
    torch.cuda.synchronize()
    assert (store[:, Hq:] == 3.0).all()
    assert torch.equal(torch.nan_to_num(out.float(), nan=77.0), torch.nan_to_num(dense.float(), nan=77.0))
    nan = torch.isnan(out.float()).all(dim=-1)
    assert nan[3:, 20:].all() and not torch.isnan(out[:3].float()).any() and not torch.isnan(out[3:, :20].float()).any()


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHARED + LONGER, ids=lambda s: "x".join(map(str, s)))
def test_shares_and_the_other_forms_match_oracle(shape):
    """Twice with room for all pieces, once without."""
    test_gpu_attend_split.test_split_forward_matches_oracle(shape)
