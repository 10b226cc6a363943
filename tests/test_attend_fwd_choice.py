"""The form that the forward pass takes, replayed on the CPU: every key tile of every row block of a plan of eight or four waves
belongs to exactly one workgroup and the merge reads the slots that were written; the GPU tests' shapes take the form they are
for, as it is launched; and of the two plans shapes measured in both have the faster one."""
import ctypes
import random

import pytest
import torch

import helpers
import test_gpu_attend_fwd_narrow
import test_gpu_attend_merge_score
import test_gpu_attend_split
from paper_2506_01215_amd import binding


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    return helpers.load_attend_plan(tmp_path_factory)


@pytest.mark.parametrize("G", list(range(1, 17)) + [32, 71])
def test_every_tile_has_one_workgroup(plan, G):
    rng = random.Random(G)
    narrow = 0
    for _ in range(300):
        Hkv, d = rng.choice([1, 2, 4, 8, 32]), rng.choice([64, 128])
        M = rng.choice([0, rng.randint(0, 300), rng.randint(0, 70000)])
        Ct = rng.choice([rng.randint(1, 40), rng.randint(1, 400), rng.randint(1, 6000)])
        scored, cus = rng.randint(0, 1), rng.choice([256, 256, 32, 304])
        assert plan.replay_chosen(Hkv, G, d, M, Ct, scored, cus) == 0, (Hkv, G, d, M, Ct, scored, cus)
        narrow += plan.plan_form(Hkv, G, d, M, Ct, 0, scored, cus) & 1
    assert narrow > 20


@pytest.mark.parametrize("Hkv,G", [(1, 16), (2, 16), (1, 71), (8, 4), (1, 128)])
def test_caches_whose_keys_times_heads_pass_32_bits(plan, Hkv, G):
    for M in [(1 << 31) // G - 300, (1 << 31) // G + 300, (1 << 32) // G + 77, (1 << 30) - 65]:
        if Hkv * M > (1 << 30):
            continue
        for Ct in (1, 256 // G + 1, 33, 700):
            for d in (64, 128):
                assert plan.replay_chosen(Hkv, G, d, M, Ct, 0, 256) == 0, (Hkv, G, d, M, Ct)


@pytest.mark.parametrize("Hkv,G,d,M,Ct", [
    (1, 8, 64, 4194304, 4096),        # 43.7 ms shared out, 69.7 whole: 128 row blocks on 256 compute units
    (1, 8, 128, 4194304, 4096),
    (1, 1, 64, 8388608, 16384),
    (2, 4, 64, 1 << 25, 1024),
])
def test_lists_too_long_for_every_share_are_shared_by_fewer(plan, Hkv, G, d, M, Ct):
    """A place in the list times the number of shares has to stay in 32 bits; the form is chosen by what is then run."""
    assert plan.form(Hkv, G, d, M, Ct, 0, 0, 256) & 2
    assert plan.replay_chosen(Hkv, G, d, M, Ct, 0, 256) == 0


@pytest.mark.parametrize("Hq,Hkv,d,M,Ct,W,form", test_gpu_attend_fwd_narrow.NARROW +
                         test_gpu_attend_fwd_narrow.BY_THE_SHORT_FORM)
def test_the_shapes_of_the_gpu_test_take_the_form_they_are_for(plan, Hq, Hkv, d, M, Ct, W, form):
    assert plan.form(Hkv, Hq // Hkv, d, M, Ct, W, 1, 256) == form


@pytest.mark.parametrize("Hq,Hkv,d,M,Ct,W,form", test_gpu_attend_split.SHAPES + test_gpu_attend_merge_score.MERGED +
                         test_gpu_attend_merge_score.WHOLE)
def test_the_shapes_of_the_tests_of_shares_and_merging_take_the_form_they_are_for(plan, Hq, Hkv, d, M, Ct, W, form):
    assert plan.form(Hkv, Hq // Hkv, d, M, Ct, W, 1, 256) == form


def test_less_room_than_all_reaches_every_form(plan):
    """The forms that a workspace between none and all leads to, as in test_gpu_attend_split."""
    reached = set()
    for Hq, Hkv, d, M, Ct, W, form in test_gpu_attend_split.PARTLY:
        args = (Hkv, Hq // Hkv, d, M, Ct, W, 1, 256)
        assert plan.form(*args) == form, args
        q, k = torch.empty((Hq, Ct, d), dtype=torch.bfloat16), torch.empty((Hkv, M + Ct, d), dtype=torch.bfloat16)
        need = binding.attend_workspace_bytes(binding.attn_desc(q, k, q, M, 0.1, W)) - (Hq * Ct * 4 + 255) // 256 * 256
        at = [plan.form_in(*args, ctypes.c_long(int(part * need))) for part in test_gpu_attend_split.PARTS]
        reached |= {(f & 9, f & 6) for f in at}
    # eight waves, four, attn_fwd_short: whole, shared out, merged by the score's launch; what four waves share out, attn_fwd_short
    # takes whole
    assert reached == {(form, bits) for form in (0, 1, 8) for bits in (0, 2, 6)} - {(1, 0)}


@pytest.mark.parametrize("Hq,Hkv,d,M,Ct", test_gpu_attend_split.MANY)
def test_many_row_blocks_are_taken_whole_by_eight_waves(plan, Hq, Hkv, d, M, Ct):
    assert plan.form(Hkv, Hq // Hkv, d, M, Ct, 0, 0, 256) == 0


def test_shared_out_row_blocks_of_eight_waves_have_their_shapes():
    """Several row blocks, at either width, with one head to a wave's rows, with a wave to each head and neither."""
    def kind(shape):
        Hq, Hkv, d, M, Ct = shape[:5]
        G = Hq // Hkv
        return d, "one head" if G == 1 else "a wave to a head" if 8 % G == 0 and Ct >= 32 else "rows"
    kinds = {kind(s) for s in test_gpu_attend_split.SHAPES if s[6] == 2 and s[0] // s[1] * s[4] > 256}
    assert kinds == {(d, k) for d in (64, 128) for k in ("one head", "a wave to a head", "rows")}


@pytest.mark.parametrize("Hq,Hkv,d,M,Ct,form", [
    (32, 8, 128, 0, 312, 1),          # 16.2 us with eight waves, 12.1 with four
    (32, 8, 128, 0, 1998, 1),         # 55.8, 50.5
    (16, 4, 128, 7942, 78, 3),        # 27.4, 23.2
    (32, 8, 64, 0, 4907, 1),          # 131, 115
    (32, 8, 128, 12603, 335, 2),      # 82.9, 96.6
    (8, 8, 128, 1113, 4033, 2),       # 69.3, 77.0
    (16, 4, 64, 10178, 873, 2),       # 56.8, 61.5
    (32, 8, 128, 569, 2651, 0),       # 87.5, 98.4
    (32, 8, 128, 32768, 32768, 0),
    # more than one round of row blocks at 64
    (8, 8, 64, 0, 12040, 2),          # 187.8, whole 204.7
    (14, 2, 64, 4010, 5232, 2),       # 160.1, whole 173.0
    (16, 4, 64, 0, 5379, 1),          # 95.6 whole, 91.9 in shares, 82.0
    (16, 4, 64, 0, 4763, 1),          # 77.6 in shares, 71.8
    # shares of many tiles
    (8, 8, 128, 51873, 379, 2),       # 98.5, 120.3
    (8, 8, 128, 53803, 284, 2),       # 94.7, 111.7
    (12, 4, 128, 94625, 86, 2),       # 84.3, 108.2
    (24, 8, 128, 46280, 127, 2),      # 90.7, 107.8
    (4, 4, 128, 18726, 344, 2),       # 32.9, 38.1
    (14, 2, 128, 31140, 53, 2),       # 31.3, 36.2
    (16, 4, 64, 76065, 90, 3),        # 54.7, 52.0
    (14, 2, 128, 6287, 69, 3),        # 25.6, 22.3
    (8, 8, 64, 31055, 281, 3),        # 48.4, 44.1
    (12, 4, 64, 14271, 117, 3),       # 26.1, 22.2
])
def test_the_faster_plan_is_taken(plan, Hq, Hkv, d, M, Ct, form):
    assert plan.plan_form(Hkv, Hq // Hkv, d, M, Ct, 0, 0, 256) == form
