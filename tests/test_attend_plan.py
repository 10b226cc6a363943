"""The plans of the attention, replayed on the CPU: every key tile of every row block of a forward pass split in the form
of eight waves belongs to exactly one workgroup, and the merge reads the slots that were written; the form that the GPU tests'
shapes take; and what is planned for a workspace without room for all of it.  The header that the kernels use is
compiled as host code (attend_plan_replay.cpp)."""
import ctypes
import random

import pytest
import torch

import helpers
import test_gpu_attend_score_narrow
import test_gpu_attend_score_waves
import test_gpu_attend_score_wide
import test_gpu_attend_split
from paper_2506_01215_amd import binding

EIGHT, FOUR, NARROW = 8, 4, 2      # kScoreEight, kScoreFour, kScoreNarrow


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    return helpers.load_attend_plan(tmp_path_factory)


@pytest.fixture(scope="module")
def replay(plan):
    return plan.replay_eight


@pytest.mark.parametrize("G", range(1, 33))
def test_every_tile_has_one_workgroup(replay, G):
    rng = random.Random(G)
    split = 0
    for _ in range(300):
        Hkv = rng.choice([1, 2, 4, 8, 32])
        M = rng.choice([0, rng.randint(0, 300), rng.randint(0, 70000)])
        Ct = rng.choice([1, rng.randint(1, 40), rng.randint(1, 6000)])
        rc = replay(Hkv, G, rng.choice([64, 128]), M, Ct, rng.choice([256, 256, 32, 304]))
        assert rc in (0, 1), (Hkv, G, M, Ct, rc)
        split += rc == 0
    assert split > 50


@pytest.mark.parametrize("Hkv,G", [(1, 16), (1, 32), (2, 16), (1, 71), (8, 4), (1, 128)])
def test_caches_whose_keys_times_heads_pass_32_bits(replay, Hkv, G):
    """K and V of 2^30 keys of 64 bf16 elements fill the card: G * keys reaches 2^37 for G = 128."""
    rng = random.Random(G)
    for M in [(1 << 31) // G - 300, (1 << 31) // G + 300, (1 << 32) // G + 77, (1 << 30) - 65]:
        if Hkv * M > (1 << 30):
            continue
        for Ct in (1, 256 // G + 1, 16, 33, 700):
            assert replay(Hkv, G, 64, M + rng.randint(0, 63), Ct, 256) in (0, 1), (Hkv, G, M, Ct)


def score_form(plan, shape):
    Hq, Hkv, d, M, Ct, W = shape
    return plan.score_form(Hkv, Hq // Hkv, d, M, Ct, W, 256)


def form_and_slices(plan, shape):
    return divmod(score_form(plan, shape), 1000)


def test_the_score_shapes_of_the_gpu_tests_take_the_form_they_are_for(plan):
    for shape in test_gpu_attend_split.SLICED:
        assert form_and_slices(plan, shape)[0] and form_and_slices(plan, shape)[1] > 1, shape
    for shape in test_gpu_attend_split.FEW_ROWS:
        assert score_form(plan, shape) == 1, shape
    for shape in test_gpu_attend_score_waves.FOUR_WAVES:
        assert score_form(plan, shape) == 4, shape
    for shape in test_gpu_attend_score_waves.TILED:
        assert form_and_slices(plan, shape)[0], shape


@pytest.mark.parametrize("shape", test_gpu_attend_score_narrow.NARROW)
def test_score_shapes_of_the_narrow_tests_take_the_narrow_form_in_slices(plan, shape):
    form, slices = form_and_slices(plan, shape)
    assert form == NARROW and slices > 1


@pytest.mark.parametrize("shape", test_gpu_attend_score_wide.EIGHT)
def test_score_shapes_of_the_tests_of_eight_waves_take_them(plan, shape):
    assert form_and_slices(plan, shape) == (EIGHT, 1)


@pytest.mark.parametrize("shape", test_gpu_attend_score_wide.FOUR)
def test_score_shapes_of_the_tests_of_four_waves_take_them_in_slices(plan, shape):
    form, slices = form_and_slices(plan, shape)
    assert form == FOUR and slices > 1


@pytest.mark.parametrize("Hq,Hkv,d,M,Ct,W", [
    (8, 8, 128, 8686, 141, 0),        # score alone 14.9 us tiled, 28.5 us with four waves to 32 keys
    (24, 8, 128, 4366, 45, 0),        # 15.1, 17.1
    (32, 8, 128, 4096, 40, 0),        # 18.4, 19.2
    (16, 4, 128, 94, 381, 0),         # 12.3, 15.1
    (16, 4, 128, 812, 381, 0),        # 96 blocks, 152 workgroups: 1.13 times
    (14, 2, 128, 620, 173, 0),        # 77 blocks, 50 workgroups: 1.05 times
    (8, 8, 64, 8686, 141, 0),         # 11.8, 16.0
    (24, 8, 64, 6158, 45, 0),         # 11.2, 13.0
])
def test_score_forms_measured_faster_tiled_stay_tiled(plan, Hq, Hkv, d, M, Ct, W):
    assert score_form(plan, (Hq, Hkv, d, M, Ct, W)) >= 1000


@pytest.mark.parametrize("Hq,Hkv,d,M,Ct,W", [
    (16, 4, 128, 1614, 45, 0),        # 10.4 us tiled, 6.3 us with four waves
    (14, 2, 128, 3406, 141, 0),       # 16.2, 11.7
    (8, 8, 128, 2510, 141, 0),        # 14.7, 11.3
    (32, 8, 64, 958, 253, 0),         # 14.1, 11.1
    (32, 8, 128, 64, 269, 0),         # 68 blocks, 88 workgroups: 0.87 times
    (24, 8, 128, 52, 461, 0),         # 87 blocks, 136 workgroups: 0.89 times
    (64, 8, 128, 524, 189, 0),        # 96 blocks, 184 workgroups: 0.94 times
    (14, 2, 64, 14641, 47, 0),
])
def test_score_forms_measured_faster_with_four_waves_take_them(plan, Hq, Hkv, d, M, Ct, W):
    assert score_form(plan, (Hq, Hkv, d, M, Ct, W)) == 4


def shares_in(plan, shape, scratch, scored=0):
    Hq, Hkv, d, M, Ct = shape
    need = ctypes.c_long()
    shares = plan.fwd_shares(Hkv, Hq // Hkv, d, M, Ct, scored, 256, ctypes.c_long(scratch), ctypes.byref(need))
    return shares, need.value


@pytest.mark.parametrize("shape", [
    (32, 8, 128, 16640, 1),           # one token: 290 us whole, 18 us with 32 shares
    (8, 8, 128, 4096, 17),
    (16, 4, 64, 30000, 40),
    (8, 8, 128, 51873, 379),
    (32, 8, 128, 2000, 100),
])
def test_the_forward_pass_takes_the_shares_that_its_scratch_holds(plan, shape):
    most, need = shares_in(plan, shape, -1)
    assert most >= 8
    assert shares_in(plan, shape, need) == (most, need)
    fewer, less = shares_in(plan, shape, need - 1)
    assert fewer >= 2 and 0.7 * need < less < need
    some, used = shares_in(plan, shape, need // 3)
    assert some >= 2 and 0.5 * (need // 3) < used <= need // 3
    assert shares_in(plan, shape, 0) == (0, 0)


def test_forward_plans_fit_their_scratch(plan):
    rng = random.Random(3)
    cut = 0
    for _ in range(4000):
        Hkv, G = rng.choice([1, 2, 4, 8]), rng.choice([1, 2, 3, 4, 7, 8])
        shape = (Hkv * G, Hkv, rng.choice([64, 128]), rng.choice([0, rng.randint(0, 40000)]), int(2 ** rng.uniform(0, 13)))
        scored = rng.randint(0, 1)
        most, need = shares_in(plan, shape, -1, scored)
        for more in (0, 4096, need // 9):
            assert shares_in(plan, shape, need + more, scored) == (most, need), (shape, more)
        scratch = rng.randint(0, need)
        got, used = shares_in(plan, shape, scratch, scored)
        assert used <= scratch and (used > 0) == (got > 0) and got != 1, (shape, scratch)
        cut += 0 < got != most
    assert cut > 500


def slices_in(plan, shape, scratch):
    Hq, Hkv, d, M, Ct, W = shape
    return plan.score_slices(Hkv, Hq // Hkv, d, M, Ct, W, 256, ctypes.c_long(scratch))


@pytest.mark.parametrize("shape", [
    (14, 2, 64, 0, 12000, 0),         # uncut 994 us, in 4 slices 362, in 32 205
    (16, 4, 64, 8192, 8192, 0),       # 500, 340, in 16 289
    (16, 4, 128, 0, 4000, 0),
    (32, 8, 128, 8192, 8192, 0),
])
def test_score_takes_the_slices_that_its_scratch_holds(plan, shape):
    slice_bytes = shape[1] * (shape[3] + shape[4]) * 4
    most = slices_in(plan, shape, -1)
    assert most >= 8
    assert slices_in(plan, shape, most * slice_bytes) == most
    fewer = slices_in(plan, shape, most * slice_bytes - 1)
    assert most / 3 < fewer < most
    assert slices_in(plan, shape, 5 * slice_bytes - 1) in (3, 4)
    assert slices_in(plan, shape, 2 * slice_bytes - 1) == 1
    assert slices_in(plan, shape, 0) == 1


def test_score_plans_fit_their_scratch(plan):
    rng = random.Random(2)
    cut = 0
    for _ in range(4000):
        Hkv, G = rng.choice([1, 2, 4, 8]), rng.choice([1, 2, 3, 4, 7, 8])
        shape = (Hkv * G, Hkv, rng.choice([64, 128]), rng.choice([0, rng.randint(0, 40000)]), rng.randint(1, 9000), 0)
        most = slices_in(plan, shape, -1)
        for more in (0, 4096, most * Hkv):
            assert slices_in(plan, shape, most * Hkv * (shape[3] + shape[4]) * 4 + more) == most, (shape, more)
        scratch = rng.randint(0, most * Hkv * (shape[3] + shape[4]) * 4)
        got = slices_in(plan, shape, scratch)
        assert got >= 1, (shape, scratch)
        cut += 1 < got != most
    assert cut > 500


@pytest.mark.parametrize("Hq,Hkv,M,Ct,W", [
    (64, 8, 0, 3211, 128),            # score alone 23.9 us uncut, 17.2 us with the heads in two
    (64, 8, 2985, 487, 128),          # 23.1, 16.4
    (16, 2, 12949, 278, 117),         # 22.8, 16.3
    (14, 2, 14253, 864, 128),         # 20.5, 15.7
    (16, 4, 5121, 158, 158),          # 16.8, 13.9
])
def test_heads_are_cut_where_that_was_measured_faster(plan, Hq, Hkv, M, Ct, W):
    assert form_and_slices(plan, (Hq, Hkv, 64, M, Ct, W))[1] > 1


@pytest.mark.parametrize("Hq,Hkv,M,Ct,W", [
    (8, 8, 2408, 520, 0),             # 11.8 us uncut, 13.3 us in three slices
    (8, 8, 3606, 1084, 0),            # 17.6, 19.0
    (4, 4, 2195, 4124, 594),          # 12.3, 13.5
])
def test_one_head_to_a_group_stays_uncut_where_that_was_measured_faster(plan, Hq, Hkv, M, Ct, W):
    assert form_and_slices(plan, (Hq, Hkv, 64, M, Ct, W)) == (NARROW, 1)


@pytest.mark.parametrize("Hq,Hkv,d,M,Ct,W,merged", [
    (8, 8, 128, 59999, 1, 0, False),  # 68.1 us in two launches, 71.2 in one
    (8, 8, 128, 19970, 30, 0, False), # 35.8, 37.3
    (8, 8, 64, 19750, 250, 17, False),# 34.5, 36.5
    (14, 2, 64, 19984, 16, 0, False), # 24.4, 27.3
    (14, 2, 64, 19999, 1, 0, True),   # 17.0, 13.3
    (8, 8, 128, 13970, 30, 0, True),  # 29.9, 28.4
    (8, 8, 128, 4096, 17, 0, True),
])
def test_merging_in_the_score_launch_where_it_was_measured_faster(plan, Hq, Hkv, d, M, Ct, W, merged):
    assert plan.plan_form(Hkv, Hq // Hkv, d, M, Ct, W, 1, 256) == (6 if merged else 2)


@pytest.mark.parametrize("Hq,Hkv,d,M,Ct,shared", [
    (4, 4, 128, 124, 16, False),      # 13.0 us whole, 14.9 us with two shares
    (4, 4, 64, 120, 60, False),       # 10.0, 10.3
    (8, 2, 32, 162, 128, False),      # 11.9, 12.3
    (4, 4, 128, 184, 16, True),       # 15.5, 14.8
    (4, 4, 32, 140, 60, True),        # 8.3, 8.1
    (8, 2, 32, 272, 128, True),
    (4, 4, 64, 256, 128, True),
])
def test_fp32_key_blocks_are_shared_where_that_was_measured_faster(Hq, Hkv, d, M, Ct, shared):
    q, k = torch.empty((Hq, Ct, d)), torch.empty((Hkv, M + Ct, d))
    need = binding.attend_workspace_bytes(binding.attn_desc(q, k, q, M, 0.1))
    assert (need > (Hq * Ct * 4 + 255) // 256 * 256) == shared
