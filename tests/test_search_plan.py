"""Host-side: which problems are searched by walking whole frames, and how they are dealt to workgroups."""
import random

import pytest
import torch

from plans import CUS, kept_share, matrix_cores, params, search_guesses, search_walks, units, walk_plan

BF, F32 = torch.bfloat16, torch.float32


@pytest.mark.parametrize("B,F,H,W,C,dtype", [
    (2**18 - 1, 2, 1, 1, 65664, BF),          # 64 GiB of one-token frames in 33 channel shares
    (2**17 - 1, 4, 1, 1, 131072, BF),
    (2**18 - 1, 2, 1, 1, 33792, F32),
])
def test_a_launch_stays_below_2_to_32_threads(B, F, H, W, C, dtype):
    p = params(B, F, H, W, C, dtype)
    for frames, sums in ((F - 1, False), (F, False), (F, True)):
        plan = walk_plan(p, frames, sums)
        assert not plan.ok or units(p, plan) * 512 < 2**32


@pytest.mark.parametrize("B,frames,H,W,C,r,dtype", [
    (1, 6, 848, 16, 1024, 1, BF),             # 430 us on 24 workgroups, 75 on the tile-wise kernels
    (1, 3, 396, 16, 4096, 1, BF),
    (2, 9, 204, 16, 2048, 0, BF),
    (1, 1, 976, 32, 2048, 2, BF),             # patches
    (1, 2, 576, 32, 1024, 1, F32),
    (1, 1, 2868, 13, 896, 1, F32),
])
def test_tall_grids_fill_the_chip(B, frames, H, W, C, r, dtype):
    p = params(B, frames + 1, H, W, C, dtype, r)
    plan = walk_plan(p, frames, False)
    assert plan.ok and units(p, plan) >= 0.75 * CUS


@pytest.mark.parametrize("B,frames,C", [(2, 255, 4096), (16, 31, 4096), (8, 40, 1024)])
def test_long_runs_where_frames_fill_the_chip(B, frames, C):
    plan = walk_plan(params(B, frames + 1, 16, 16, C, BF), frames, False)
    assert plan.ok and plan.ysegs <= 4          # the kept part of a pass is measured in whole rows of a run


@pytest.mark.parametrize("B,frames,H,W,C,r,ysegs", [
    # segments: us at a power of two of runs, at this many, on the tile-wise kernels
    (1, 68, 20, 16, 3200, 2, 5),              # 71 / 58 / 69
    (2, 24, 12, 16, 3200, 2, 3),              # 44 / 37 / 43
    (8, 5, 24, 14, 2048, 2, 6),               # 40 / 34 / 46
    (1, 33, 18, 32, 2368, 1, 6),              # 57 / 48.5 / 57
    (1, 2, 33, 16, 1152, 2, 8),               # (tied) 48.5 / 49 with five
    (2, 256, 16, 16, 4096, 1, 4),
])
def test_runs_that_fill_the_chip(B, frames, H, W, C, r, ysegs):
    plan = walk_plan(params(B, frames, H, W, C, BF, r), frames, False)
    assert plan.ok and plan.ysegs == ysegs


def _limit(B, H, W, C, dtype, r):
    """The most frames of a clip that still walks."""
    return max(F for F in range(2, 400) if search_walks(params(B, F, H, W, C, dtype, r)))


@pytest.mark.parametrize("B,H,W,C,dtype,r,most", [
    (1, 16, 20, 1024, BF, 2, 31),             # products of all frames in the room of the anchor's copy
    (1, 14, 14, 1088, BF, 1, 62),
    (1, 18, 18, 2048, BF, 2, 69),
    (1, 16, 16, 4096, F32, 1, None),
])
def test_a_segment_walks_where_its_clip_does(B, H, W, C, dtype, r, most):
    limit = _limit(B, H, W, C, dtype, r)
    assert limit < 399 and most in (None, limit), limit
    for F in range(2, limit + 3):
        assert search_walks(params(B, F - 1, H, W, C, dtype, r), segment=True) == search_walks(params(B, F, H, W, C, dtype, r)), F


def test_a_segment_takes_the_search_of_its_clip():
    rng = random.Random(7)
    for _ in range(4000):
        B, F = rng.choice([1, 1, 2, 3, 4, 8, 16]), rng.choice([2, 3, 4, 5, 9, 10, 17, 18, 31, 55, 64, 65, 100, 154, 200])
        H, W = rng.choice([1, 2, 3, 8, 14, 16, 18, 32]), rng.choice([1, 4, 8, 13, 14, 16, 17, 18, 20, 24, 32, 33, 40, 48])
        C = rng.choice([64, 256, 768, 1000, 1024, 1056, 1088, 1152, 2048, 2112, 4096, 4160])
        dtype, r = rng.choice([BF, BF, F32]), rng.choice([0, 1, 1, 2])
        clip, seg = params(B, F, H, W, C, dtype, r), params(B, F - 1, H, W, C, dtype, r)
        assert search_walks(seg, True) == search_walks(clip), (B, F, H, W, C, dtype, r)
        assert matrix_cores(seg, True) == matrix_cores(clip), (B, F, H, W, C, dtype, r)


def test_only_problems_that_walk_guess_their_anchor():
    """The search of a problem, and so the bits of its similarities, do not depend on the setting."""
    rng, guessing = random.Random(8), 0
    for _ in range(6000):
        B, F = rng.choice([1, 2, 3, 4, 8, 16, 40]), rng.choice([1, 2, 3, 6, 9, 16, 32, 64, 100, 200])
        H, W = rng.choice([1, 4, 8, 13, 14, 16, 32, 64]), rng.choice([3, 13, 14, 16, 16, 17, 24, 32, 32, 48])
        C, r = rng.choice([512, 1000, 1024, 1056, 1152, 2048, 4096]), rng.choice([0, 1, 1, 2, 3])
        p = params(B, F, H, W, C, rng.choice([BF, BF, F32]), r)
        guesses = [search_guesses(p, mode) >= 0 for mode in (-1, 0, 1)]
        assert not guesses[0] and guesses[1] <= guesses[2] <= search_walks(p), (B, F, H, W, C, r, guesses)
        guessing += guesses[2]
    assert guessing > 300


@pytest.mark.parametrize("B,F,H,W,C,r,clear,taken", [
    # us with the guesses, with them dropped, without guessing
    (16, 32, 16, 16, 4096, 1, 16, True),      # 340 / - / 455
    (16, 32, 16, 16, 4096, 1, 12, False),     # 556 / 523 / 494
    (8, 20, 24, 24, 2048, 1, 6, False),       # 290 / 226 / 195
    (4, 64, 16, 16, 4096, 1, 3, False),       # 304 / 279 / 253
    (8, 16, 32, 32, 2048, 1, 4, False),       # 421 / 317 / 285
    (12, 32, 14, 14, 4096, 1, 6, False),      # 435 / 346 / 320
    (128, 16, 16, 16, 2048, 1, 124, True),    # 927 / - / 1013
    (64, 32, 14, 14, 2048, 1, 61, True),      # 706 / 820 / 767
    (32, 20, 24, 24, 2048, 1, 31, True),      # 679 / 765 / 683
    (64, 16, 16, 16, 2048, 1, 56, False),     # 577 / 537 / 499
])
def test_guesses_taken_with_so_many_clear_clips(B, F, H, W, C, r, clear, taken):
    need = search_guesses(params(B, F, H, W, C, BF, r), 0)
    assert (0 <= need <= clear) == taken


def test_default_frame_counts_of_the_guess():
    took = [F for F in range(2, 130) if search_guesses(params(16, F, 16, 16, 4096, BF), 0) >= 0]
    assert took == list(range(12, 129))       # F 12: 203 us two-pass, 163 with the guesses; F 15: 242 / 195


@pytest.mark.parametrize("B,F,H,W,C,r,taken,dtype", [
    # us two-pass / with the guess of clips of one scene, and of scenes of 32 frames
    (8, 128, 16, 16, 4096, 1, True, BF),      # 968 / 672, 1351 / 1398
    (16, 66, 16, 16, 2048, 1, True, BF),      # 489 / 422, 602 / 647
    (8, 72, 16, 16, 4096, 0, True, BF),       # 494 / 403, 639 / 674
    (6, 66, 32, 32, 3072, 2, True, BF),       # 1163 / 1096, 1458 / 1529
    (4, 100, 16, 16, 4096, 1, True, F32),     # 748 / 609, 1008 / 1050
    (2, 100, 16, 16, 4096, 0, False, BF),     # 202 / 175, 258 / 290
    (4, 100, 24, 24, 2048, 1, False, BF),     # 408 / 378, 552 / 593
    (14, 84, 20, 28, 1024, 0, False, BF),     # 595 / 560, 766 / 845
    (16, 100, 14, 14, 1024, 1, False, BF),    # 308 / 323, 396 / 460
    (8, 129, 16, 16, 4096, 1, False, BF),
])
def test_guess_of_long_clips(B, F, H, W, C, r, taken, dtype):
    assert (search_guesses(params(B, F, H, W, C, dtype, r), 0) >= 0) == taken


@pytest.mark.parametrize("B,F,H,W,C,r,taken,dtype", [
    (2, 64, 32, 32, 1024, 1, False, BF),      # all clear: 157 us two-pass, 176 with the guesses
    (4, 40, 32, 26, 1536, 2, False, BF),      # 205 / 265
    (8, 12, 32, 32, 2048, 2, False, BF),      # 197 / 224
    (4, 64, 32, 32, 4096, 2, True, BF),       # 986 / 816
    (16, 12, 16, 16, 4096, 1, True, BF),      # 203 / 163
    (16, 64, 16, 16, 1024, 1, True, BF),      # 248 / 233
    (1, 14, 400, 32, 2048, 2, False, BF),     # 345 / 411
    (18, 64, 16, 14, 1024, 0, False, BF),     # 250 / 281
    (23, 14, 32, 16, 2048, 1, True, BF),      # 321 / 271
    (1, 16, 300, 16, 2048, 1, False, BF),     # 157 / 183
    (1, 64, 64, 64, 1024, 1, False, BF),      # 271 / 283
    (2, 24, 36, 64, 2048, 2, False, BF),      # 222 / 244
    (1, 32, 200, 16, 4096, 1, True, BF),      # 360 / 311
    (4, 16, 128, 16, 2048, 1, True, BF),      # 242 / 222
    (7, 33, 32, 16, 1088, 1, True, F32),      # 323 / 312
    (16, 32, 16, 16, 2048, 1, True, F32),     # 470 / 396
])
def test_guess_where_it_pays(B, F, H, W, C, r, taken, dtype):
    assert (search_guesses(params(B, F, H, W, C, dtype, r), 0) >= 0) == taken


@pytest.mark.parametrize("B,F,H,W,C,r,dtype", [
    (33, 40, 2, 14, 1024, 1, BF),             # many frames of few tokens: no room for sums beside the products
    (2, 300, 2, 16, 1024, 1, BF),
    (70, 60, 1, 28, 1152, 1, BF),
    (3, 64, 16, 16, 1056, 1, F32),            # no room for the sums of two runs
    (5, 40, 4, 13, 1056, 1, F32),
])
def test_the_guess_finds_room_for_its_sums(B, F, H, W, C, r, dtype):
    p = params(B, F, H, W, C, dtype, r)
    assert search_walks(p) and search_guesses(p, 1) == 0


def test_guess_is_available_wherever_such_shapes_walk():
    rng = random.Random(9)
    for _ in range(3000):
        B, F = rng.choice([1, 3, 16, 70]), rng.choice([2, 5, 12, 40, 64, 100, 300])
        H, W = rng.randint(1, 40), rng.choice([12, 13, 14, 16, 16, 24, 30, 32, 48, 64])
        C, r = rng.choice([1024, 1152, 2048, 2176, 4096, 4224]), rng.choice([0, 1, 2])
        p = params(B, F, H, W, C, BF, r)
        strips = H * W // 32 if (W == 16 and H % 4 == 0) or (W == 32 and H % 2 == 0) else (
            (H + 1) // 2 if W <= 16 else H * (((W + 15) // 16 + 1) // 2))
        if search_walks(p) and 10 * H * W >= 7 * 32 * strips:
            assert search_guesses(p, 1) == 0, (B, F, H, W, C, r)


@pytest.mark.parametrize("B,F,H,W,C,segment,walks", [
    # 5x5 window: time of the other search, time of the walk, us
    (64, 40, 2, 16, 1024, True, False),       # 66 / 88
    (64, 40, 2, 12, 1024, False, False),      # 123 / 140 (tied)
    (32, 24, 2, 12, 1152, True, False),       # 37 / 42
    (32, 24, 2, 8, 1152, True, True),         # 37 / 34
    (64, 24, 2, 14, 1536, True, False),       # 61 / 69
    (64, 8, 2, 16, 1536, False, True),        # 103 / 100 (tied)
    (32, 8, 2, 16, 2048, True, True),         # 40 / 30
    (1, 10, 48, 16, 2048, False, False),      # 41 / 48.5
    (1, 10, 64, 16, 1536, True, False),       # 30 / 33
    (4, 5, 88, 16, 1280, False, True),        # 75 / 65
])
def test_lines_of_the_5x5_window(B, F, H, W, C, segment, walks):
    assert search_walks(params(B, F, H, W, C, BF, 2), segment) == walks


@pytest.mark.parametrize("B,F,H,C,walks", [
    # fp32 on rows of 32 cells: time of the other search, time of the walk, us
    (1, 33, 64, 3424, False),                 # 503 / 539
    (8, 33, 32, 832, False),                  # 526 / 551
    (1, 73, 32, 3584, True),                  # 583 / 518
    (2, 34, 16, 3104, True),                  # 237 / 199 (segment)
    (4, 48, 32, 1024, True),                  # 473 / 444 (tied)
    (1, 9, 32, 3008, True),                   # 176 / 95
])
def test_fp32_rows_of_32_cells(B, F, H, C, walks):
    assert search_walks(params(B, F, H, 32, C, F32, 1)) == walks


@pytest.mark.parametrize("H,W,C,dtype,r,want", [
    (2, 2, 1024, BF, 5, "mfma_bf16_padded"),  # a radius beyond the grid is the grid's own: 2
    (1, 1, 256, BF, 9, "mfma_bf16_padded"),
    (3, 2, 1024, BF, 5, "general"),           # 3
])
def test_route_of_a_radius_beyond_the_grid(H, W, C, dtype, r, want):
    import paper_2605_07355_amd as ttf
    assert ttf.ttf_search_route(2, 4, H, W, C, dtype, r=r) == ttf.ttf_search_route(2, 4, H, W, C, dtype, r=max(H, W)) == want


@pytest.mark.parametrize("B,F,H,W,C,dtype,r,kept", [
    (1, 4, 14, 16, 4096, F32, 1, 0.0),        # wave-per-token search below 16 MiB: us left in the caches / not, 75.5 / 56.5
    (2, 6, 16, 15, 1280, F32, 2, 0.0),        # 62.5 / 57.5
    (3, 2, 32, 24, 1000, F32, 0, 1.0),        # above: 45.8 / 54.8
    (1, 10, 24, 16, 2048, F32, 1, 1.0),       # 50.5 / 56
    (1, 4, 16, 16, 2048, BF, 1, 1.0),         # on the matrix cores
    (2, 256, 16, 16, 4096, BF, 1, 0.3125),
])
def test_what_the_frame_sums_leave_in_the_caches(B, F, H, W, C, dtype, r, kept):
    p = params(B, F, H, W, C, dtype, r)
    assert kept_share(p, search_walks(p), matrix_cores(p)) == kept
