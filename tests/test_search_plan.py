"""Host-side: how the search that walks whole frames is dealt to workgroups."""
import pytest
import torch

from plans import CUS, params, units, walk_plan

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
