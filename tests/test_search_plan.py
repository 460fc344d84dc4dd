"""Host-side: how the search that walks whole frames is dealt to workgroups."""
import pytest
import torch

from plans import params, units, walk_plan

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
