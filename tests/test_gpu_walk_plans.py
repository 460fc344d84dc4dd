"""GPU parity of the search that walks whole frames, at deals that are asserted and not assumed: how many runs of rows
and frame groups a problem is cut into is read from the library's own plan."""
import pytest
import torch

from workloads import CONFIGS

from helpers import compare_with_oracle, run_gpu
from plans import params, walk_plan
from test_gpu_parity import _prepared

pytestmark = pytest.mark.gpu


def _cfg(B, F, H, W, C, r, dtype="bf16"):
    return CONFIGS["qwen3vl_2b"].scaled(B=B, F=F, H=H, W=W, C=C, r=r, max_offset=min(max(r, 1), 2), sigma=0.5, dtype=dtype)


def _torch(dtype):
    return torch.float32 if dtype == "f32" else torch.bfloat16


@pytest.mark.parametrize("B,F,H,W,C,r,dtype", [
    (1, 3, 150, 13, 1024, 1, "bf16"),
    (1, 2, 171, 16, 1088, 0, "bf16"),
    (1, 3, 170, 16, 1024, 2, "bf16"),          # 43 rows of patches, the last half empty
    (1, 3, 290, 13, 1024, 1, "f32"),
])
def test_tall_grids_in_many_runs(B, F, H, W, C, r, dtype):
    plan = walk_plan(params(B, F, H, W, C, _torch(dtype), r), F - 1, False)
    assert plan.ok and plan.ysegs > 4, plan.ysegs
    cfg = _cfg(B, F, H, W, C, r, dtype)
    batch, res = _prepared(cfg, seed=1200 + H)
    for mode in (-1, 1):
        _, out = run_gpu(batch.x, r, cfg.t[0], speculation=mode)
        compare_with_oracle(batch.x, out, res)
