"""GPU parity of the search that walks whole frames, at deals that are asserted and not assumed: how many runs of rows
and frame groups a problem is cut into is read from the library's own plan."""
import pytest
import torch

from workloads import CONFIGS

from helpers import compare_with_oracle, run_gpu
from plans import matrix_cores, params, search_walks, walk_plan
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


@pytest.mark.parametrize("B,F,H,W,C,r,dtype", [
    (1, 31, 16, 20, 1024, 2, "bf16"),          # the last clip that walks ...
    (1, 32, 16, 20, 1024, 2, "bf16"),          # ... and the first that does not
    (1, 62, 14, 14, 1088, 1, "bf16"),
    (1, 63, 14, 14, 1088, 1, "bf16"),
    (3, 10, 16, 16, 256, 1, "f32"),            # matrix cores from nine source frames on
    (3, 9, 16, 16, 256, 1, "f32"),
])
def test_segment_gives_the_bits_of_its_clip(B, F, H, W, C, r, dtype):
    """The first frame as a fixed anchor, and the rest of the clip as a segment against it."""
    import paper_2605_07355_amd as ttf
    torch_dtype = _torch(dtype)
    clip = params(B, F, H, W, C, torch_dtype, r)
    assert search_walks(clip) == (F in (31, 62)) and (dtype == "bf16" or matrix_cores(clip) == (F == 10))
    g = torch.Generator(device="cuda").manual_seed(F)
    a = torch.randn((B, 1, H, W, C), device="cuda", generator=g)
    amp = 1.6 * torch.rand((B, F - 1, H, W, 1), device="cuda", generator=g)
    x = torch.cat([a, a + amp * torch.randn((B, F - 1, H, W, C), device="cuda", generator=g)], 1).to(torch_dtype)
    whole = ttf.TTFBuffers.allocate(B, F, H, W, C, x.dtype, x.device)
    seg = ttf.TTFBuffers.allocate(B, F - 1, H, W, C, x.dtype, x.device)
    ttf.ttf_compress(x, r=r, t=0.7, anchor=0, buffers=whole)
    ttf.ttf_compress_segment(x[:, 1:].contiguous(), x[:, 0].contiguous(), 0, r=r, t=0.7, buffers=seg)
    torch.cuda.synchronize()
    assert torch.equal(seg.best_sim, whole.best_sim[:, 1:])
    assert torch.equal(seg.best_idx, whole.best_idx[:, 1:])
    assert torch.equal(seg.fuse_map, whole.fuse_map[:, 1:])
