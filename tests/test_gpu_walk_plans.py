"""GPU parity of the search that walks whole frames, at deals that are asserted and not assumed: how many runs of rows
and frame groups a problem is cut into is read from the library's own plan."""
import pytest
import torch

from workloads import CONFIGS, make_clip_batch

from helpers import compare_with_oracle, run_gpu
from plans import matrix_cores, params, search_guesses, search_walks, walk_plan
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


@pytest.mark.parametrize("B,F,H,W,C,r", [(1, 12, 16, 16, 3072, 1), (1, 33, 16, 16, 1024, 1), (1, 9, 32, 32, 1024, 0),
                                          (1, 13, 12, 19, 3296, 1), (1, 22, 9, 17, 2976, 0)])
def test_fp32_error_is_no_larger_than_the_wave_per_token_search(B, F, H, W, C, r):
    """fp32 problems that are too small for the tile-wise matrix-core search walk all the same.  Relative error of
    the similarities against 64 bits, over the tokens that match their own cell: 7.5e-8 to 8.6e-8 on the wave-per-token
    kernels over 30 such shapes."""
    import paper_2605_07355_amd as ttf
    p = params(B, F, H, W, C, torch.float32, r)
    assert search_walks(p) and not matrix_cores(p)
    g = torch.Generator(device="cuda").manual_seed(C + F)
    a = torch.randn((B, 1, H, W, C), device="cuda", generator=g)
    amp = 0.3 + 1.4 * torch.rand((B, F - 1, H, W, 1), device="cuda", generator=g)
    x = torch.cat([a, a + amp * torch.randn((B, F - 1, H, W, C), device="cuda", generator=g)], 1).contiguous()
    buf = ttf.TTFBuffers.allocate(B, F, H, W, C, x.dtype, x.device)
    ttf.ttf_compress(x, r=r, t=0.7, anchor=0, buffers=buf)
    torch.cuda.synchronize()
    xd = x.double()
    n = xd.norm(dim=-1)
    want = ((xd[:, 1:] * xd[:, :1]).sum(-1) / (n[:, 1:] * n[:, :1])).flatten(2)
    own = buf.best_idx[:, 1:] == torch.arange(H * W, device="cuda", dtype=torch.int32)
    assert own.float().mean() > 0.9
    err = (buf.best_sim[:, 1:].double() - want)[own]
    assert (err.norm() / want[own].norm()).item() < 7.4e-8


@pytest.mark.parametrize("B,F,H,W,C,r,dtype,guesses", [
    (3, 6, 16, 16, 1024, 1, "bf16", False),     # below the line from which such grids walk
    (2, 6, 16, 16, 1024, 2, "bf16", False),
    (2, 9, 8, 32, 1024, 1, "bf16", False),
    (1, 7, 16, 16, 2048, 0, "bf16", False),
    (2, 33, 16, 16, 1024, 1, "bf16", False),
    (16, 8, 16, 16, 2048, 1, "bf16", True),
    (2, 6, 13, 16, 1024, 1, "bf16", True),
    (2, 11, 14, 14, 1024, 2, "bf16", True),
    (4, 18, 16, 16, 1024, 1, "f32", True),
])
def test_bits_do_not_depend_on_the_setting(B, F, H, W, C, r, dtype, guesses):
    assert search_guesses(params(B, F, H, W, C, _torch(dtype), r), 1) == guesses
    batch = make_clip_batch(_cfg(B, F, H, W, C, r, dtype), seed=1300 + F)
    first = None
    for mode in (-1, 1, None):
        _, out = run_gpu(batch.x, r, 0.7, speculation=mode)
        b, n = out.buffers, int(out.buffers.row_offsets[-1])
        got = (b.best_sim, b.best_idx, b.fuse_map, b.anchor_index, b.row_offsets, b.src_index[:n])
        first = first or got
        assert all(torch.equal(u, v) for u, v in zip(first, got)), mode
