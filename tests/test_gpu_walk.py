"""GPU parity of the search whose workgroups walk whole frames (bf16, C >= 1024, grids that are not whole 16-
or 32-wide tiles take it at every size): the ends of its column strips, patches, channel shares and frame
groups, as a pass on both anchor routes, as a segment and as a tied batch."""
import pytest
import torch

from workloads import CONFIGS

from helpers import compare_with_oracle, run_gpu
from test_gpu_next import _compare_tied, _run_tied, _tied_case
from test_gpu_parity import _prepared

pytestmark = pytest.mark.gpu

SHAPES = [
    # B, F,  H,  W,  C,    r
    (1, 4, 5, 17, 1024, 1),      # two strips, eight and nine cells wide
    (2, 5, 3, 30, 1088, 1),      # three strips; 17 groups of 64 channels over eight waves
    (1, 3, 1, 16, 2112, 0),      # one grid row; two shares of the channels, 66 K-steps
    (1, 36, 2, 14, 1024, 1),     # more frames than a workgroup takes
    (1, 6, 10, 18, 4160, 1),     # three shares
    (1, 9, 7, 40, 1024, 0),      # three strips without a margin
    (2, 3, 6, 13, 1024, 2),      # patches that end inside the grid's last rows and columns
    (1, 5, 9, 33, 2176, 2),      # patches, two shares, frame groups of two
    (1, 2, 1, 3, 1024, 2),       # a grid smaller than the window
    (1, 7, 30, 12, 1152, 2),     # 18 groups over eight waves
]


def _cfg(B, F, H, W, C, r):
    return CONFIGS["qwen3vl_2b"].scaled(B=B, F=F, H=H, W=W, C=C, r=r, max_offset=min(max(r, 1), 2), sigma=0.5)


@pytest.mark.parametrize("B,F,H,W,C,r", SHAPES)
def test_walking_search(B, F, H, W, C, r):
    import paper_2605_07355_amd as ttf
    cfg = _cfg(B, F, H, W, C, r)
    batch, res = _prepared(cfg, seed=900 + C + r)
    for mode in (-1, 1):
        x, out = run_gpu(batch.x, r, cfg.t[0], speculation=mode)
        compare_with_oracle(batch.x, out, res)
    # the first frame as a fixed anchor, and the rest of the clip as a segment against it: the same tokens
    # meet the same anchor in the same order, so the similarities are the same bits
    _, fixed = run_gpu(batch.x, r, cfg.t[0], anchor=0)
    seg = x[:, 1:].contiguous()
    buf = ttf.TTFBuffers.allocate(B, F - 1, H, W, C, x.dtype, x.device)
    ttf.ttf_compress_segment(seg, x[:, 0].contiguous(), 0, r=r, t=cfg.t[0], buffers=buf)
    torch.cuda.synchronize()
    assert torch.equal(buf.best_sim, fixed.buffers.best_sim[:, 1:])
    assert torch.equal(buf.fuse_map, fixed.buffers.fuse_map[:, 1:])


@pytest.mark.parametrize("B,F,H,W,C,r", [(2, 5, 9, 19, 1024, 1), (3, 4, 6, 13, 2112, 2), (2, 4, 5, 33, 1024, 0)])
def test_walking_search_tied(B, F, H, W, C, r):
    cfg = _cfg(B, F, H, W, C, r)
    batch, res = _tied_case(cfg, cfg.t[0])
    _compare_tied(batch.x, _run_tied(batch.x, r, cfg.t[0]), res)
