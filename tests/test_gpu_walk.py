"""GPU parity of the search whose workgroups walk whole frames (bf16, C >= 1024: grids that are not whole 16-
or 32-wide tiles take it at every size; fp32): the ends of its column strips, patches and channel shares, as a
pass (on both anchor routes where the guess is available), as a segment and as a tied batch.  Most problems this small
are dealt one frame to a workgroup; several frames a workgroup, asserted, are in test_gpu_walk_plans.py."""
import numpy as np
import pytest
import torch

from workloads import CONFIGS, make_clip_batch

from helpers import compare_with_oracle, run_gpu
from test_gpu_next import _compare_tied, _run_tied, _tied_case
from test_gpu_parity import _prepared
from test_gpu_speculative import TRUST_GAP, _with_foreign_guess_channels, anchor_scores, guess_channels

pytestmark = pytest.mark.gpu

SHAPES = [
    # B, F,  H,  W,  C,    r
    (1, 4, 5, 17, 1024, 1),      # two strips, eight and nine cells wide
    (2, 5, 3, 30, 1088, 1),      # three strips; 17 groups of 64 channels over eight waves
    (1, 3, 1, 16, 2112, 0),      # one grid row; two shares of the channels, 66 K-steps
    (1, 36, 2, 14, 1024, 1),     # many frames of two rows; also beside a guess
    (1, 6, 10, 18, 4160, 1),     # three shares
    (1, 9, 7, 40, 1024, 0),      # three strips without a margin
    (2, 3, 6, 13, 1024, 2),      # patches that end inside the grid's last rows and columns
    (1, 5, 9, 33, 2176, 2),      # patches, two shares
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


F32_SHAPES = [
    # B, F,  H,  W,  C,    r   (enough work for the matrix cores, see ttf_search_route)
    (4, 18, 16, 16, 1024, 1),    # a whole tile per row
    (5, 13, 14, 14, 1056, 1),    # 33 groups of 32 channels over two shares
    (6, 9, 9, 31, 1024, 0),      # two strips, 1x1 window
    (3, 8, 16, 32, 2048, 1),     # three strips
    (6, 9, 5, 17, 3104, 1),      # two strips of eight and nine cells, four shares
    (1, 33, 16, 16, 1024, 1),    # 33 MiB in too few strips for the other matrix-core search
]


@pytest.mark.parametrize("B,F,H,W,C,r", F32_SHAPES)
def test_walking_search_fp32(B, F, H, W, C, r):
    import paper_2605_07355_amd as ttf
    assert ttf.ttf_search_route(B, F, H, W, C, torch.float32, r=r) == "mfma_f32"
    cfg = _cfg(B, F, H, W, C, r).scaled(dtype="f32")
    batch, res = _prepared(cfg, seed=950 + C + r)
    for mode in (-1, 1):
        x, out = run_gpu(batch.x, r, cfg.t[0], speculation=mode)
        compare_with_oracle(batch.x, out, res)
    _, fixed = run_gpu(batch.x, r, cfg.t[0], anchor=0)
    buf = ttf.TTFBuffers.allocate(B, F - 1, H, W, C, x.dtype, x.device)
    ttf.ttf_compress_segment(x[:, 1:].contiguous(), x[:, 0].contiguous(), 0, r=r, t=cfg.t[0], buffers=buf)
    torch.cuda.synchronize()
    assert torch.equal(buf.best_sim, fixed.buffers.best_sim[:, 1:])


def test_fp32_guesses_of_all_kinds():
    """fp32 clips whose guess holds, whose trusted guess is wrong, and that have no clear guess, in one batch."""
    from oracle import margins
    cfg = CONFIGS["qwen3vl_2b"].scaled(B=4, F=10, C=1024, dtype="f32")
    batch = _with_foreign_guess_channels(cfg, seed=4300)
    flat = make_clip_batch(cfg.scaled(clean_sigma=1.0), seed=4300)
    batch.x[2] = flat.x[2]
    batch.amplitude[2], batch.changed[2], batch.offsets[2] = flat.amplitude[2], flat.changed[2], flat.offsets[2]
    res = margins.enforce_margins(batch, cfg.r, cfg.t, want_tokens=False)
    kinds = []
    for b in range(cfg.B):
        score = anchor_scores(batch.x[b].reshape(cfg.F, -1, cfg.C)[:, :, guess_channels(cfg.C)].sum(1, dtype=np.float64))
        best, second = np.argsort(-score, kind="stable")[:2]
        kinds.append("fallback" if score[best] - score[second] < TRUST_GAP
                     else ("confirmed" if best == res.anchor_index[b] else "refuted"))
    assert kinds == ["refuted", "confirmed", "fallback", "confirmed"]
    for mode in (1, -1):
        _, out = run_gpu(batch.x, cfg.r, cfg.t[0], speculation=mode)
        compare_with_oracle(batch.x, out, res)
