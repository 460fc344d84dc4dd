"""GPU parity of bf16 rows that end inside a 32-channel K-step (C % 32 != 0, C % 8 == 0, C >= 768): the
matrix-core search reads their last K-step with the missing 16-byte pieces as zeros.  The same calls on a
workspace without room for that step take the wave-per-token kernels and must agree."""
import numpy as np
import pytest
import torch

from workloads import CONFIGS, make_clip_batch

from helpers import SIM_TOL, compare_with_oracle, run_gpu, to_device
from test_gpu_next import _compare_tied, _run_tied, _tied_case
from test_gpu_parity import _prepared

pytestmark = pytest.mark.gpu

SHAPES = [
    # B, F,  H,  W,  C,    r   (at least 96 workgroups of four frames, 144 on grids wider than 32)
    (3, 33, 14, 14, 776, 1),     # one piece in the last K-step, padding columns
    (2, 26, 16, 16, 1000, 2),    # a 16x16 grid, odd number of passes
    (1, 13, 32, 32, 1016, 0),    # three pieces, 1x1 window on a 32-wide grid
    (1, 13, 34, 31, 888, 1),     # 31 wide, three pieces
    (1, 14, 33, 20, 792, 2),     # 5x5 window on two column tiles (one wave per SIMD)
    (1, 17, 12, 72, 1000, 1),    # wider than 32: a half-empty last strip
    (1, 17, 18, 40, 808, 0),
    (2, 25, 15, 9, 1552, 1),     # two pieces, odd height: the last strip has one real row
]


def _cfg(B, F, H, W, C, r):
    return CONFIGS["qwen3vl_2b"].scaled(B=B, F=F, H=H, W=W, C=C, r=r, max_offset=min(max(r, 1), 2), sigma=0.5)


def _without_tail_room(ttf, buf, sizes):
    """The same workspace, too small for the last K-step (large enough for the rows as they are)."""
    room = ttf.ttf_workspace_size(*sizes, torch.bfloat16) - 256
    skip = -buf.workspace.data_ptr() % 256
    buf.workspace = buf.workspace[:skip + room]


@pytest.mark.parametrize("B,F,H,W,C,r", SHAPES)
def test_rows_that_end_inside_a_k_step(B, F, H, W, C, r):
    import paper_2605_07355_amd as ttf
    assert ttf.ttf_search_route(B, F, H, W, C, torch.bfloat16, r=r) == "mfma_bf16_padded"
    cfg = _cfg(B, F, H, W, C, r)
    batch, res = _prepared(cfg, seed=700 + C + r)
    x, out = run_gpu(batch.x, r, cfg.t[0])
    compare_with_oracle(batch.x, out, res)
    # the whole route as a segment against an external anchor, on both workspaces
    anchor = x[:, 0].contiguous()
    seg = x[:, 1:].contiguous()
    outs = []
    for small in (False, True):
        buf = ttf.TTFBuffers.allocate(B, F - 1, H, W, C, x.dtype, x.device)
        if small:
            _without_tail_room(ttf, buf, (B, F - 1, H, W, C))
        ttf.ttf_compress_segment(seg, anchor, 0, r=r, t=cfg.t[0], buffers=buf)
        outs.append(buf)
    torch.cuda.synchronize()
    assert (outs[0].best_sim - outs[1].best_sim).abs().max().item() <= 2 * SIM_TOL
    near = (outs[1].best_sim - cfg.t[0]).abs() <= 2 * SIM_TOL          # the only tokens that may be gated differently
    assert ((outs[0].fuse_map < 0) == (outs[1].fuse_map < 0))[~near].all()


def test_workspace_without_room_for_the_last_k_step():
    import paper_2605_07355_amd as ttf
    B, F, H, W, C, r = SHAPES[0]
    cfg = _cfg(B, F, H, W, C, r)
    batch, res = _prepared(cfg, seed=31)
    x = to_device(batch.x)
    _, want = run_gpu(batch.x, r, cfg.t[0])
    buf = want.buffers
    _without_tail_room(ttf, buf, (B, F, H, W, C))
    out = ttf.ttf_compress(x, r=r, t=cfg.t[0], buffers=buf)
    torch.cuda.synchronize()
    compare_with_oracle(batch.x, out, res)
    assert C % 8 == 0 and ttf.ttf_search_route(B, F, H, W, C + 4, torch.bfloat16, r=r) == "general"
    assert ttf.ttf_search_route(B, F, H, W, 760, torch.bfloat16, r=r) == "general"
    assert ttf.ttf_search_route(1, 5, H, W, C, torch.bfloat16, r=r) == "general"
    assert ttf.ttf_search_route(1, 17, 12, 72, C, torch.bfloat16, r=2) == "general"


@pytest.mark.parametrize("H,W,C,r", [(14, 14, 776, 1), (24, 20, 1000, 2)])
def test_tied_rows_that_end_inside_a_k_step(H, W, C, r):
    import paper_2605_07355_amd as ttf
    cfg = _cfg(3, 21, H, W, C, r)
    assert ttf.ttf_search_route(cfg.B, cfg.F, H, W, C, torch.bfloat16, r=r) == "mfma_bf16_padded"
    batch, res = _tied_case(cfg, cfg.t[0])
    _compare_tied(batch.x, _run_tied(batch.x, r, cfg.t[0]), res)


def test_non_finite_values_in_the_last_pieces():
    """Infinities, NaN and values whose squares overflow in the row's last piece: as on the wave-per-token
    kernels, and nothing leaks into the neighbouring rows."""
    import paper_2605_07355_amd as ttf
    B, F, H, W, C, r = 2, 26, 16, 16, 1000, 1
    g = torch.Generator().manual_seed(9)
    x = torch.randn((B, F, H, W, C), generator=g).to(torch.bfloat16)
    x[0, 3, 5, 5, C - 1] = float("inf")
    x[0, 4, 2, 7, C - 3] = float("nan")
    x[1, 6, 9, 1, C - 2] = 3e38
    x[1, 7, 0, 0, 0] = -3e38
    x = x.cuda()
    outs = []
    for small in (False, True):
        buf = ttf.TTFBuffers.allocate(B, F, H, W, C, x.dtype, x.device)
        if small:
            _without_tail_room(ttf, buf, (B, F, H, W, C))
        ttf.ttf_compress(x, r=r, t=0.7, anchor=0, buffers=buf)
        outs.append(buf)
    torch.cuda.synchronize()
    a, b = outs[0].best_sim, outs[1].best_sim
    assert torch.equal(torch.isnan(a), torch.isnan(b))
    fin = torch.isfinite(b)
    assert torch.equal(a[~fin & ~torch.isnan(b)], b[~fin & ~torch.isnan(b)]) and (~fin).any()
    assert (a[fin] - b[fin]).abs().max().item() <= 2 * SIM_TOL
    assert torch.equal(outs[0].kept_count, outs[1].kept_count)


@pytest.mark.parametrize("B,F,H,W,C,r", [
    (6, 5, 16, 16, 1000, 1),     # five frames are walked, in two groups of four: 96 workgroups
    (6, 4, 16, 16, 1000, 1),     # four: 48, wave per token
    (4, 9, 14, 18, 776, 0),
])
def test_a_segment_takes_the_search_of_its_clip(B, F, H, W, C, r):
    """A segment is the clip [anchor ; segment] with its anchor fixed to frame 0: the same kernels, the same bits."""
    import paper_2605_07355_amd as ttf
    x = torch.randn((B, F + 1, H, W, C), generator=torch.Generator().manual_seed(C)).to(torch.bfloat16).cuda()
    x[:, 2:] += x[:, :1]
    clip = ttf.ttf_compress(x, r=r, t=0.6, anchor=0).buffers
    seg = ttf.ttf_compress_segment(x[:, 1:].contiguous(), x[:, 0].contiguous(), 0, r=r, t=0.6).buffers
    torch.cuda.synchronize()
    assert torch.equal(seg.best_sim, clip.best_sim[:, 1:])
    assert torch.equal(seg.best_idx, clip.best_idx[:, 1:])
    assert torch.equal(seg.fuse_map, clip.fuse_map[:, 1:])


@pytest.mark.parametrize("C", [776, 4072])
@pytest.mark.parametrize("B,F,H,W,r", [(2, 33, 14, 14, 1), (2, 25, 16, 24, 2), (1, 17, 20, 40, 0)])
def test_similarities_are_as_exact_as_on_the_wave_per_token_kernels(B, F, H, W, r, C):
    """Error against 64 bits of 12 000 similarities and more, each at the token's own cell of the anchor.  Ratio of the
    two: 0.97 at C 776 and 0.85 at C 4072; 1.02 and 0.9 with the anchor's norms summed and inverted in fp32; 1.07 and
    1.1 without the compensation of the folded sums."""
    import paper_2605_07355_amd as ttf
    g = torch.Generator(device="cuda").manual_seed(C)
    a = torch.randn((B, 1, H, W, C), device="cuda", generator=g)
    amp = 0.3 + 1.4 * torch.rand((B, F - 1, H, W, 1), device="cuda", generator=g)
    x = torch.cat([a, a + amp * torch.randn((B, F - 1, H, W, C), device="cuda", generator=g)], 1).to(torch.bfloat16)
    n = x.double().norm(dim=-1)
    exact = ((x[:, 1:].double() * x[:, :1].double()).sum(-1) / (n[:, 1:] * n[:, :1])).flatten(2)
    errors = []
    for small in (False, True):
        buf = ttf.TTFBuffers.allocate(B, F, H, W, C, x.dtype, x.device)
        if small:
            _without_tail_room(ttf, buf, (B, F, H, W, C))
        ttf.ttf_compress(x, r=r, t=0.7, anchor=0, buffers=buf)
        torch.cuda.synchronize()
        own = buf.best_idx[:, 1:] == torch.arange(H * W, device="cuda", dtype=torch.int32)
        assert own.sum().item() > 12000
        errors.append((buf.best_sim[:, 1:].double() - exact)[own].norm().item())
    assert errors[0] <= errors[1]
