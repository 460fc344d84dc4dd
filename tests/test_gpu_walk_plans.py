"""GPU parity of the search that walks whole frames, at deals that are asserted and not assumed: how many runs of rows
and frame groups a problem is cut into is read from the library's own plan."""
import numpy as np
import pytest
import torch

from workloads import CONFIGS, make_clip_batch

from helpers import compare_with_oracle, run_gpu
from plans import matrix_cores, params, search_guesses, search_walks, walk_plan
from test_gpu_nonfinite import test_nonfinite_entries as nonfinite_entries
from test_gpu_parity import _prepared, test_graph_capture_and_replay as graph_capture_and_replay
from test_gpu_speculative import TRUST_GAP, anchor_scores, guess_channels
from workloads.ttf_gen import bf16_bits_to_f32

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


@pytest.mark.parametrize("B,F,H,W,C,r,dtype,ysegs", [
    (1, 16, 9, 9, 1024, 2, "bf16", 3),         # three rows of patches, the last a quarter full
    (1, 10, 17, 9, 1024, 2, "bf16", 5),
    (1, 9, 22, 9, 1088, 2, "bf16", 6),
    (1, 23, 9, 9, 1024, 0, "bf16", 6),         # runs of one and two rows
    (1, 27, 9, 9, 1024, 1, "bf16", 5),
    (1, 53, 9, 9, 1024, 1, "bf16", 3),
    (1, 14, 12, 20, 1024, 1, "f32", 6),
    (2, 34, 9, 9, 1088, 0, "f32", 5),          # three frames a workgroup
])
def test_uneven_runs(B, F, H, W, C, r, dtype, ysegs):
    import paper_2605_07355_amd as ttf
    p = params(B, F, H, W, C, _torch(dtype), r)
    assert search_walks(p) and walk_plan(p, F - 1, False).ysegs == ysegs
    cfg = _cfg(B, F, H, W, C, r, dtype)
    batch, res = _prepared(cfg, seed=1250 + F + H)
    x, out = run_gpu(batch.x, r, cfg.t[0], speculation=-1)
    compare_with_oracle(batch.x, out, res)
    _, whole = run_gpu(batch.x, r, cfg.t[0], anchor=0)
    seg = ttf.TTFBuffers.allocate(B, F - 1, H, W, C, x.dtype, x.device)
    ttf.ttf_compress_segment(x[:, 1:].contiguous(), x[:, 0].contiguous(), 0, r=r, t=cfg.t[0], buffers=seg)
    torch.cuda.synchronize()
    assert torch.equal(seg.best_sim, whole.buffers.best_sim[:, 1:])
    assert torch.equal(seg.fuse_map, whole.buffers.fuse_map[:, 1:])


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
    assert (search_guesses(params(B, F, H, W, C, _torch(dtype), r), 1) >= 0) == guesses
    batch = make_clip_batch(_cfg(B, F, H, W, C, r, dtype), seed=1300 + F)
    first = None
    for mode in (-1, 1, None):
        _, out = run_gpu(batch.x, r, 0.7, speculation=mode)
        b, n = out.buffers, int(out.buffers.row_offsets[-1])
        got = (b.best_sim, b.best_idx, b.fuse_map, b.anchor_index, b.row_offsets, b.src_index[:n])
        first = first or got
        assert all(torch.equal(u, v) for u, v in zip(first, got)), mode


def _guess(clip):
    """Guessed frame of a clip and its lead, from the rule that the header documents."""
    v = clip.reshape(clip.shape[0], -1, clip.shape[-1])[:, :, guess_channels(clip.shape[-1])]
    score = anchor_scores((bf16_bits_to_f32(v) if v.dtype == np.uint16 else v).sum(1, dtype=np.float64))
    best, second = np.argsort(-score, kind="stable")[:2]
    return best, score[best] - score[second]


def _kinds(x, anchors):
    """What becomes of every clip's guess."""
    kinds = []
    for clip, anchor in zip(x, anchors):
        best, gap = _guess(clip)
        assert abs(gap - TRUST_GAP) > 0.005, "guess too close to the trust threshold for a robust test"
        kinds.append("unclear" if gap < TRUST_GAP else ("confirmed" if best == anchor else "refuted"))
    return kinds


def _mixed(cfg, seed, refuted, unclear):
    """A batch of clear clips but for `refuted` (the guess channels are those of a clip with another low-noise frame)
    and `unclear` (no frame stands out); the batch and the oracle's result."""
    from oracle import margins
    batch = make_clip_batch(cfg, seed=seed)
    idx = guess_channels(cfg.C)
    for b in refuted:
        for other_seed in range(seed + 1, seed + 40):
            other = make_clip_batch(cfg.scaled(B=1), seed=other_seed + 100 * b)
            if other.clean_frame[0, 0] != batch.clean_frame[b, 0]:
                batch.x[b][..., idx] = other.x[0][..., idx]
                break
    for b in unclear:
        flat = next(f for f in (make_clip_batch(cfg.scaled(B=1, clean_sigma=1.2), seed=seed + 7000 + b + 1000 * i) for i in range(9))
                    if _guess(f.x[0])[1] < 0.9 * TRUST_GAP)
        batch.x[b] = flat.x[0]
        batch.amplitude[b], batch.changed[b], batch.offsets[b] = flat.amplitude[0], flat.changed[0], flat.offsets[0]
    res = margins.enforce_margins(batch, cfg.r, cfg.t, want_tokens=False)
    want = ["refuted" if b in refuted else ("unclear" if b in unclear else "confirmed") for b in range(cfg.B)]
    return batch, res, want


@pytest.mark.parametrize("B,F,H,W,C,r,dtype,nf,refuted,unclear", [
    (33, 11, 6, 14, 1024, 1, "bf16", 4, (0, 32), (5, 31)),           # more clips than the second walk picks in its prologue
    (70, 10, 2, 14, 1024, 1, "bf16", 4, (0, 34, 69), (1, 35, 65)),   # more than one word of clips; groups of 4, 4 and 2 frames
    (70, 9, 2, 14, 1024, 2, "bf16", 2, (3, 66), (64,)),              # patches; the last group holds one frame
    (70, 10, 3, 25, 1024, 0, "bf16", 4, (69,), (0, 68)),             # two strips
    (40, 25, 6, 14, 1024, 1, "bf16", 3, (), tuple(range(40))),       # no clear guess: the second walk is dealt as without one
    (33, 11, 16, 16, 1024, 1, "bf16", 4, (0, 20), (32,)),            # grids exactly 16 and 32 wide
    (20, 11, 8, 32, 2048, 1, "bf16", 3, (19,), (0, 7)),
    (70, 13, 2, 14, 1024, 1, "f32", 5, (0, 40), (2, 69)),            # groups of 5, 5 and 3
    (70, 23, 2, 14, 1024, 0, "f32", 8, (12, 64), (63,)),             # groups of 8, 8 and 7
])
def test_batches_of_all_kinds(B, F, H, W, C, r, dtype, nf, refuted, unclear):
    p = params(B, F, H, W, C, _torch(dtype), r)
    plan = walk_plan(p, F, True)
    assert search_guesses(p, 1) >= 0 and plan.nf == nf and plan.groups * nf > F
    cfg = CONFIGS["qwen3vl_2b"].scaled(B=B, F=F, H=H, W=W, C=C, r=r, max_offset=min(max(r, 1), 2), sigma=1.2,
                                       clean_sigma=0.1, dtype=dtype)
    batch, res, want = _mixed(cfg, 5000 + B + F, refuted, unclear)
    assert _kinds(batch.x, res.anchor_index) == want
    for mode in (1, -1):
        _, out = run_gpu(batch.x, r, cfg.t[0], speculation=mode)
        compare_with_oracle(batch.x, out, res)


def test_guesses_are_dropped_where_too_few_are_clear():
    """256 MiB at the default setting: with three clips of eight refuted or unclear, the guess is taken for none, or,
    forced, for all that are clear; either way the outputs are those of the two-pass route."""
    B, F, H, W, C, r = 8, 16, 16, 16, 4096, 1
    p = params(B, F, H, W, C, torch.bfloat16, r)
    cfg = CONFIGS["qwen3vl_2b"].scaled(B=B, F=F, H=H, W=W, C=C, r=r, max_offset=1, sigma=1.2, clean_sigma=0.1)
    batch, res, want = _mixed(cfg, 5300, (0,), (2, 5))
    assert _kinds(batch.x, res.anchor_index) == want
    assert search_guesses(p, 0) > B - 2 and search_guesses(p, 1) == 0
    bits = []
    for mode in (None, 1, -1):
        _, out = run_gpu(batch.x, r, cfg.t[0], speculation=mode)
        compare_with_oracle(batch.x, out, res)
        bits.append(out.buffers.best_sim)
    assert torch.equal(bits[0], bits[2]) and torch.equal(bits[1], bits[2])


@pytest.mark.parametrize("B,F,H,W,C,r,dtype", [
    (3, 40, 2, 14, 1024, 1, "bf16"),
    (2, 60, 2, 16, 1024, 2, "bf16"),
    (5, 40, 4, 13, 1056, 1, "f32"),
])
def test_sums_of_one_run_stand_with_the_frame_sums(B, F, H, W, C, r, dtype):
    """Many frames of few tokens, whose sums find no room beside the products; an unclear clip among them."""
    p = params(B, F, H, W, C, _torch(dtype), r)
    plan = walk_plan(p, F, True)
    assert search_guesses(p, 1) == 0 and plan.lsegs * plan.ysegs == 1
    cfg = CONFIGS["qwen3vl_2b"].scaled(B=B, F=F, H=H, W=W, C=C, r=r, max_offset=min(max(r, 1), 2), sigma=1.2,
                                       clean_sigma=0.1, dtype=dtype)
    batch, res, want = _mixed(cfg, 5600 + F, (), (1,))
    assert _kinds(batch.x, res.anchor_index) == want
    for mode in (1, -1):
        _, out = run_gpu(batch.x, r, cfg.t[0], speculation=mode)
        compare_with_oracle(batch.x, out, res)


@pytest.mark.parametrize("B,F,H,W,C,r,dtype,spec", [
    (8, 6, 14, 14, 1056, 1, "f32", None),
    (8, 6, 14, 14, 1056, 0, "f32", 1),
    (6, 5, 9, 31, 1024, 1, "f32", 1),          # two strips
    (2, 5, 9, 33, 2176, 2, "bf16", None),      # patches, two shares
])
@pytest.mark.parametrize("anchor", [1, "auto"])
def test_nonfinite_values_in_the_walk(oracle, B, F, H, W, C, r, dtype, spec, anchor):
    p = params(B, F, H, W, C, _torch(dtype), r)
    assert search_walks(p) and (spec is None or search_guesses(p, spec) == 0)
    nonfinite_entries(oracle, "walk", B, F, H, W, C, dtype, r, spec, anchor)


@pytest.mark.parametrize("B,F,H,W,C,r,dtype,spec", [
    (8, 6, 14, 14, 1056, 1, "f32", 1),
    (70, 10, 2, 14, 1024, 1, "bf16", 1),       # four frames a workgroup, more clips than the second walk picks in its prologue
    (8, 16, 16, 16, 4096, 1, "bf16", None),    # 256 MiB: guesses that may be dropped
])
def test_walk_in_a_graph(B, F, H, W, C, r, dtype, spec):
    assert search_guesses(params(B, F, H, W, C, _torch(dtype), r), spec or 0) >= 0
    graph_capture_and_replay("walk", B, F, H, W, C, dtype, r, spec)


@pytest.mark.parametrize("B,F,H,W,C,r,dtype,unclear", [
    (5, 70, 2, 14, 1024, 1, "bf16", (1,)),
    (5, 70, 2, 14, 1024, 2, "bf16", (0, 1, 2, 3, 4)),   # no guess is left: the second walk picks clip by clip
    (3, 129, 2, 13, 1024, 0, "bf16", ()),
    (4, 67, 3, 13, 1056, 1, "f32", (2,)),
])
def test_guess_of_clips_of_more_frames_than_its_registers_hold(B, F, H, W, C, r, dtype, unclear):
    p = params(B, F, H, W, C, _torch(dtype), r)
    assert F > 64 and search_guesses(p, 1) == 0
    cfg = CONFIGS["qwen3vl_2b"].scaled(B=B, F=F, H=H, W=W, C=C, r=r, max_offset=min(max(r, 1), 2), sigma=1.2,
                                       clean_sigma=0.1, dtype=dtype)
    batch, res, want = _mixed(cfg, 5700 + F, (), unclear)
    assert _kinds(batch.x, res.anchor_index) == want
    for mode in (1, -1):
        _, out = run_gpu(batch.x, r, cfg.t[0], speculation=mode)
        compare_with_oracle(batch.x, out, res)
