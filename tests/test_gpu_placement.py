"""GPU parity of the row placement at the limits of its forms: everything in one launch (at most 256 keep
words), offsets with the ids (at most 4096, rows of 1 KiB and more), and behind a scan (beyond, or short rows)."""
import statistics

import numpy as np
import pytest
import torch

from workloads import CONFIGS, similarity_field

from helpers import SENTINEL
from test_gpu_next import _compare_segment, _compare_tied, _run_segment, _run_tied, _segment_case, _tied_case
from test_gpu_parity import _parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("anchor", ["auto", 0, -1])
@pytest.mark.parametrize("B,F,H,W,C", [
    (2, 64, 9, 9, 64),       # 256 words: the last that are placed in one launch; ragged words
    (1, 257, 3, 3, 512),     # 257 words of 1 KiB rows: ids with the offsets, one word in the last run
    (3, 86, 2, 3, 504),      # 258 words of rows below 1 KiB: behind the scan
    (7, 5, 9, 17, 512),      # 105 words, clips of 15: runs that end inside a clip do not exist
    (5, 33, 9, 9, 512),      # 330 words, clips of 66: four whole runs and one of two words
    (2, 2048, 1, 2, 512),    # 4096 words: the last without a scan
    (1, 4097, 1, 2, 512),    # 4097 words
    (3, 86, 32, 33, 512),    # 4386 words, 17 a frame, the last one half full: behind the scan, rows of 1 KiB
])
def test_row_placement(B, F, H, W, C, anchor):
    cfg = CONFIGS["qwen3vl_2b"].scaled(B=B, F=F, H=H, W=W, C=C, sigma=0.5)
    if anchor == "auto" and F > 300:
        anchor = F // 2                              # (thousands of frames of one scene: no clear winner to demand)
    _parity(cfg, seed=40 + F, anchor=anchor)


@pytest.mark.parametrize("pieces", [1, 63, 64, 65, 255, 256, 257, 320, 511, 512, 513, 576, 577, 640])
def test_every_end_of_a_row_copied_by_a_wave(pieces):
    """Rows of so many 16-byte pieces: whole rounds of 512, and what is left of at most 64, 256 or 512."""
    _parity(CONFIGS["qwen3vl_2b"].scaled(B=2, F=3, H=3, W=5, C=8 * pieces, sigma=0.5), seed=pieces, anchor=1)


def _regate_us(B, F, H, W, row_bytes):
    """Time of a re-gating call with a third of the tokens kept, from replays of a graph of ten."""
    import paper_2605_07355_amd as ttf
    C = row_bytes // 2
    x = torch.randn((B, F, H, W, C), device="cuda", dtype=torch.bfloat16)
    buf = ttf.TTFBuffers.allocate(B, F, H, W, C, x.dtype, x.device)
    buf.best_sim.copy_(torch.rand((B, F, H * W), generator=torch.Generator().manual_seed(F)))
    buf.best_idx.zero_()
    buf.anchor_index.fill_(F // 2)
    out = ttf.TTFOutput(buf, B, F, H, W, C)
    ttf.ttf_regate(x, out, t=0.33)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for _ in range(10):
            ttf.ttf_regate(x, out, t=0.33)
    times = []
    for _ in range(12):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(3):
            graph.replay()
        e1.record()
        torch.cuda.synchronize()
        times.append(e0.elapsed_time(e1) / 30 * 1e3)
    return statistics.median(times[2:])


@pytest.mark.parametrize("B,F,H,W,row_bytes,times", [
    (64, 4, 4, 4, 8192, 1.7),        # one filled quarter a word: 14 us, 26 where they meet on two XCDs
    (1, 4, 8, 8, 131072, 3.2),       # four words of long rows: 24 us, 52 with a wave per row
])
def test_time_of_unusual_row_sets(B, F, H, W, row_bytes, times):
    """Against 64 whole words of 8 KiB rows, as many bytes (11 us)."""
    plain = _regate_us(1, 64, 8, 8, 8192)
    assert _regate_us(B, F, H, W, row_bytes) <= times * plain


@pytest.mark.parametrize("B,F,H,W,C,one_launch", [
    (1, 49, 16, 4, 2504, True),      # 5008-byte rows
    (1, 49, 16, 4, 3592, True),      # 7184: single pieces at their end
    (1, 8, 8, 8, 4096, True),        # 8 KiB: one whole round a lane
    (1, 8, 8, 8, 5120, True),        # the longest
    (1, 8, 8, 8, 5128, False),
    (1, 8, 8, 8, 8192, False),
    (1, 8, 8, 8, 4097, True),        # no whole 16-byte pieces: a wave a row in every form
])
def test_rows_that_are_placed_by_waves(B, F, H, W, C, one_launch):
    """The list of source rows at the end of the workspace is written by the two-launch form only."""
    import paper_2605_07355_amd as ttf
    x = torch.randn((B, F, H, W, C), device="cuda").to(torch.bfloat16)
    buf = ttf.TTFBuffers.allocate(B, F, H, W, C, x.dtype, x.device)
    buf.workspace.fill_(0xCD)
    ttf.ttf_compress(x, buffers=buf)
    torch.cuda.synchronize()
    head = -buf.workspace.data_ptr() % 256
    end = head + ttf.ttf_workspace_size(B, F, H, W, C, x.dtype)
    size = (B * F * H * W * 4 + 255) // 256 * 256
    assert (buf.workspace[end - size:end] == 0xCD).all().item() == one_launch


def _expected_rows(sim, anchor, t, N):
    """Flat index (over clips and frames) of every output row, and the rows of every clip, at threshold t."""
    rows, counts = [], []
    B, F = sim.shape[:2]
    for b in range(B):
        keep = sim[b] <= t
        first = [] if anchor[b] < 0 else list(anchor[b] * N + np.arange(N))
        if anchor[b] >= 0:
            keep[anchor[b]] = False
        clip = np.concatenate([np.array(first, np.int64), np.flatnonzero(keep.reshape(-1))])
        rows.append(clip + b * F * N)
        counts.append(clip.size)
    return np.concatenate(rows), np.array(counts)


@pytest.mark.parametrize("segment", [False, True])
@pytest.mark.parametrize("B,F,H,W,C", [
    (3, 86, 32, 33, 512),        # 4386 words behind the scan, 17 a frame
    (2, 129, 16, 64, 512),       # 4128 words, 16 a frame, all full
    (64, 65, 3, 5, 520),         # 4160 words of 15 tokens
    (3, 80, 32, 33, 512),        # 4080 words: ids with the offsets
    (5, 51, 9, 7, 500),          # 255 words, 1000-byte rows: one launch
    (16, 5, 13, 15, 1024),       # 320 words, four a frame
])
def test_rows_of_stored_similarities(B, F, H, W, C, segment):
    """Placement alone, behind the re-gating entry point: every output row, id, count and offset, rows past the last
    untouched.  No decision margins are needed: the similarities are given."""
    import paper_2605_07355_amd as ttf
    N, t = H * W, 0.6
    sim, anchor = similarity_field(B, F, N, seed=B + F)
    if segment:
        anchor = np.full(B, -1, np.int32)
    x = torch.randint(-2 ** 15, 2 ** 15, (B, F, H, W, C), dtype=torch.int16, device="cuda",
                      generator=torch.Generator(device="cuda").manual_seed(7)).view(torch.bfloat16)
    buf = ttf.TTFBuffers.allocate(B, F, H, W, C, x.dtype, x.device)
    buf.tokens_out.view(torch.uint8).fill_(0x7A)
    for v in (buf.pos_ids, buf.src_index, buf.row_offsets, buf.kept_count, buf.fuse_map):
        v.fill_(SENTINEL)
    buf.workspace.fill_(0xCD)
    buf.best_sim.copy_(torch.from_numpy(sim))
    buf.best_idx.copy_(torch.arange(N, dtype=torch.int32, device="cuda"))
    buf.anchor_index.copy_(torch.from_numpy(anchor))
    ttf.ttf_regate(x, ttf.TTFOutput(buf, B, F, H, W, C), t=t)
    torch.cuda.synchronize()
    rows, counts = _expected_rows(sim, anchor, np.float32(t), N)
    total = rows.size
    np.testing.assert_array_equal(buf.kept_count.cpu().numpy(), counts)
    np.testing.assert_array_equal(buf.row_offsets.cpu().numpy(), np.concatenate([[0], np.cumsum(counts)]))
    src, pos = buf.src_index.cpu().numpy(), buf.pos_ids.cpu().numpy()
    flat = rows % (F * N)
    np.testing.assert_array_equal(src[:total], flat)
    np.testing.assert_array_equal(pos[:, :total], np.stack([flat // N, flat % N // W, flat % N % W]))
    assert (src[total:] == SENTINEL).all() and (pos[:, total:] == SENTINEL).all()
    want = x.view(torch.int16).view(B * F * N, C)[torch.from_numpy(rows).cuda()]
    assert torch.equal(buf.tokens_out.view(torch.int16)[:total], want)
    assert (buf.tokens_out.view(torch.int16)[total:] == 0x7A7A).all()


@pytest.mark.parametrize("B,F,H,W,C", [
    (2, 260, 32, 33, 512),       # 4420 shared words behind the scan, rows of 1 KiB
    (3, 130, 9, 9, 512),         # 260 words: ids with the offsets
    (3, 127, 9, 9, 64),          # 254: one launch
])
def test_tied_row_placement(B, F, H, W, C):
    cfg = CONFIGS["qwen3vl_2b"].scaled(B=B, F=F, H=H, W=W, C=C, sigma=0.5, shared_motion=True)
    batch, res = _tied_case(cfg, cfg.t[0], F // 2)
    _compare_tied(batch.x, _run_tied(batch.x, cfg.r, cfg.t[0], F // 2), res)
    assert 0 < (res.fuse_map >= 0).mean() < 1


def test_segment_row_placement_behind_the_scan():
    from oracle import streaming as S
    cfg = CONFIGS["qwen3vl_2b"].scaled(B=3, F=87, H=32, W=33, C=512, sigma=0.5)
    batch = _segment_case(cfg, cfg.t[0])
    anchor, seg = batch.x[:, 0], np.ascontiguousarray(batch.x[:, 1:])
    want = S.compress_segment(seg, anchor, cfg.r, cfg.t[0], frame_offset=5)
    _compare_segment(seg, _run_segment(seg, anchor, 5, cfg.r, cfg.t[0]), want)
