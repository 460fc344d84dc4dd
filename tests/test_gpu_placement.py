"""GPU parity of the row placement at the limits of its forms: everything in one launch (at most 256 keep
words), offsets with the ids (at most 4096, rows of 1 KiB and more), and behind a scan (beyond, or short rows)."""
import statistics

import pytest
import torch

from workloads import CONFIGS

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
])
def test_row_placement(B, F, H, W, C, anchor):
    cfg = CONFIGS["qwen3vl_2b"].scaled(B=B, F=F, H=H, W=W, C=C, sigma=0.5)
    if anchor == "auto" and F > 300:
        anchor = F // 2                              # (thousands of frames of one scene: no clear winner to demand)
    _parity(cfg, seed=40 + F, anchor=anchor)


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
    (1, 49, 16, 4, 3592, False),     # 7184: single pieces at their end (regate of 128 words: 17.7 us, by waves 22.9)
    (1, 49, 16, 4, 4072, False),
    (1, 8, 8, 8, 4096, True),        # 8 KiB: one whole round a lane
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
