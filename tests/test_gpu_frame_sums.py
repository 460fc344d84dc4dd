"""Frame sums of the anchor rule: their rate on inputs whose rows are not whole 4 KiB slabs, and where
frames are summed in runs of rows."""
import statistics

import numpy as np
import pytest
import torch


def _frame_sums_ms(B, F, H, W, C):
    """Median time of the frame-sum stage over several calls, after warm-up (two-pass route)."""
    import paper_2605_07355_amd as ttf
    x = torch.randn((B, F, H, W, C), device="cuda").to(torch.bfloat16)
    buf = ttf.TTFBuffers.allocate(B, F, H, W, C, x.dtype, x.device)
    ttf.ttf_set_speculation(-1)
    try:
        for _ in range(5):
            ttf.ttf_compress(x, buffers=buf)
        ttf.ttf_profile_enable(25)
        for _ in range(25):
            ttf.ttf_compress(x, buffers=buf)
        torch.cuda.synchronize()
        return statistics.median(ttf.ttf_profile_read(i)["frame_sums"] for i in range(25))
    finally:
        ttf.ttf_profile_enable(0)
        ttf.ttf_set_speculation(0)


@pytest.mark.gpu
@pytest.mark.parametrize("B,F,H,W,C", [(64, 32, 16, 16, 256), (1, 300, 32, 32, 512)])
def test_rows_that_are_not_whole_slabs_are_summed_at_the_slab_rate(B, F, H, W, C):
    """About 256 MiB in blocks of 512 channels against 256 MiB in 4 KiB slabs (B8 F32 16x16 C2048).  Both read
    HBM once: 45 against 43 us.  A body whose loads wait for each other takes 74 and 128 us."""
    slabs = _frame_sums_ms(8, 32, 16, 16, 2048)
    rows = _frame_sums_ms(B, F, H, W, C)
    per_byte = rows / (B * F * H * W * C) * (8 * 32 * 256 * 2048)
    assert per_byte <= 1.35 * slabs, f"{rows * 1e3:.1f} us against {slabs * 1e3:.1f} us for the same bytes in slabs"


@pytest.mark.gpu
@pytest.mark.parametrize("B,F,H,W,C,dtype,parts", [
    (1, 256, 16, 16, 512, torch.bfloat16, False),       # 256 blocks; the fragment copy holds half a share
    (2, 60, 32, 32, 1024, torch.bfloat16, True),        # 240 blocks: two runs of each frame
    (1, 86, 32, 32, 1528, torch.bfloat16, True),        # 258 blocks: two runs, or some CUs had two blocks and most one
    (1, 130, 32, 32, 1528, torch.bfloat16, False),      # 390 blocks
    (9, 34, 32, 32, 320, torch.float32, False),         # 612 blocks (two runs: 82 us, one: 72)
    (1, 32, 6, 10, 2048, torch.bfloat16, False),        # 60 rows: too short for two runs
    (1, 60, 8, 8, 2048, torch.bfloat16, False),         # 240 blocks; the fragment copy holds one share
    (1, 8, 8, 8, 2048, torch.bfloat16, True),           # 64 rows: two runs
])
def test_frames_are_summed_in_runs_only_where_blocks_are_few(B, F, H, W, C, dtype, parts):
    """Sums of whole frames stand at the head of the workspace; shares of frames stand elsewhere and leave it."""
    import paper_2605_07355_amd as ttf
    x = torch.randn((B, F, H, W, C), device="cuda").to(dtype)
    buf = ttf.TTFBuffers.allocate(B, F, H, W, C, dtype, x.device)
    buf.workspace.fill_(0xCD)
    ttf.ttf_compress(x, buffers=buf)
    torch.cuda.synchronize()
    head = -buf.workspace.data_ptr() % 256
    left = (buf.workspace[head:head + B * F * C * 4] == 0xCD).all().item()
    assert left == parts


# ----------------------------------------------------------------- every row decides the anchor
def _balanced(F, N, C, winner, plus, minus, channels):
    """Frames of ones; every frame but the winner carries 8 or -8 more (as many of each) in `channels` at token `plus`,
    the winner 40 more there and 40 less at token `minus`.  Whole sums: the winner's is the mean of all, cosine 1, the
    others' lie off it.  With the row `plus` or `minus` lost or counted twice the winner's is off by 40, the mean
    by 40 / F, and another frame is nearer."""
    x = np.ones((F, N, C), np.float32)
    sign = 1.0
    for k in range(F):
        if k != winner:
            x[k, plus, channels] += 8.0 * sign
            sign = -sign
    x[winner, plus, channels] += 40.0
    x[winner, minus, channels] -= 40.0
    return x


def _anchor(sums):
    """The anchor rule on frame sums [F,C]: lowest index of the largest cosine with the clip's sum."""
    g = sums.sum(0)
    return int(np.argmax((sums @ g) / (np.linalg.norm(sums, axis=1) * np.linalg.norm(g))))


@pytest.mark.parametrize("N,parts", [(432, 3), (256, 4), (261, 8), (100, 2)])
def test_a_run_lost_or_counted_twice_would_show(N, parts):
    """The inputs below, on sums in which one run is left out or doubled: another frame is chosen."""
    F, C, winner = 5, 48, 3
    per = -(-(-(-N // parts)) // 16) * 16
    runs = [(lo, min(N, lo + per)) for lo in range(0, N, per)]
    assert len(runs) > 1
    for i, (lo, hi) in enumerate(runs):
        for plus in (lo, hi - 1):
            minus = (plus + per) % N
            other = [j for j, (a, b) in enumerate(runs) if a <= minus < b][0]
            if other == i:
                minus, other = (plus - per) % N, (i - 1) % len(runs)
            x = _balanced(F, N, C, winner, plus, minus, slice(C - 8, C)).astype(np.float64)
            shares = np.stack([x[:, a:b].sum(1) for a, b in runs], 1)
            assert _anchor(shares.sum(1)) == winner
            for j in (i, other):
                for times in (0.0, 2.0):
                    weight = np.ones(len(runs))
                    weight[j] = times
                    assert _anchor((shares * weight[None, :, None]).sum(1)) != winner


@pytest.mark.gpu
@pytest.mark.parametrize("B,F,H,W,C,dtype", [
    (3, 23, 24, 18, 1000, torch.bfloat16),      # three runs of 144 rows; last slice of channels partly empty
    (1, 33, 16, 16, 2048, torch.bfloat16),      # three runs of 96, 96 and 64 rows
    (1, 9, 9, 29, 1000, torch.bfloat16),        # 261 rows: an odd end
    (1, 41, 16, 16, 512, torch.bfloat16),       # long clip of short rows: the fragment copy holds three shares
    (2, 7, 27, 27, 1152, torch.float32),
    (1, 5, 16, 16, 264, torch.bfloat16),        # wave-per-token search
    (1, 3, 5, 8, 256, torch.bfloat16),          # whole frames
])
def test_every_row_decides_the_anchor(B, F, H, W, C, dtype):
    """The evidence for each clip's anchor lies in two rows, moved over the ends of all runs and of the frame; the
    workspace holds NaN, or the previous call's sums.  Plain pass and tied batch."""
    import paper_2605_07355_amd as ttf
    N = H * W
    buf = ttf.TTFBuffers.allocate(B, F, H, W, C, dtype, "cuda")
    tied = ttf.TTFTiedBuffers.allocate(B, F, H, W, C, dtype, "cuda", r=0)
    edges = sorted({0, 1, N - 1, N - 2} | {q + d for q in range(16, N, 16) for d in (-1, 0)} & set(range(N)))
    channels = (slice(0, C, 2), slice(C - 8, C))
    for n, plus in enumerate(edges):
        minus = (plus + N // 2) % N
        winners = [1 + (n + b) % (F - 1) for b in range(B)]
        x = np.stack([_balanced(F, N, C, w, plus, minus, channels[n % 2]) for w in winners])
        xd = torch.from_numpy(x).view(B, F, H, W, C).to(dtype).cuda()
        if n % 3 == 0:
            buf.workspace.fill_(0xFF)
            tied.workspace.fill_(0xFF)
        ttf.ttf_compress(xd, r=0, buffers=buf)
        same = torch.from_numpy(x[:1]).view(1, F, H, W, C).to(dtype).cuda().expand(B, -1, -1, -1, -1).contiguous()
        ttf.ttf_compress_tied(same, r=0, buffers=tied)
        torch.cuda.synchronize()
        assert buf.anchor_index.tolist() == winners, (plus, minus)
        assert tied.anchor_index.tolist() == [winners[0]] * B, (plus, minus)
