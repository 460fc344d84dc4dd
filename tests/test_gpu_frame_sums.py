"""Frame sums of the anchor rule: their rate on inputs whose rows are not whole 4 KiB slabs, and where
frames are summed in runs of rows."""
import statistics

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
    (1, 86, 32, 32, 1536, torch.bfloat16, False),       # 258 blocks: with two runs more than two a CU
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
