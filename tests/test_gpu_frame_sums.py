"""Frame sums of the anchor rule: their rate on inputs whose rows are not whole 4 KiB slabs."""
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
