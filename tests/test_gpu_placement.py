"""GPU parity of the row placement at the limits of its forms: everything in one launch (at most 256 keep
words), offsets with the ids (at most 4096, rows of 1 KiB and more), and behind a scan (beyond, or short rows)."""
import pytest

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
