"""Host-side: which bf16 rows that end inside a 32-channel K-step are sent to the matrix-core search.  The sizes are
measured ones, with the time of a whole call there over its time on the wave-per-token kernels."""
import pytest
import torch

WAVE_PER_TOKEN = [
    # B,  F,  H,  W,  C,   r
    (1, 49, 16, 1, 4072, 1),      # 1.57: one column of sixteen
    (2, 25, 32, 2, 4072, 1),      # 1.36
    (8, 9, 16, 4, 4072, 1),       # 1.37
    (24, 2, 32, 2, 776, 1),       # 1.87: groups of four frames with one in them
    (24, 2, 24, 2, 776, 2),       # 1.58
    (8, 2, 14, 28, 1512, 1),      # 1.32
    (1, 33, 12, 12, 1000, 1),     # too few workgroups
    (6, 2, 16, 72, 1512, 1),      # 1.69
    (8, 2, 14, 36, 2040, 0),      # 1.28
]
MATRIX_CORES = [
    (3, 23, 24, 18, 1000, 1),     # 0.52
    (3, 33, 20, 4, 1512, 1),      # 0.74
    (48, 9, 1, 12, 3048, 0),      # 0.46
    (24, 5, 8, 16, 776, 2),       # 0.36
    (2, 25, 9, 18, 4072, 1),      # 0.85
    (1, 13, 32, 32, 4072, 0),     # 0.65
    (16, 64, 32, 2, 1000, 1),     # 0.76
    (12, 5, 8, 33, 4072, 1),      # 0.82
    (1, 25, 24, 60, 776, 0),      # 0.38
]


@pytest.mark.parametrize("shapes,there", [(WAVE_PER_TOKEN, False), (MATRIX_CORES, True)])
def test_routes_of_rows_that_end_inside_a_k_step(shapes, there):
    import paper_2605_07355_amd as ttf
    for B, F, H, W, C, r in shapes:
        want = "mfma_bf16_padded" if there else "general"
        assert ttf.ttf_search_route(B, F, H, W, C, torch.bfloat16, r=r) == want, (B, F, H, W, C, r)
