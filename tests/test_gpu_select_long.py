"""GPU parity of the threshold selection around the sizes where its forms change: clips of one round of loads
(8192 values) and more, keys listed once at most 8192 match, and fields that never thin out (equal values)."""
import numpy as np
import pytest
import torch

from workloads.ttf_gen import similarity_field

from test_gpu_next import _FakeOut

pytestmark = pytest.mark.gpu


def _check(sim, anchor, H, W, fraction):
    import paper_2605_07355_amd as ttf
    from oracle import adaptive as A
    t = ttf.ttf_select_threshold(_FakeOut(sim, anchor, H, W), fraction)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(t.cpu().numpy(), A.select_threshold(sim, anchor, fraction))


@pytest.mark.parametrize("ties", [False, True])
@pytest.mark.parametrize("fraction", [0.0, 0.33, 0.67, 1.0])
@pytest.mark.parametrize("B,F,H,W", [(2, 32, 16, 16), (2, 33, 16, 16), (3, 65, 12, 21), (1, 5, 128, 26), (2, 90, 32, 17)])
def test_long_clips(B, F, H, W, fraction, ties):
    sim, anchor = similarity_field(B, F, H * W, seed=B * 100 + F, ties=ties)
    _check(sim, anchor, H, W, fraction)
    _check(sim, np.full(B, -1, np.int32), H, W, fraction)


@pytest.mark.parametrize("n_equal", [8191, 8192, 8193, 17000])
def test_values_that_share_their_leading_digits(n_equal):
    """Keys that match after two digits: one fewer than the list holds, as many, one more, and all."""
    rng = np.random.default_rng(n_equal)
    sim = (0.9 + 1e-4 * rng.random(17000)).astype(np.float32)          # one 16-bit prefix or two
    sim[n_equal:] = rng.uniform(-1, 0.2, 17000 - n_equal).astype(np.float32)
    if n_equal == 8193:
        sim[:n_equal] = np.float32(0.9)                               # equal values: no digit thins them out
    sim = rng.permutation(sim).reshape(1, 17, 1000)
    for fraction in (0.1, 0.3, 0.4999, 0.6):
        _check(sim, np.full(1, -1, np.int32), 25, 40, fraction)
        _check(sim, np.full(1, 3, np.int32), 25, 40, fraction)
