"""Census codes and arms at the ends of the packed channel test (the smallest and
largest tau1, channels at 0 and 255, one channel deciding alone) and of both
tile heights, bit for bit against the CPU oracle."""
import numpy as np
import pytest

import oracle
from gpu_util import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tau", [1, 2, 20, 128, 255, 256])
@pytest.mark.parametrize("W,H", [(70, 25), (1090, 135)])  # tiles of 8 and of 16 rows
def test_arms_any_tau(W, H, tau):
    from paper_2203_02300_amd import StereoMatcher
    rng = np.random.default_rng(W + tau)
    img = np.empty((H, W, 3), np.uint8)
    lv = np.array([0, 1, tau - 1, min(tau, 255), min(tau + 1, 255), 254, 255], np.uint8)
    for c in range(3):  # steps of exactly tau - 1, tau and tau + 1 in each channel
        img[..., c] = np.repeat(lv[rng.integers(0, len(lv), (H, W // 5 + 1))], 5, axis=1)[:, :W]
    img[H // 2:, : W // 2] = 77
    img[H // 2:, : W // 2, rng.integers(0, 3)] = rng.integers(0, 256, (H - H // 2, W // 2))
    print(f"arms {W}x{H} tau={tau}", flush=True)
    with StereoMatcher(W, H, 8, arm_tau1=tau) as m:
        codes, arms = m.census(dev(img))
    assert np.array_equal(host(arms), oracle.arms(img, tau1=tau))
    assert np.array_equal(host(codes).view(np.uint64), oracle.census(oracle.grey(img)))
