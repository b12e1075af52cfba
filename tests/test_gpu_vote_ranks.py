"""The region vote's windows over the disparities that occur, against the CPU
oracle, bit for bit: fewer, as many and more of them than a window holds, ranges
of one word, of one per lane and above (the scan in LDS), and frames around the
16 x 30 tiles."""
import numpy as np
import pytest

import oracle
from gpu_util import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H,D,values", [
    (65, 30, 20, 3), (64, 31, 33, 14), (79, 29, 64, 15), (97, 61, 90, 90), (130, 33, 128, 29),
    (330, 45, 300, 300), (2060, 20, 2048, 600), (2200, 33, 2100, 1500),
])
def test_vote_windows(W, H, D, values):
    import torch
    from paper_2203_02300_amd import StereoMatcher
    rng = np.random.default_rng(W + D)
    img = rng.integers(0, 256, (H, W // 9 + 1, 3), dtype=np.uint8)
    img = np.ascontiguousarray(np.repeat(img, 9, axis=1)[:, :W])
    img[::3] = img[0]
    arms = oracle.arms(img)
    some = np.sort(rng.choice(D, values, replace=False))
    some[-1] = D - 1
    base = some[(np.arange(W)[None] // 11 + np.arange(H)[:, None] // 7) % values]
    noise = some[rng.integers(0, values, (H, W))]
    dL = np.where(rng.random((H, W)) < 0.6, base, noise).astype(np.int16)
    valid = (rng.random((H, W)) < 0.8).astype(np.uint8)
    print(f"vote {W}x{H} D={D} values={values}", flush=True)
    agg = torch.zeros((D, H, W), dtype=torch.float32, device="cuda")
    with StereoMatcher(W, H, D) as m:
        for iters in (1, 2, 3):
            disp, ok, dv = m.vote_refine(dev(arms), agg, dev(dL), dev(valid), iters)
            want = oracle.vote(dL, valid, arms, D, iters)
            assert np.array_equal(host(dv), want), iters
            assert np.array_equal(host(ok), (want >= 0).astype(np.uint8))
            assert np.array_equal(host(disp), np.maximum(want, 0).astype(np.float32))
