"""The soft path's large volumes, which are stored past the caches: a batch just
above the line against its pairs one by one, which are below it.

Each run is held to 1e-3 px and 1e-3 of the largest gradient component against
the oracle (test_gpu_soft_rows.py), so two runs are at most 2e-3 apart; a store
that went wrong would show as whole disparities.
"""
import numpy as np
import pytest

from gpu_util import dev, host
from paper_2203_02300_amd import synth

pytestmark = pytest.mark.gpu


# one and several disparity groups per workgroup; a last block of 8 columns
@pytest.mark.parametrize("W,H,D,B", [(328, 113, 63, 8), (1288, 400, 32, 2), (712, 120, 130, 2)])
def test_batch_matches_pairs(W, H, D, B):
    from paper_2203_02300_amd import StereoMatcher
    from paper_2203_02300_amd.soft import soft_backward, soft_forward
    import torch
    assert W % 8 == 0 and W * H * D <= 16 << 20 < B * W * H * D
    ps = [synth.make_slanted_pair(W, H, D, 70 + i, n_planes=2, dmin=2.0, dmax=D - 3.0,
                                  noise_sigma=2.0, occl_strip_frac=0.03) for i in range(B)]
    gd = np.random.default_rng(D).normal(0, 1e-3, (B, H, W)).astype(np.float32)
    th = torch.tensor((10.0, 30.0, 0.5), dtype=torch.float32, device="cuda")
    print(f"soft {B} of {W}x{H} D={D}", flush=True)

    def run(k):
        L, R = (dev(np.stack([ps[i][n] for i in k])) for n in ("left", "right"))
        with StereoMatcher(W, H, D) as m:
            dh, lse = soft_forward(m, L, R, th)
            g = soft_backward(m, L, R, th, dh, lse, dev(gd[k]), reuse=True)
            return host(dh), host(g).astype(np.float64)

    dh, g = run(list(range(B)))
    ref = np.zeros(3)
    for i in range(B):
        dh1, g1 = run([i])
        assert np.abs(dh[i] - dh1[0]).max() < 2e-3
        ref += g1
    assert np.all(np.abs(g - ref) <= 2e-3 * np.abs(ref).max()), (g, ref)
