"""GPU parity of the soft path's fused column sums at the sizes where their row
segments, ring turns and column blocks end: fewer rows than one range reaches,
a turn more or less a row, several segments with a ragged last one, and a
last column block of one column.

Tolerances as for the whole soft path (FP32 sums of at most 35 terms per range
and an FP32 softmax, summed in another order by the FP64 oracle): dhat within
1e-3, each gradient component within 1e-3 of the largest one.
"""
import numpy as np
import pytest

import oracle
from gpu_util import dev, host
from paper_2203_02300_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H,D,B", [
    (64, 9, 16, 1),     # every range is clipped at both ends
    (65, 40, 16, 2),    # one turn of rows; a column block of one column
    (97, 41, 16, 1),
    (128, 121, 20, 1),  # more segments than whole turns, ragged
    (72, 203, 16, 1),
    (640, 59, 63, 8),   # planes alone fill the device: one segment
])
def test_column_sums_match_oracle(W, H, D, B):
    import torch
    from paper_2203_02300_amd import StereoMatcher
    from paper_2203_02300_amd.soft import soft_backward, soft_forward
    ps = [synth.make_slanted_pair(W, H, D, 700 + i, n_planes=2, dmin=2.0, dmax=D - 3.0,
                                  noise_sigma=2.0, occl_strip_frac=0.03) for i in range(B)]
    rng = np.random.default_rng(W * H)
    gd = rng.normal(0, 1e-3, (B, H, W)).astype(np.float32)
    theta = torch.tensor([10.0, 30.0, 0.5], dtype=torch.float32, device="cuda")
    with StereoMatcher(W, H, D) as m:
        L = dev(np.stack([p["left"] for p in ps]))
        R = dev(np.stack([p["right"] for p in ps]))
        dh, lse = soft_forward(m, L, R, theta)
        g = host(soft_backward(m, L, R, theta, dh, lse, dev(gd), reuse=True)).astype(np.float64)
        dh = host(dh)
    ref = np.zeros(3)
    for b, p in enumerate(ps):
        Lb, Rb = p["left"], p["right"]
        cL, cR, aL = oracle.census(oracle.grey(Lb)), oracle.census(oracle.grey(Rb)), oracle.arms(Lb)
        want, _ = oracle.soft_forward(Lb, Rb, cL, cR, aL, D, lam_ad=10.0, lam_c=30.0, T=0.5,
                                      want_volume=True)
        assert np.abs(dh[b] - want).max() < 1e-3
        ref += oracle.soft_grad(Lb, Rb, cL, cR, aL, D, gd[b], lam_ad=10.0, lam_c=30.0, T=0.5)
    assert np.all(np.abs(g - ref) <= 1e-3 * np.abs(ref).max()), (g, ref)
