"""GPU parity of the soft path's matrix-core row sums (costs and their gradient)
where their tiling ends: disparity groups of 16 with one or all but one of the
last in use, more groups than a workgroup has wavefronts, rows that are no
multiple of 4, 16 or 64 columns, rows in several parts, blocks left of the
first partner, and thetas whose costs span other ranges of the fixed point.

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


@pytest.mark.parametrize("W,H,D,B,theta", [
    (64, 7, 16, 1, (10.0, 30.0, 0.5)),
    (65, 7, 17, 2, (10.0, 30.0, 0.5)),
    (95, 7, 31, 1, (10.0, 30.0, 0.5)),
    (96, 7, 32, 1, (10.0, 30.0, 0.5)),
    (97, 7, 33, 1, (10.0, 30.0, 0.5)),
    (130, 7, 65, 1, (10.0, 30.0, 0.5)),   # a second round of disparity groups
    (222, 7, 130, 1, (10.0, 30.0, 0.5)),  # a third, of one group
    (333, 7, 20, 2, (10.0, 30.0, 0.5)),   # rows in several parts
    (128, 7, 24, 1, (2000.0, 3000.0, 0.01)),
    (128, 7, 24, 1, (0.7, 0.9, 0.5)),
    (128, 7, 24, 1, (4.0, 500.0, 0.1)),
])
def test_row_sums_match_oracle(W, H, D, B, theta):
    import torch
    from paper_2203_02300_amd import StereoMatcher
    from paper_2203_02300_amd.soft import soft_backward, soft_forward
    ps = [synth.make_slanted_pair(W, H, D, 900 + i, n_planes=2, dmin=2.0, dmax=D - 3.0,
                                  noise_sigma=2.0, occl_strip_frac=0.03) for i in range(B)]
    rng = np.random.default_rng(W * D)
    gd = rng.normal(0, 1e-3, (B, H, W)).astype(np.float32)
    th = torch.tensor(theta, dtype=torch.float32, device="cuda")
    with StereoMatcher(W, H, D) as m:
        L = dev(np.stack([p["left"] for p in ps]))
        R = dev(np.stack([p["right"] for p in ps]))
        dh, lse = soft_forward(m, L, R, th)
        g = host(soft_backward(m, L, R, th, dh, lse, dev(gd), reuse=True)).astype(np.float64)
        dh = host(dh)
    ref = np.zeros(3)
    la, lc, T = (float(v) for v in np.float32(theta))
    for b, p in enumerate(ps):
        Lb, Rb = p["left"], p["right"]
        cL, cR, aL = oracle.census(oracle.grey(Lb)), oracle.census(oracle.grey(Rb)), oracle.arms(Lb)
        want, _ = oracle.soft_forward(Lb, Rb, cL, cR, aL, D, lam_ad=la, lam_c=lc, T=T,
                                      want_volume=True)
        assert np.abs(dh[b] - want).max() < 1e-3
        ref += oracle.soft_grad(Lb, Rb, cL, cR, aL, D, gd[b], lam_ad=la, lam_c=lc, T=T)
    assert np.all(np.abs(g - ref) <= 1e-3 * np.abs(ref).max()), (g, ref)


def test_row_sums_keep_nan_of_theta():
    """lambda = 0 leaves the tables undefined: nothing finite may come out."""
    import torch
    from paper_2203_02300_amd import StereoMatcher
    from paper_2203_02300_amd.soft import soft_forward
    p = synth.make_slanted_pair(96, 8, 16, 950, n_planes=2, dmin=2.0, dmax=13.0,
                                noise_sigma=2.0, occl_strip_frac=0.03)
    with StereoMatcher(96, 8, 16) as m:
        for theta in ((0.0, 30.0, 1.0), (10.0, float("nan"), 1.0)):
            th = torch.tensor(theta, dtype=torch.float32, device="cuda")
            dh, _ = soft_forward(m, dev(p["left"][None]), dev(p["right"][None]), th)
            assert torch.isnan(dh).any()


def test_row_adjoint_follows_growing_gradients():
    """Gradients that grow by 2^9 per block of 64 columns (each block rescales the
    fixed point), and shrink again: as close as ever to the largest component."""
    import torch
    from paper_2203_02300_amd import StereoMatcher
    from paper_2203_02300_amd.soft import soft_backward, soft_forward
    W, H, D = 300, 9, 20
    p = synth.make_slanted_pair(W, H, D, 960, n_planes=2, dmin=2.0, dmax=D - 3.0,
                                noise_sigma=2.0, occl_strip_frac=0.03)
    Lb, Rb = p["left"], p["right"]
    cL, cR, aL = oracle.census(oracle.grey(Lb)), oracle.census(oracle.grey(Rb)), oracle.arms(Lb)
    base = np.random.default_rng(3).normal(0, 1e-3, (1, H, W))
    th = torch.tensor((10.0, 30.0, 0.5), dtype=torch.float32, device="cuda")
    with StereoMatcher(W, H, D) as m:
        L, R = dev(Lb[None]), dev(Rb[None])
        dh, lse = soft_forward(m, L, R, th)
        for e in (np.arange(W) / 7.0, -np.arange(W) / 7.0, np.abs(np.arange(W) - 150) / -7.0):
            gd = (base * 2.0 ** e).astype(np.float32)
            g = host(soft_backward(m, L, R, th, dh, lse, dev(gd), reuse=True)).astype(np.float64)
            ref = oracle.soft_grad(Lb, Rb, cL, cR, aL, D, gd[0], lam_ad=10.0, lam_c=30.0, T=0.5)
            assert np.all(np.abs(g - ref) <= 1e-3 * np.abs(ref).max()), (g, ref)
        gd = base.astype(np.float32)
        for bad in (np.inf, np.nan):
            gd[0, 4, 130] = bad
            g = host(soft_backward(m, L, R, th, dh, lse, dev(gd), reuse=True))
            assert not np.isfinite(g).any()
