"""What the soft path's fixed-point row sums keep of their FP32 values.

Costs: where every cost in reach is far below the largest that theta allows, the
log-sum-exp shows A2 / T itself.  Its FP32 roundings are counted one by one (units
of 2^-24): the table's x, x / lambda, expm1 (2), alpha, the product, E1, the column
sum and its quotient, E2, A2's sum, reciprocal (2) and product, 1 / T and the last
product: 16, and 4 for log sum exp.

Gradients: each component against the sum of the magnitudes of its own terms, so a
component far below the largest one is held too.  1e-4 of it, as for the benchmark
batch in test_gpu_soft.py: about 16 roundings per factor of a term, the softmax's
exponent (|A2 / T| 2^-24, A2 / T up to 100 here) and expf's argument (x / lambda up
to 40) stay below 1e-5 together.
"""
import numpy as np
import pytest

import oracle
from gpu_util import dev, host
from paper_2203_02300_amd import synth

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


def codes(L, R):
    return oracle.census(oracle.grey(L)), oracle.census(oracle.grey(R)), oracle.arms(L)


@pytest.mark.parametrize("la,lc", [
    (10.0, 30.0),
    (2000.0, 3000.0),
    (1e5, 2.0),      # the colour term is 2^-22 of what the census term may be
    (-1.0, 30.0),    # costs without a finite bound, none of which occurs
])
def test_small_costs_keep_their_bits(la, lc):
    """Flat views that differ by one level in one channel: equal small costs."""
    import torch
    from paper_2203_02300_amd import StereoMatcher
    from paper_2203_02300_amd.soft import soft_forward
    W, H, D = 160, 40, 4
    L = np.full((H, W, 3), 100, np.uint8)
    R = L.copy()
    R[..., 0] += 1
    cost = abs(np.expm1(-1.0 / (3.0 * la)))
    theta = np.float32([la, lc, cost / 300.0])
    _, A2 = oracle.soft_forward(L, R, *codes(L, R), D, lam_ad=float(theta[0]),
                                lam_c=float(theta[1]), T=float(theta[2]), want_volume=True)
    e = -A2 / float(theta[2])
    want = e.max(0) + np.log(np.exp(e - e.max(0)).sum(0))
    with StereoMatcher(W, H, D) as m:
        _, lse = soft_forward(m, dev(L[None]), dev(R[None]), torch.tensor(theta, device="cuda"))
        lse = host(lse)[0].astype(np.float64)
    x = slice(2 * 17 + D, None)  # no partner outside the image in reach
    scale = np.abs(e).max(0)[:, x]
    assert 5 < scale.min() and scale.max() < 300
    assert np.all(np.abs(lse - want)[:, x] <= 20 * U * (scale + np.log(D)))


def grad(pairs, D, theta, gd):
    """Gradient of the batch, the oracle's, and its terms' magnitudes."""
    import torch
    from paper_2203_02300_amd import StereoMatcher
    from paper_2203_02300_amd.soft import soft_backward, soft_forward
    H, W = pairs[0][0].shape[:2]
    th = torch.tensor(theta, dtype=torch.float32, device="cuda")
    with StereoMatcher(W, H, D) as m:
        L, R = (dev(np.stack([p[k] for p in pairs])) for k in (0, 1))
        dh, lse = soft_forward(m, L, R, th)
        g = host(soft_backward(m, L, R, th, dh, lse, dev(gd), reuse=True)).astype(np.float64)
    la, lc, T = (float(v) for v in np.float32(theta))
    want, mag = np.zeros(3), np.zeros(3)
    for b, (Lb, Rb) in enumerate(pairs):
        args = (Lb, Rb, *codes(Lb, Rb), D, gd[b])
        want += oracle.soft_grad(*args, lam_ad=la, lam_c=lc, T=T)
        mag += oracle.soft_grad_mag(*args, lam_ad=la, lam_c=lc, T=T)
    return g, want, mag


@pytest.mark.parametrize("W,H,D,B,theta", [
    (97, 7, 33, 1, (10.0, 30.0, 0.5)),
    (130, 7, 65, 1, (10.0, 30.0, 0.5)),
    (333, 7, 20, 2, (10.0, 30.0, 0.5)),
    (128, 7, 24, 1, (2000.0, 3000.0, 0.01)),
    (128, 7, 24, 1, (0.7, 0.9, 0.5)),
    (128, 7, 24, 1, (4.0, 500.0, 0.1)),
    (1000, 35, 49, 1, (10.0, 30.0, 0.5)),
])
def test_each_gradient_component(W, H, D, B, theta):
    ps = [synth.make_slanted_pair(W, H, D, 900 + i, n_planes=2, dmin=2.0, dmax=D - 3.0,
                                  noise_sigma=2.0, occl_strip_frac=0.03) for i in range(B)]
    gd = np.random.default_rng(W * D).normal(0, 1e-3, (B, H, W)).astype(np.float32)
    g, want, mag = grad([(p["left"], p["right"]) for p in ps], D, theta, gd)
    assert np.all(np.abs(g - want) <= 1e-4 * mag), (g, want, mag)


@pytest.mark.parametrize("theta", [(5.0, 2.0, 0.5), (5.0, 1.0, 0.5), (3.0, 3.0, 0.5)])
def test_gradient_of_poor_matches(theta):
    """Views that slope opposite ways: census distances of 31 to 56 and lambdas far
    below them, so derivatives of 2^-20 to 2^-70 of the largest that the tables
    hold.  Only inner pixels count (border windows repeat pixels)."""
    W, H, D = 150, 40, 20
    x, y = np.arange(W)[None], np.arange(H)[:, None]
    steps = 12 * ((x + y) // 6 % 2) * (x // 11 % 2)
    L, R = (np.repeat(v[..., None], 3, 2).astype(np.uint8) for v in (x + 0 * y, 245 - x + steps))
    gd = np.zeros((1, H, W), np.float32)
    gd[0, 15:25, 70:80] = np.random.default_rng(5).normal(0, 1.0, (10, 10))
    g, want, mag = grad([(L, R)], D, theta, gd)
    assert np.all(np.abs(g - want) <= 1e-4 * mag), (g, want, mag)


def test_gradients_that_grow_along_the_rows():
    """2^9 per block of 64 columns (each block rescales the fixed point), both ways."""
    W, H, D = 300, 9, 20
    p = synth.make_slanted_pair(W, H, D, 960, n_planes=2, dmin=2.0, dmax=D - 3.0,
                                noise_sigma=2.0, occl_strip_frac=0.03)
    base = np.random.default_rng(3).normal(0, 1e-3, (1, H, W))
    for e in (np.arange(W) / 7.0, -np.arange(W) / 7.0, np.abs(np.arange(W) - 150) / -7.0):
        gd = (base * 2.0 ** e).astype(np.float32)
        g, want, mag = grad([(p["left"], p["right"])], D, (10.0, 30.0, 0.5), gd)
        assert np.all(np.abs(g - want) <= 1e-4 * mag), (g, want, mag)
