"""The contour kernels at the ends of their tiles and words, bit for bit against
the CPU oracle: frames around 64-pixel words, 64 x 16 tiles, one to a few rows,
odd sizes, box radii around the unrolled one, and busy scenes whose weak chains
cross tiles; the launch count equals the host model of the tiled growth."""
import numpy as np
import pytest

import oracle
from gpu_util import dev, host
from test_gpu_contour import _launch_model

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H", [(2, 2), (3, 5), (63, 17), (64, 16), (65, 15), (66, 18), (68, 33),
                                 (127, 66), (129, 64), (257, 97), (131, 7)])
@pytest.mark.parametrize("R", [0, 1, 2, 3])
def test_contour_sizes(W, H, R):
    from paper_2203_02300_amd import ContourFilter
    rng = np.random.default_rng(W * 100 + H + R)
    rgb = rng.integers(0, 256, (H, W, 3), dtype=np.uint8)
    # smooth it a little: gradients of all sizes and directions
    s = rgb.astype(np.int32)
    rgb = ((s + np.roll(s, 1, 0) + np.roll(s, 1, 1) + np.roll(s, (1, 1), (0, 1))) // 4)
    rgb = rgb.astype(np.uint8)
    past = rng.normal(0, 2, (H // 2, W // 2, 2)).astype(np.float32)
    future = rng.normal(0, 2, (H // 2, W // 2, 2)).astype(np.float32)
    kw = dict(Thigh=0.75, Tlow=0.2, Tdepth=0.1)
    print(f"contour {W}x{H} R={R}", flush=True)
    want_B, want_MI, want_Mn = oracle.depth_contour(rgb, past, future, R=R, **kw)
    with ContourFilter(W, H, box_radius=R, T_high=0.75, T_low=0.2, T_depth=0.1) as f:
        for _ in range(2):
            B, MI, Mn = f.run(dev(rgb), dev(past), dev(future))
            n = f.launches()
            assert np.array_equal(host(Mn).view(np.uint32), want_Mn.view(np.uint32))
            assert np.array_equal(host(MI).view(np.uint32), want_MI.view(np.uint32))
            assert np.array_equal(host(B), want_B)
    grey = oracle.grey(rgb)
    strong, _ = oracle.contour(grey, want_Mn, Thigh=0.75, Tlow=0.75, Tdepth=0.1)
    # every candidate: none is dropped when the low threshold decides alone
    cand, _ = oracle.contour(grey, want_Mn, Thigh=0.2, Tlow=0.2, Tdepth=0.1)
    assert n == _launch_model(cand.astype(np.uint8) + strong.astype(np.uint8))
