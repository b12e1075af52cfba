"""The row kernel of the winner-take-all and the left-right check at the ends of
its quads and threads, bit for bit against the CPU oracle: rows of less than
four columns, a ragged last quad, one to several turns of a workgroup, ranges
around one batch of loads, volumes at any 4-byte alignment."""
import numpy as np
import pytest

import oracle
from gpu_util import dev, host

pytestmark = pytest.mark.gpu

SHAPES = [(2, 1, 1), (2, 3, 1), (3, 2, 2), (4, 3, 3), (5, 4, 4), (6, 3, 5), (9, 5, 8),
          (63, 4, 21), (65, 3, 43), (1023, 2, 44), (1025, 3, 45), (2049, 2, 17), (4099, 1, 9)]


@pytest.mark.parametrize("offset", [0, 1, 3])
@pytest.mark.parametrize("W,H,D", SHAPES)
def test_staged_volumes(W, H, D, offset):
    import torch
    from paper_2203_02300_amd import StereoMatcher
    rng = np.random.default_rng(W + 7 * H + D)
    vols = [rng.integers(0, 6, (D, H, W)).astype(np.float32) / 4 for _ in range(2)]  # many ties
    dl, del_l = oracle.wta(vols[0])
    dr, _ = oracle.wta(vols[1])
    disp, valid = oracle.lrcheck(dl, del_l, dr, maxdiff=1)
    on = []
    for v in vols:
        buf = torch.empty(v.size + 4, dtype=torch.float32, device="cuda")
        t = buf[offset:offset + v.size].view(D, H, W)
        t.copy_(dev(v))
        on.append(t)
    print(f"staged WTA {W}x{H} D={D} offset={offset}", flush=True)
    with StereoMatcher(W, H, D, census_w=1, census_h=1, lr_max_diff=1) as m:
        got = m.wta_lrcheck(*on)
    for g, w in zip(got, (disp, valid, dl, dr)):
        assert np.array_equal(host(g), w)


@pytest.mark.parametrize("iters", [1, 2])
@pytest.mark.parametrize("W,H,D", SHAPES)
def test_one_call(W, H, D, iters):
    from paper_2203_02300_amd import StereoMatcher
    rng = np.random.default_rng(W * 31 + H + D)
    L = rng.integers(0, 256, (H, W, 3), dtype=np.uint8)
    R = np.ascontiguousarray(np.roll(L, -(D // 2), axis=1))
    R[::2] ^= 3
    st = oracle.stages(L, R, D, cw=1, ch=1, iters=iters)
    print(f"one call {W}x{H} D={D} iters={iters}", flush=True)
    with StereoMatcher(W, H, D, census_w=1, census_h=1, agg_iters=iters) as m:
        disp, valid = m.match(dev(L), dev(R))
        dL, dR = m.last_disparities()
    for g, w in zip((disp, valid, dL, dR), (st["disp"], st["valid"], st["dL"], st["dR"])):
        assert np.array_equal(host(g), w)
