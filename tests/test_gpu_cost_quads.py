"""The staged cost volume around the ends of its quads, blocks and chunks of
disparities, in a volume that is only 4-byte aligned, bit for bit against the
CPU oracle; nothing is written before or after the volume."""
import numpy as np
import pytest

import oracle
from gpu_util import dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("W,H,D", [(2, 1, 1), (3, 2, 2), (127, 3, 63), (128, 2, 64), (129, 3, 65),
                                   (130, 2, 7), (131, 2, 72), (259, 3, 131), (76, 4, 75)])
def test_cost_volume(W, H, D, offset):
    import torch
    from paper_2203_02300_amd import StereoMatcher
    rng = np.random.default_rng(W + D)
    L, R = (rng.integers(0, 256, (H, W, 3), dtype=np.uint8) for _ in range(2))
    # any codes and arms that a caller may bring
    cL, cR = (rng.integers(0, 1 << 63, (H, W)).astype(np.uint64) * 2 + 1 for _ in range(2))
    arms = rng.integers(0, 18, (H, W, 4)).astype(np.uint8)
    n = D * H * W
    print(f"cost {W}x{H} D={D} offset {offset}", flush=True)
    with StereoMatcher(W, H, D, census_w=1, census_h=1) as m:
        for ref in (0, 1):
            buf = torch.full((n + offset + 5,), -7.0, device="cuda")
            out = buf[offset:offset + n].view(D, H, W)
            m.cost_volume(ref, dev(L), dev(R), dev(cL.view(np.int64)), dev(cR.view(np.int64)),
                          dev(arms), out=out)
            q = oracle.cost_q(ref, L, R, cL, cR, arms, D)
            want = (q.astype(np.float64) * 2.0 ** -20).astype(np.float32)
            assert np.array_equal(host(out).view(np.uint32), want.view(np.uint32)), ref
            assert (host(buf[:offset]) == -7).all() and (host(buf[offset + n:]) == -7).all()
