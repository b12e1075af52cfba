"""The two-stage aggregation kernel at the edges of its strips, quads, chunks
and row bands, against the CPU oracle, bit for bit: both aggregated volumes
and the maps of the one-call match, and the staged aggregation."""
import numpy as np
import pytest

import oracle
from gpu_util import dev, host

pytestmark = pytest.mark.gpu

# inner strips are 184 output columns (aprons of 36), the first and the last
# 20 more, a lone one 224; lanes own aligned quads of columns, rows go in
# chunks of four, rings hold 36 rows; small frames are split into a top and a
# bottom half
SHAPES = [
    (9, 7, 3),        # the smallest frame: one quad and one column
    (184, 37, 5),     # one strip, an odd range (a lone last slice)
    (223, 36, 4),     # one strip, its last column missing
    (224, 35, 1),     # one strip exactly, one slice only
    (225, 34, 7),     # two strips, the second of 21 columns
    (226, 8, 2),
    (407, 33, 8),     # two strips, the last column missing
    (408, 71, 6),     # two strips exactly
    (409, 38, 3),     # three strips
    (592, 70, 16),    # three strips exactly
    (593, 39, 2),
    (410, 37, 3),     # the border cuts a quad of the second strip's apron too
    (411, 21, 5),
    (10, 9, 4),
    (11, 8, 5),
]


def scene(W, H, D):
    """Piecewise-constant colours (arms up to the limit), shifted by D / 2,
    with a few noisy rows so that short arms occur too."""
    from paper_2203_02300_amd import synth
    rng = np.random.default_rng(W * 1000 + H)
    L = synth.make_patchwork(W, H, seed=W + H, n=max(3, W * H // 600))
    L[::5] = rng.integers(0, 256, L[::5].shape, dtype=np.uint8)
    R = np.roll(L, -(D // 2), axis=1)
    return np.ascontiguousarray(L), np.ascontiguousarray(R)


@pytest.mark.parametrize("W,H,D", SHAPES)
def test_one_call_volumes_and_maps(W, H, D):
    from paper_2203_02300_amd import StereoMatcher
    L, R = scene(W, H, D)
    st = oracle.stages(L, R, D)
    print(f"one call {W}x{H} D={D}", flush=True)
    with StereoMatcher(W, H, D) as m:
        disp, valid = m.match(dev(L), dev(R))
        for view, tag in ((0, "L"), (1, "R")):
            got = host(m.agg_slices(view))
            assert np.array_equal(got.view(np.uint32), st["agg" + tag].view(np.uint32)), tag
        assert np.array_equal(host(valid), st["valid"])
        assert np.array_equal(host(disp).view(np.uint32), st["disp"].view(np.uint32))


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("W,H,D", [(184, 37, 5), (225, 34, 7), (408, 71, 6), (226, 20, 3),
                                   (227, 19, 4), (411, 21, 5), (3, 5, 2), (2, 4, 1)])
def test_staged_aggregation_any_alignment(W, H, D, offset):
    """Volumes that start `offset` floats into their buffers, rows of any length:
    only 4-byte aligned, with a last quad of one to four columns (words where a
    row has less than four)."""
    import torch
    from paper_2203_02300_amd import StereoMatcher
    L, R = scene(W, H, D)
    cw = 9 if W >= 9 and H >= 7 else 1
    st = oracle.stages(L, R, D, cw=cw, ch=min(cw, 7))
    n = D * H * W
    print(f"staged {W}x{H} D={D} offset {offset}", flush=True)
    with StereoMatcher(W, H, D, census_w=cw, census_h=min(cw, 7)) as m:
        for tag in ("L", "R"):
            q = (st["q" + tag].astype(np.float64) * 2.0 ** -20).astype(np.float32)
            cost = torch.zeros(n + offset, device="cuda")
            cost[offset:] = dev(q).reshape(-1)
            out = torch.zeros(n + offset, device="cuda")
            agg = m.aggregate(cost[offset:].view(D, H, W), dev(st["arms" + tag]),
                              out=out[offset:].view(D, H, W))
            assert np.array_equal(host(agg).view(np.uint32), st["agg" + tag].view(np.uint32)), tag
            assert offset == 0 or float(out[0]) == 0.0
