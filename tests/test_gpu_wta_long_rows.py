"""WTA and left-right check where they are two launches of quads: rows past 2048
columns, many short rows, few deep ones, and the shapes next to those (one workgroup
per row).  Against a plain scan of the volumes, every element, at rows that end
anywhere within a quad and at workgroups that span several rows."""
import numpy as np
import pytest

from gpu_util import dev, host

pytestmark = pytest.mark.gpu


def plain(aggL, aggR):
    """Eq. 3 and the check in numpy: dL, dR, valid, and the parabola's disparity."""
    D, H, W = aggL.shape
    dL, dR = aggL.argmin(0), aggR.argmin(0)
    x = np.arange(W)[None] - dL
    ok = (x >= 0) & (dL == np.take_along_axis(dR, np.maximum(x, 0), 1))
    at = lambda d: np.take_along_axis(aggL, np.clip(d, 0, D - 1)[None], 0)[0]
    m, c, p = at(dL - 1), at(dL), at(dL + 1)
    den = (m - c) + (p - c)
    with np.errstate(divide="ignore", invalid="ignore"):
        off = np.clip((m - p) / (np.float32(2) * den), np.float32(-0.5), np.float32(0.5))
    off = np.where((dL > 0) & (dL < D - 1) & (den > 0), off, np.float32(0)).astype(np.float32)
    return dL, dR, ok, np.where(ok, dL.astype(np.float32) + off, np.float32(0))


# the longest row of one workgroup, the shortest past it, remainders of 1 to 3 pixels;
# short rows of 4 to 66 columns (33 x 3574: the last before the rule's edge); rows of
# more and of fewer than 192 Ki costs
@pytest.mark.parametrize("W,H,D", [(2047, 4, 9), (2048, 4, 9), (2049, 8, 5), (2052, 3, 64),
                                   (2050, 7, 257), (2081, 2, 1), (3001, 9, 300), (4099, 40, 17),
                                   (8191, 7, 33), (4000, 257, 8), (16383, 7, 60), (2561, 2, 2000),
                                   (4, 3200, 3), (5, 3200, 4), (33, 3574, 7), (33, 3575, 7),
                                   (17, 16384, 6), (66, 4301, 12), (2047, 7, 97), (2047, 7, 96),
                                   (1801, 128, 110), (1801, 129, 110)])
def test_long_rows(W, H, D):
    from paper_2203_02300_amd import StereoMatcher
    rng = np.random.default_rng(W + D)
    # few values, so that equal costs are common and the views agree often
    vol = [rng.integers(1, 5, (D, H, W)).astype(np.float32) for _ in range(2)]
    keep = rng.random((H, W)) < 0.5
    d = rng.integers(0, min(D, 40), (H, 1))
    for v in vol:
        np.put_along_axis(v, np.broadcast_to(d, (H, W))[None], np.where(keep, 0.5, 1.5)[None], 0)
    want = plain(*vol)
    print(f"wta {W}x{H} D={D}", flush=True)
    with StereoMatcher(W, H, D, census_w=1, census_h=1) as m:
        disp, valid, dL, dR = (host(t) for t in m.wta_lrcheck(dev(vol[0]), dev(vol[1])))
    assert np.array_equal(dL, want[0]) and np.array_equal(dR, want[1])
    assert np.array_equal(valid, want[2]) and want[2].any()
    assert np.array_equal(disp.view(np.uint32), want[3].view(np.uint32))


@pytest.mark.parametrize("W,H,D", [(2048, 8, 5), (2049, 8, 5), (2309, 9, 40), (4099, 12, 17),
                                   (34, 3600, 7), (19, 9000, 8), (2046, 19, 98)])
def test_long_rows_of_one_call(W, H, D):
    """The one call (paired volumes) against the staged calls."""
    from paper_2203_02300_amd import StereoMatcher
    rng = np.random.default_rng(W)
    L = np.repeat(rng.integers(0, 256, (H, W // 4 + 1, 3), dtype=np.uint8), 4, 1)[:, :W]
    L = np.ascontiguousarray(L + rng.integers(0, 3, L.shape, dtype=np.uint8))
    R = np.roll(L, -3, axis=1)
    with StereoMatcher(W, H, D) as m:
        one = [host(t) for t in m.match(dev(L), dev(R))]
        staged = [host(t) for t in m.match_staged(dev(L), dev(R))[:2]]
    for a, b in zip(one, staged):
        assert np.array_equal(a.view(np.uint8), b.view(np.uint8))
    assert one[1].any()
