"""The one-launch densification solve at the edges of its tiles (32 x 32 k
pixels, k = 1 .. 4 pixels per thread) against the oracle's direct FP64 solve,
with the bound of tests/test_gpu_densify.py: a solution of relative residual
1e-9 within 1e-5 of the largest depth."""
import numpy as np
import pytest

from gpu_util import dev, host
from oracle import densify as dz

pytestmark = pytest.mark.gpu

# W, H: a tile less a row and a column, exactly one, one more of each; tiles
# of two, three and four rows of 32 (wide grids take taller tiles)
SHAPES = [(31, 31), (32, 32), (33, 33), (257, 65), (640, 97), (1024, 130), (1279, 129)]


def inputs(W, H, seed):
    """Depth on a few pixels, smooth maps, a contour of random lines."""
    rng = np.random.default_rng(seed)
    depth = 5 + 3 * np.sin(np.arange(W) / 17.0)[None] + np.cos(np.arange(H) / 11.0)[:, None]
    Ds = np.where(rng.random((H, W)) < 0.5, depth, 0).astype(np.float32)
    Dpre = np.where(rng.random((H, W)) < 0.3, depth * 1.01, 0).astype(np.float32)
    B = np.zeros((H, W), np.uint8)
    B[rng.integers(0, H, 3)] = 1
    B[:, rng.integers(0, W, 3)] = 1
    Mf, MI = (rng.random((H, W)).astype(np.float32) for _ in range(2))
    return Ds, Dpre, B, Mf, MI


@pytest.mark.parametrize("W,H", SHAPES)
def test_tile_edges(W, H):
    from paper_2203_02300_amd import Densifier
    Ds, Dpre, B, Mf, MI = inputs(W, H, W + H)
    want = dz.densify(Ds, Dpre, B, Mf, MI)
    print(f"densify tiles {W}x{H}", flush=True)
    with Densifier(W, H) as z:
        D = host(z.run(dev(Ds), dev(B), dev(Mf), dev(MI), Dpre=dev(Dpre)))
        it, rel = z.stats()
    assert rel <= 1e-9 and 0 < it < 400
    assert np.abs(D - want).max() <= 1e-5 * np.abs(want).max()


def test_solves_on_two_streams_and_threads():
    """Solves of different sizes at the same time give what each gives alone."""
    import threading
    import torch
    from paper_2203_02300_amd import Densifier
    sizes = [(640, 97), (200, 120)]
    alone, both = [None] * 2, [[] for _ in sizes]
    args = [[dev(a) for a in inputs(W, H, 9)] for W, H in sizes]

    def solve(k, out, reps):
        with torch.cuda.stream(torch.cuda.Stream()):
            with Densifier(*sizes[k]) as z:
                Ds, Dpre, B, Mf, MI = args[k]
                for _ in range(reps):
                    out.append(host(z.run(Ds, B, Mf, MI, Dpre=Dpre)))

    torch.cuda.synchronize()
    for k in range(2):
        got = []
        solve(k, got, 1)
        alone[k] = got[0]
    ts = [threading.Thread(target=solve, args=(k, both[k], 3)) for k in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for k in range(2):
        assert len(both[k]) == 3
        for D in both[k]:
            assert np.array_equal(D.view(np.uint32), alone[k].view(np.uint32))


def test_abandoned_solve_falls_back(monkeypatch):
    """A wait bound of zero makes the workgroups give the one-launch solve up
    at the first word that is not there yet; the solve is then repeated as a
    sequence of launches and gives the same depths within the tolerance."""
    from paper_2203_02300_amd import Densifier
    W, H = 200, 120
    Ds, Dpre, B, Mf, MI = inputs(W, H, 3)
    want = dz.densify(Ds, Dpre, B, Mf, MI)
    monkeypatch.setenv("DCO_DENSIFY_WAIT", "0")
    with Densifier(W, H) as z:
        D = host(z.run(dev(Ds), dev(B), dev(Mf), dev(MI), Dpre=dev(Dpre)))
        it, rel = z.stats()
    assert rel <= 1e-9 and 0 < it < 400
    assert np.abs(D - want).max() <= 1e-5 * np.abs(want).max()


def test_largest_one_launch_grid_and_beyond():
    """1280 x 768 takes the tallest tiles on 256 CUs, 1312 x 832 the sequence
    of launches: constant data on a few pixels gives a constant depth."""
    from paper_2203_02300_amd import Densifier
    for W, H in ((1280, 768), (1312, 832)):
        Ds = np.zeros((H, W), np.float32)
        Ds[::7, ::5] = 2.5
        zero = np.zeros((H, W), np.float32)
        with Densifier(W, H) as z:
            D = host(z.run(dev(Ds), dev(zero.astype(np.uint8)), dev(zero), dev(zero)))
        assert np.allclose(D, 2.5, rtol=1e-6), (W, H)
