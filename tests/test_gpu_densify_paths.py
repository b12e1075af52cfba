"""The two ways a densification solve runs on its tiles: as one launch, and as the
sequence of launches that repeats a solve whose workgroups gave up waiting for each
other (a wait bound of zero makes them).  Both form every value and every sum in the
same order, so depth, iterations and residual are the same bits; the sequence is also
held to the oracle's direct FP64 solve with the bound of test_gpu_densify.py, on
inputs with varying texture, contour and stability maps."""
import numpy as np
import pytest

from gpu_util import dev, host
from oracle import densify as dz
from test_gpu_densify_tiles import inputs

pytestmark = pytest.mark.gpu


def solve(W, H, a, **kw):
    from paper_2203_02300_amd import Densifier
    Ds, Dpre, B, Mf, MI = a
    with Densifier(W, H, **kw) as z:
        D = host(z.run(dev(Ds), dev(B), dev(Mf), dev(MI), Dpre=dev(Dpre)))
        return D.view(np.uint32), z.stats(), z.launches()


# one pixel per thread; two, three and four (edges of tiles, odd rows and columns)
@pytest.mark.parametrize("W,H", [(200, 120), (33, 65), (257, 130), (640, 97), (1000, 200),
                                 (639, 361), (1279, 129), (1100, 701)])
def test_given_up_solve_has_the_same_bits(monkeypatch, W, H):
    a = inputs(W, H, W + H)
    print(f"densify paths {W}x{H}", flush=True)
    one = solve(W, H, a)
    monkeypatch.setenv("DCO_DENSIFY_WAIT", "0")
    many = solve(W, H, a)
    assert one[2] == 0 and many[2] > 0
    assert np.array_equal(one[0], many[0]) and one[1] == many[1]
    assert many[1][1] <= 1e-9 and 0 < many[1][0] < 400
    if W * H < 200000:
        want = dz.densify(*a)
        assert np.abs(many[0].view(np.float32) - want).max() <= 1e-5 * np.abs(want).max()


@pytest.mark.parametrize("max_iters", [0, 2, 7])
def test_iteration_limit_is_the_same(monkeypatch, max_iters):
    W, H = 200, 120
    a = inputs(W, H, 5)
    kw = dict(max_iters=max_iters, iters_per_launch=2)
    one = solve(W, H, a, **kw)
    monkeypatch.setenv("DCO_DENSIFY_WAIT", "0")
    many = solve(W, H, a, **kw)
    assert many[2] == (max_iters + 1) // 2
    assert np.array_equal(one[0], many[0]) and one[1] == many[1]
    assert one[1][0] == 2 * ((max_iters + 1) // 2)


def test_launches_of_a_large_grid():
    """A grid beyond one launch: the linear kernels against the oracle."""
    W, H = 1312, 832
    a = inputs(W, H, 8)
    D, (it, rel), launches = solve(W, H, a)
    assert launches > 0 and rel <= 1e-9 and 0 < it < 400
    want = dz.densify(*a)
    assert np.abs(D.view(np.float32) - want).max() <= 1e-5 * np.abs(want).max()


@pytest.mark.parametrize("wait", [None, "0"])
@pytest.mark.parametrize("which", [0, 1, 3, 4])  # Ds, Dpre, Mfuse, MI
def test_output_on_an_input(monkeypatch, which, wait):
    """The inputs stay whole until the solve has ended, given up or not."""
    from paper_2203_02300_amd import Densifier
    W, H = 200, 120
    a = inputs(W, H, 6)
    want = solve(W, H, a)[0]
    if wait:
        monkeypatch.setenv("DCO_DENSIFY_WAIT", wait)
    t = [dev(v) for v in a]
    with Densifier(W, H) as z:
        D = z.run(t[0], t[2], t[3], t[4], Dpre=t[1], out=t[which])
        assert D.data_ptr() == t[which].data_ptr()
        assert np.array_equal(host(D).view(np.uint32), want)
        assert (z.launches() > 0) == bool(wait)


@pytest.mark.parametrize("wait", ["", "abc", "-1", "0x", "1e9", " 0", "0 "])
def test_wait_that_is_no_number_is_ignored(monkeypatch, wait):
    W, H = 200, 120
    monkeypatch.setenv("DCO_DENSIFY_WAIT", wait)
    assert solve(W, H, inputs(W, H, 7))[2] == 0


def test_given_up_solves_are_remembered(monkeypatch):
    """After one, 16 solves go as launches without a try; after the next, 32."""
    from paper_2203_02300_amd import Densifier
    W, H = 200, 120
    monkeypatch.setenv("DCO_DENSIFY_WAIT", "0")
    Ds, Dpre, B, Mf, MI = (dev(v) for v in inputs(W, H, 7))
    with Densifier(W, H) as z:
        tries = []
        for _ in range(1 + 16 + 1 + 32 + 1):
            z.run(Ds, B, Mf, MI, Dpre=Dpre)
            assert z.launches() > 0
            tries.append(z.given_up())
    assert tries == [1] * 17 + [2] * 33 + [3]


def test_a_long_queue_holds_up_its_own_solve_only():
    """A solve behind half a second of work on its stream; one on an idle stream,
    started later, ends first."""
    import threading
    import time
    import torch
    from paper_2203_02300_amd import Densifier
    W, H = 200, 120
    a = [dev(v) for v in inputs(W, H, 9)]
    slow, idle = torch.cuda.Stream(), torch.cuda.Stream()

    def sleep_ms(cycles):  # one thread of the GPU counts
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        e[0].record()
        torch.cuda._sleep(cycles)
        e[1].record()
        torch.cuda.synchronize()
        return e[0].elapsed_time(e[1])

    sleep_ms(1000)
    cycles = int(1_000_000 * 500 / sleep_ms(1_000_000))
    ended, queued = {}, threading.Event()

    def run(stream, name, before):
        with torch.cuda.stream(stream), Densifier(W, H) as z:
            z.run(a[0], a[2], a[3], a[4], Dpre=a[1])
            if before:
                torch.cuda._sleep(before)
                queued.set()
            else:
                queued.wait()
                time.sleep(0.05)  # the other is in its solve
            t = time.perf_counter()
            z.run(a[0], a[2], a[3], a[4], Dpre=a[1])
            ended[name] = time.perf_counter(), time.perf_counter() - t

    ts = [threading.Thread(target=run, args=v) for v in ((slow, "slow", cycles), (idle, "idle", 0))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert ended["slow"][1] > 0.3
    assert ended["idle"][0] < ended["slow"][0] and ended["idle"][1] < 0.1, ended
