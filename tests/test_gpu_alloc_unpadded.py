"""A handle whose scratch does not fit the card with padded volume rows takes rows of
W columns instead, with the same results.  dco_debug_fail_alloc makes one allocation
of the first try fail."""
import ctypes as C

import numpy as np
import pytest

from gpu_util import dev, host
from paper_2203_02300_amd import synth

pytestmark = pytest.mark.gpu

OOM = -4


def create(W, H, D, **kw):
    from paper_2203_02300_amd import _lib
    L = _lib.lib()
    p = _lib.Params()
    L.dco_default_params(C.byref(p))
    for k, v in kw.items():
        setattr(p, k, v)
    h = C.c_void_p()
    return L.dco_stereo_create(C.byref(h), W, H, D, C.byref(p), None), h


@pytest.mark.parametrize("W,H,D,vote", [(50, 40, 16, 0), (61, 33, 17, 2), (228, 24, 9, 1)])
def test_matcher_without_padding(W, H, D, vote):
    import torch
    from paper_2203_02300_amd import _lib
    L = _lib.lib()
    p = synth.make_slanted_pair(W, H, D, 31, n_planes=2, dmin=2.0, dmax=D - 3.0,
                                noise_sigma=2.0, occl_strip_frac=0.03)
    a, b = dev(p["left"]), dev(p["right"])

    def run(h):
        disp, valid = torch.empty((H, W), device="cuda"), torch.empty((H, W), dtype=torch.uint8,
                                                                      device="cuda")
        agg = torch.empty((2, D, H, W), device="cuda")
        torch.cuda.synchronize()  # the handle runs on the default stream
        assert L.dco_stereo_match(h, a.data_ptr(), b.data_ptr(), disp.data_ptr(),
                                  valid.data_ptr()) == 0
        for v in range(2):
            assert L.dco_stereo_agg_slices(h, v, 0, D, agg[v].data_ptr()) == 0
        torch.cuda.synchronize()
        return [host(t) for t in (disp, valid, agg)]

    base = L.dco_debug_live_allocations()
    st, h = create(W, H, D, vote_iters=vote)
    assert st == 0
    want = run(h)
    live = L.dco_debug_live_allocations()
    L.dco_stereo_destroy(h)
    tables = 4  # the tables have no second try
    try:
        for k in range(1, live - base + 1):
            L.dco_debug_fail_alloc(k)
            st, h = create(W, H, D, vote_iters=vote)
            L.dco_debug_fail_alloc(0)
            if k <= tables:
                assert st == OOM and not h.value
                continue
            assert st == 0, k
            assert L.dco_debug_live_allocations() == live
            for g, w in zip(run(h), want):
                assert np.array_equal(g, w), k
            L.dco_stereo_destroy(h)
            assert L.dco_debug_live_allocations() == base
        # one stage has no padding to do without
        L.dco_debug_fail_alloc(tables + 1)
        assert create(W, H, D, agg_iters=1)[0] == OOM
    finally:
        L.dco_debug_fail_alloc(0)
    assert L.dco_debug_live_allocations() == base


# less than a quad, a cut quad of one, two and three columns, one and several groups
@pytest.mark.parametrize("W,H,D,B", [(11, 12, 5, 2), (97, 21, 20, 2), (130, 9, 40, 1),
                                     (67, 30, 66, 1), (332, 8, 17, 1)])
def test_soft_path_without_padding(W, H, D, B):
    """Every allocation of the soft scratch failing once: the same bits."""
    import torch
    from paper_2203_02300_amd import StereoMatcher, _lib
    from paper_2203_02300_amd.soft import soft_backward, soft_forward
    D = min(D, W - 1)
    L = _lib.lib()
    rng = np.random.default_rng(W)
    a = rng.integers(0, 256, (B, H, W, 3), dtype=np.uint8)
    b = np.roll(a, -2, axis=2)
    gd = dev(rng.normal(0, 1e-2, (B, H, W)).astype(np.float32))
    a, b = dev(a), dev(b)
    theta = torch.tensor([10.0, 30.0, 0.5], dtype=torch.float32, device="cuda")

    def run(k):
        with StereoMatcher(W, H, D) as m:
            L.dco_debug_fail_alloc(k)
            try:
                dh, lse = soft_forward(m, a, b, theta)
            finally:
                L.dco_debug_fail_alloc(0)
            g = soft_backward(m, a, b, theta, dh, lse, gd, reuse=True)
            return [host(t) for t in (dh, lse, g)]

    want = run(0)
    for k in (1, 7, 8, 9, 11):  # maps, the three volumes, partial sums
        for g, w in zip(run(k), want):
            assert np.isfinite(w).all() and np.array_equal(g, w), k
