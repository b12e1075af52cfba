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
