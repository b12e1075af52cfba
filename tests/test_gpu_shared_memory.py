"""Outputs that share memory with an input that the call reads to its end."""
import numpy as np
import pytest

import oracle
from gpu_util import dev, host
from paper_2203_02300_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H,D", [(64, 16000, 8), (61, 9000, 5)])
@pytest.mark.parametrize("view", [0, 1])
def test_wta_outputs_on_a_volume(W, H, D, view):
    """Output bytes of the first rows lie on volume rows that are read last: more rows
    than the GPU runs at once."""
    import torch
    from paper_2203_02300_amd import StereoMatcher
    from paper_2203_02300_amd._lib import check, lib
    P = W * H
    agg = [torch.rand((D * P,), device="cuda", generator=torch.Generator("cuda").manual_seed(k))
           for k in (1, 2)]
    with StereoMatcher(W, H, D) as m:
        want = [host(t) for t in m.wta_lrcheck(*(a.view(D, H, W) for a in agg))]

        def run(disp, valid):
            dL, dR = (torch.empty((H, W), dtype=torch.int16, device="cuda") for _ in range(2))
            m._begin()
            check(lib().dco_wta_lrcheck(m._h, agg[0].data_ptr(), agg[1].data_ptr(),
                                        disp.data_ptr(), valid.data_ptr(), dL.data_ptr(),
                                        dR.data_ptr()))
            return [host(t) for t in (disp, valid, dL, dR)]

        saved = [a.clone() for a in agg]
        free_d, free_v = torch.empty(P, device="cuda"), torch.empty(P, dtype=torch.uint8,
                                                                    device="cuda")
        for n in range(2):
            # the end of a slice: row 0's outputs on rows near its last
            disp = agg[view][2 * P - 40 * W:3 * P - 40 * W] if n == 0 else free_d
            valid = agg[view].view(torch.uint8)[4 * (2 * P) - P:4 * (2 * P)] if n else free_v
            got = run(disp, valid)
            for g, w in zip(got, want):
                assert np.array_equal(g.reshape(H, W), w)
            for a, s in zip(agg, saved):
                a.copy_(s)
