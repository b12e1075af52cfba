"""Outputs that share memory with an input that the call reads to its end."""
import numpy as np
import pytest

from gpu_util import host

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


@pytest.mark.parametrize("iters", [1, 2, 3])
@pytest.mark.parametrize("which", ["disp", "valid", "dvote"])
def test_vote_outputs_on_the_arms(iters, which):
    """The first rows' outputs on the arms of rows whose tiles vote last."""
    import torch
    from paper_2203_02300_amd import StereoMatcher
    from paper_2203_02300_amd._lib import check, lib
    W, H, D = 128, 16000, 6
    P = W * H
    g = torch.Generator("cuda").manual_seed(3)
    agg = torch.rand((D, H, W), device="cuda", generator=g)
    dL = torch.randint(0, D, (H, W), device="cuda", generator=g).to(torch.int16)
    valid = torch.randint(0, 2, (H, W), device="cuda", generator=g).to(torch.uint8)
    arms = torch.randint(0, 8, (H, W, 4), device="cuda", generator=g).to(torch.uint8)
    y = torch.arange(H, device="cuda")[:, None]
    arms[..., 2] = torch.minimum(arms[..., 2], y.clamp(max=255).to(torch.uint8))
    arms[..., 3] = torch.minimum(arms[..., 3], (H - 1 - y).clamp(max=255).to(torch.uint8))
    x = torch.arange(W, device="cuda")[None]
    arms[..., 0] = torch.minimum(arms[..., 0], x.to(torch.uint8))
    arms[..., 1] = torch.minimum(arms[..., 1], (W - 1 - x).to(torch.uint8))
    with StereoMatcher(W, H, D) as m:
        want = dict(zip(("disp", "valid", "dvote"),
                        (host(t) for t in m.vote_refine(arms, agg, dL, valid, iters))))
        out = dict(disp=torch.empty(P, device="cuda"),
                   valid=torch.empty(P, dtype=torch.uint8, device="cuda"),
                   dvote=torch.empty(P, dtype=torch.int16, device="cuda"))
        # 8 P bytes: the arms in the first half, the output from row 15000's arms on
        both = torch.empty(8 * P, dtype=torch.uint8, device="cuda")
        both[:4 * P] = arms.reshape(-1)
        at = 4 * W * 15000
        n = out[which].numel() * out[which].element_size()
        out[which] = both[at:at + n].view(out[which].dtype)
        m._begin()
        check(lib().dco_vote_refine(m._h, both.data_ptr(), agg.data_ptr(), dL.data_ptr(),
                                    valid.data_ptr(), iters, out["disp"].data_ptr(),
                                    out["valid"].data_ptr(), out["dvote"].data_ptr()))
        for k, t in out.items():
            assert np.array_equal(host(t).reshape(H, W), want[k]), k
