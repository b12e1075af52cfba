"""Performance cases of the stereo framework: the calls a user's program makes.

``listed()`` names the cases, ``draw()`` gives further ones of the same
ranges, ``prepare()`` makes what the program has in hand before the call (the
inputs, on the GPU, and the handle it keeps), ``run()`` is one pass through
the public entry points and ``work()`` what the path cannot do without.
``exact()`` computes the outputs of ``run()`` in plain torch with 64-bit
integers and floats, without this repository's code.

A case's ``kind`` is the entry point it calls:

  match    ``StereoMatcher.match``, one rectified pair (``vote``: passes of
           the region vote)
  half     ``StereoMatcher.match_half``: the full pair reduced to a quarter
           of its area, matched, and turned into depth
  staged   the same match through ``StereoMatcher``'s staged calls, with the
           volumes in memory
  batch    ``BatchMatcher.match``: pairs of mixed size and range in one call
  soft     ``soft_argmin_disparity``: forward and backward (``train``) or
           the forward alone
  densify  ``Densifier.run``: dense depth from the sparse map
  contour  ``ContourFilter.run``: depth contour from a frame and its flows
"""
from __future__ import annotations

import math

import torch

from paper_2203_02300_amd import (BatchMatcher, ContourFilter, Densifier, StereoMatcher,
                                  soft_argmin_disparity)

FB = 1000.0                 # focal length x baseline of the depth conversion
THETA0 = (10.0, 30.0, 1.0)  # initial (lambda_AD, lambda_census, T) of the soft path
L1, TAU1 = 17, 20           # matcher defaults
GAMMA, EPS = 1.0, 0.8

# Sizes and ranges of the pairs a batch mixes.
BATCH_SIZES = ((320, 240), (640, 480), (960, 540), (1280, 720))
BATCH_DISPS = (32, 64, 96, 128)


def listed():
    return [
        # The smallest frame: launches and latency are all there is.
        dict(name="match_64x48_d16", kind="match", W=64, H=48, D=16, vote=0),
        # A cropped region of interest: ragged width, few rows, odd range.
        dict(name="match_437x93_d40", kind="match", W=437, H=93, D=40, vote=0),
        # A VGA camera.
        dict(name="match_640x480_d64", kind="match", W=640, H=480, D=64, vote=0),
        # The full frame with the full range: the headline workload.
        dict(name="match_1280x720_d128", kind="match", W=1280, H=720, D=128, vote=0),
        # A mid-size frame with the region vote switched on.
        dict(name="vote_960x540_d96", kind="match", W=960, H=540, D=96, vote=2),
        # The paper's operating point: quarter-size front end, vote and depth.
        dict(name="half_1280x720_d64", kind="half", W=640, H=360, D=64, vote=2),
        # The staged calls, for a program that uses the volumes in between.
        dict(name="staged_640x480_d64", kind="staged", W=640, H=480, D=64),
        # Offline processing of a mixed set of pairs.
        dict(name="batch_8_mixed", kind="batch", n=8, mix=100),
        # A training step of the differentiable head.
        dict(name="soft_train_8x640x480_d64", kind="soft", B=8, W=640, H=480, D=64, train=True),
        # The differentiable head used for inference on one small pair.
        dict(name="soft_infer_1x320x240_d32", kind="soft", B=1, W=320, H=240, D=32, train=False),
        # Dense depth on the reduced grid of the operating point.
        dict(name="densify_640x360", kind="densify", W=640, H=360),
        # Depth contour of a full frame from flows on the quarter grid.
        dict(name="contour_1280x720", kind="contour", W=1280, H=720),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: a kind by use, sizes spread over the log of its range,
    and no more work than the largest listed case."""
    most = max(work(c)["flops"] for c in listed())
    case = _drawn(rng)
    while work(case)["flops"] > most:
        case = _drawn(rng)
    return case


def _drawn(rng):
    kind = rng.choice(["match"] * 6 + ["half", "half", "staged", "batch", "soft", "soft",
                                       "densify", "contour"])
    if kind in ("match", "half", "staged"):
        most_w, most_h = (1280, 720) if kind != "half" else (640, 360)
        W, H = _log_int(rng, 64, most_w), _log_int(rng, 48, most_h)
        D = min(_log_int(rng, 16, 128 if kind == "match" else 64), W - 1)
        if kind == "staged":
            return dict(kind=kind, W=W, H=H, D=D)
        return dict(kind=kind, W=W, H=H, D=D, vote=rng.choice([0, 0, 2]) if kind == "match" else 2)
    if kind == "batch":
        return dict(kind=kind, n=rng.randint(2, 8), mix=rng.randint(0, 999))
    if kind == "soft":
        W, H, D = _log_int(rng, 64, 640), _log_int(rng, 48, 480), _log_int(rng, 16, 63)
        return dict(kind=kind, B=rng.randint(1, 8), W=W, H=H, D=D, train=rng.random() < 0.6)
    if kind == "densify":
        return dict(kind=kind, W=_log_int(rng, 160, 1280), H=_log_int(rng, 90, 720))
    return dict(kind=kind, W=_log_int(rng, 320, 1280), H=_log_int(rng, 180, 720))


# ---------------------------------------------------------------------------
# Inputs: rectified views of a scene of textured planes
# ---------------------------------------------------------------------------


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _gen(seed):
    return torch.Generator().manual_seed(int(seed))


def _noise(g, C, H, W, dev, octaves=4, period=32.0):
    """C x H x W fractal noise in about [-0.5, 0.5], with a fine component."""
    out = torch.zeros((C, H, W), device=dev)
    amp, total = 1.0, 0.0
    for _ in range(octaves):
        lat = torch.rand((1, C, int(H / period) + 3, int(W / period) + 3), generator=g).to(dev)
        up = torch.nn.functional.interpolate(lat, size=(H, W), mode="bilinear", align_corners=False)
        out += amp * (up[0] - 0.5)
        total += amp
        amp, period = amp / 2, max(period / 2, 2.0)
    return out / total


def _scene(W, H, D, seed, boxes=6):
    """Left and right views (H x W x 3 uint8), the left view's disparity and
    where its pixels are visible in the right view: a slanted background and
    nearer boxes, each with a texture of its own strength (dense, medium or
    weak), noise of two grey levels and a gain of the right view."""
    g, dev = _gen(seed), _device()
    u = lambda lo, hi: lo + (hi - lo) * float(torch.rand((), generator=g))
    cx, cy = W / 2.0, H / 2.0
    layers = []
    for k in range(boxes + 1):
        bx = u(-0.04, 0.04) if k == 0 else u(-0.02, 0.02)
        by = u(-0.04, 0.04) * D / 64.0 * 480.0 / max(H, 480)
        bx *= min(1.0, 0.6 * D / max(1.0, 0.04 * W))
        lo, hi = (0.1, 0.4) if k == 0 else (0.3 + 0.08 * k, 0.42 + 0.08 * k)
        w, h = u(W / 8, W / 2), u(H / 8, H / 2)
        x0, y0 = u(0, W - w), u(0, H - h)
        rect = (0.0, 0.0, float(W), float(H)) if k == 0 else (x0, y0, x0 + w, y0 + h)
        amp = (190.0, 120.0, 45.0)[int(3 * u(0, 0.999))]
        layers.append((u(lo, hi) * D, bx, by, rect, amp, [u(70, 185) for _ in range(3)]))
    shared = _noise(g, 1, H, W, dev)
    fine = torch.rand((3, H, W), generator=g).to(dev) - 0.5
    tex = 0.8 * shared + 0.2 * fine
    ys, xs = torch.meshgrid(torch.arange(H, device=dev, dtype=torch.float32),
                            torch.arange(W, device=dev, dtype=torch.float32), indexing="ij")
    left = torch.zeros((3, H, W), device=dev)
    right = torch.zeros((3, H, W), device=dev)
    disp = torch.zeros((H, W), device=dev)
    front = torch.zeros((H, W), device=dev)  # disparity of the right view's surface
    for a, bx, by, (x0, y0, x1, y1), amp, base in layers:
        base = torch.tensor(base, device=dev)[:, None, None]
        d = (a + bx * (xs - cx) + by * (ys - cy)).clamp(1.0, D - 2.0)
        m = (xs >= x0) & (xs < x1) & (ys >= y0) & (ys < y1)
        left = torch.where(m, base + amp * tex, left)
        disp = torch.where(m, d, disp)
        xl = (xs + a - bx * cx + by * (ys - cy)) / (1.0 - bx)
        dr = (xl - xs).clamp(1.0, D - 2.0)
        xl = xs + dr
        mr = (xl >= x0) & (xl < x1) & (ys >= y0) & (ys < y1)
        if x1 >= W:  # the background goes on beyond the left view
            mr = mr | ((xl >= W) & (ys >= y0) & (ys < y1) & (front == 0))
        i0 = xl.floor().clamp(0, W - 1).long()
        f = (xl - i0).clamp(0, 1)
        i1 = (i0 + 1).clamp(max=W - 1)
        smp = torch.stack([t.gather(1, i0) * (1 - f) + t.gather(1, i1) * f for t in tex])
        right = torch.where(mr, base + amp * smp, right)
        front = torch.where(mr, dr, front)
    gain = u(0.9, 1.1)
    sig = lambda: 2.0 * torch.randn((3, H, W), generator=g).to(dev)
    to8 = lambda t: t.round().clamp(0, 255).to(torch.uint8).permute(1, 2, 0).contiguous()
    xr = (xs - disp).round()
    seen = (xr >= 0) & ((front.gather(1, xr.clamp(0, W - 1).long()) - disp).abs() < 1.5)
    return to8(left + sig()), to8(gain * right + sig()), disp, seen


def _batch_shapes(case):
    g = _gen(case["mix"])
    pick = lambda: int(torch.randint(0, 4, (), generator=g))
    return [BATCH_SIZES[pick()] + (BATCH_DISPS[pick()],) for _ in range(case["n"])]


def _full_size(case):
    """The full frame of a quarter-size case (odd where the reduced width is)."""
    return 2 * case["W"] + (case["W"] & 1), 2 * case["H"] + (case["H"] & 1)


def _inputs(case, seed):
    kind = case["kind"]
    if kind in ("match", "staged"):
        L, R, _, _ = _scene(case["W"], case["H"], case["D"], seed)
        return dict(L=L, R=R)
    if kind == "half":
        W2, H2 = _full_size(case)
        L, R, _, _ = _scene(W2, H2, 2 * case["D"], seed)
        return dict(L=L, R=R)
    if kind == "batch":
        pairs = [_scene(W, H, D, 1000 * seed + i) for i, (W, H, D) in
                 enumerate(_batch_shapes(case))]
        return dict(L=[p[0] for p in pairs], R=[p[1] for p in pairs])
    if kind == "soft":
        pairs = [_scene(case["W"], case["H"], case["D"], 1000 * seed + i) for i in
                 range(case["B"])]
        return dict(zip(("L", "R", "gt", "seen"), (torch.stack(t) for t in zip(*pairs))))
    W, H = case["W"], case["H"]
    L, _, disp, _ = _scene(W, H, 64, seed)
    g, dev = _gen(seed + 1), _device()
    rand = lambda *s: torch.rand(s, generator=g).to(dev)
    if kind == "densify":
        # Ground-truth depth at 70 % of the pixels, the previous frame's
        # depth at half of them, the contour where the disparity jumps.
        depth = FB / disp
        jump = torch.zeros((H, W), dtype=torch.bool, device=dev)
        dx = (disp[:, 1:] - disp[:, :-1]).abs() > 1
        dy = (disp[1:] - disp[:-1]).abs() > 1
        jump[:, :-1] |= dx
        jump[:, 1:] |= dx
        jump[:-1] |= dy
        jump[1:] |= dy
        pre = depth * (1 + 0.01 * torch.randn((H, W), generator=g).to(dev))
        soft01 = lambda: (_noise(g, 1, H, W, dev, 2, 16.0)[0] + 0.5).clamp(0, 1)
        zero = torch.zeros((), device=dev)
        return dict(Ds=torch.where(rand(H, W) < 0.7, depth, zero),
                    Dpre=torch.where(rand(H, W) < 0.5, pre, zero),
                    Bdp=jump.to(torch.uint8), Mfuse=soft01(), MI=soft01())
    # contour: the nearest surfaces move, the rest stands still
    h, w = H // 2, W // 2
    near = disp[:2 * h:2, :2 * w:2]
    m = (near > 0.6 * float(near.max())).float()[None, None]
    for _ in range(3):  # the motion spreads a little over its borders
        m = torch.nn.functional.avg_pool2d(m, 3, 1, 1)
    v = 1.0 + 3.0 * torch.rand((2,), generator=g).to(dev)
    flow = m[0, 0, :, :, None] * v
    jit = lambda: 0.002 * torch.randn((h, w, 2), generator=g).to(dev)
    return dict(rgb=L, past=(-flow + jit()).contiguous(), future=(flow + jit()).contiguous())


# ---------------------------------------------------------------------------
# The measured call
# ---------------------------------------------------------------------------


def prepare(case, seed):
    s = _inputs(case, seed)
    kind = case["kind"]
    s["kind"] = kind
    if kind in ("match", "half", "staged", "soft"):
        s["m"] = StereoMatcher(case["W"], case["H"], case["D"], vote_iters=case.get("vote", 0))
    elif kind == "batch":
        s["m"] = BatchMatcher(_batch_shapes(case))
    elif kind == "densify":
        s["m"] = Densifier(case["W"], case["H"])
    else:
        s["m"] = ContourFilter(case["W"], case["H"])
    if kind == "soft":
        s["train"] = case["train"]
        s["theta"] = torch.tensor(THETA0, device=s["L"].device, requires_grad=case["train"])
        s["nseen"] = s["seen"].sum()
    return s


def run(s):
    m, kind = s["m"], s["kind"]
    if kind == "match":
        disp, valid = m.match(s["L"], s["R"])
        return dict(disp=disp, valid=valid)
    if kind == "half":
        disp, valid, depth = m.match_half(s["L"], s["R"], FB)
        return dict(disp=disp, valid=valid, depth=depth)
    if kind == "staged":
        cL, aL = m.census(s["L"])
        cR, aR = m.census(s["R"])
        aggL = m.aggregate(m.cost_volume(0, s["L"], s["R"], cL, cR, aL), aL)
        aggR = m.aggregate(m.cost_volume(1, s["L"], s["R"], cL, cR, aR), aR)
        disp, valid, dL, dR = m.wta_lrcheck(aggL, aggR)
        return dict(disp=disp, valid=valid, dL=dL, dR=dR, aggL=aggL, aggR=aggR)
    if kind == "batch":
        disps, valids = m.match(s["L"], s["R"])
        return dict(disps=disps, valids=valids)
    if kind == "soft":
        if not s["train"]:
            with torch.no_grad():
                return dict(dhat=soft_argmin_disparity(m, s["L"], s["R"], s["theta"]))
        dhat = soft_argmin_disparity(m, s["L"], s["R"], s["theta"])
        loss = ((dhat - s["gt"]).abs() * s["seen"]).sum() / s["nseen"]
        grad, = torch.autograd.grad(loss, s["theta"])
        return dict(dhat=dhat.detach(), loss=loss.detach(), grad=grad)
    if kind == "densify":
        return dict(depth=m.run(s["Ds"], s["Bdp"], s["Mfuse"], s["MI"], Dpre=s["Dpre"]))
    B, MI, Mn = m.run(s["rgb"], s["past"], s["future"])
    return dict(B=B, MI=MI, Mn=Mn)


# Operations per pixel, disparity and view of the matcher: about 14 for the
# raw cost and 26 for four range sums and two divisions.
OPS_PD = 40


def work(case):
    kind = case["kind"]
    if kind == "batch":
        shapes = _batch_shapes(case)
        return dict(bytes=sum(11 * W * H for W, H, _ in shapes),
                    flops=sum(2 * OPS_PD * W * H * D for W, H, D in shapes))
    P = case["W"] * case["H"]
    if kind == "match":
        return dict(bytes=11 * P, flops=2 * OPS_PD * P * case["D"])
    if kind == "half":
        W2, H2 = _full_size(case)
        return dict(bytes=6 * W2 * H2 + 9 * P, flops=2 * OPS_PD * P * case["D"])
    if kind == "staged":
        # every stage reads its inputs and writes its outputs: per view the
        # cost volume written and read and the aggregated volume written and
        # read, the images, codes and arms, and the maps
        V = P * case["D"]
        return dict(bytes=32 * V + 103 * P, flops=2 * OPS_PD * V)
    if kind == "soft":
        V = case["B"] * P * case["D"]
        passes = 3 if case["train"] else 1  # backward: about twice the forward
        io = (6 + 4 + (5 if case["train"] else 0)) * case["B"] * P
        return dict(bytes=io, flops=passes * OPS_PD * V)
    if kind == "densify":
        # the solve takes about 60 iterations of 14 FP64 operations per pixel
        return dict(bytes=21 * P, flops=60 * 14 * P)
    return dict(bytes=3 * P + 4 * P + 5 * P + P, flops=150 * P)


# ---------------------------------------------------------------------------
# The same outputs in 64 bits, in plain torch
# ---------------------------------------------------------------------------


def _reach(img, step, tau=TAU1, most=L1):
    """Arm lengths of every pixel in one direction: how many steps stay inside
    the image and below tau in every channel."""
    H, W = img.shape[:2]
    dy, dx = step
    ys = torch.arange(H, device=img.device)[:, None]
    xs = torch.arange(W, device=img.device)[None]
    ok = torch.ones((H, W), dtype=torch.bool, device=img.device)
    arm = torch.zeros((H, W), dtype=torch.int64, device=img.device)
    for k in range(1, most + 1):
        y, x = ys + k * dy, xs + k * dx
        other = img[y.clamp(0, H - 1), x.clamp(0, W - 1)]
        ok &= (y >= 0) & (y < H) & (x >= 0) & (x < W) & ((other - img).abs().amax(-1) < tau)
        arm += ok
    return arm


def _grey(img):
    return (77 * img[..., 0] + 150 * img[..., 1] + 29 * img[..., 2] + 128) >> 8


def _census(img):
    """62 comparison bits per pixel, one int64 each."""
    Y = _grey(img)
    H, W = Y.shape
    P = torch.nn.functional.pad(Y[None, None].double(), (4, 4, 3, 3), mode="replicate")[0, 0].long()
    code, bit = torch.zeros_like(Y), 0
    for dy in range(7):
        for dx in range(9):
            if (dy, dx) != (3, 4):
                code |= (P[dy:dy + H, dx:dx + W] < Y).long() << bit
                bit += 1
    return code


def _popcount(v):
    """Bits set in non-negative 62-bit integers."""
    v = v - ((v >> 1) & 0x5555555555555555)
    v = (v & 0x3333333333333333) + ((v >> 2) & 0x3333333333333333)
    v = (v + (v >> 4)) & 0x0F0F0F0F0F0F0F0F
    v = v + (v >> 8)
    v = v + (v >> 16)
    return (v + (v >> 32)) & 0x7F


class _View:
    """Per-pixel geometry of one reference view, and its region sums."""

    def __init__(self, rgb):
        self.img = rgb.long()
        self.code = _census(self.img)
        self.l, self.r = _reach(self.img, (0, -1)), _reach(self.img, (0, 1))
        self.u, self.d = _reach(self.img, (-1, 0)), _reach(self.img, (1, 0))
        self.H, self.W = self.l.shape
        x = torch.arange(self.W, device=rgb.device)[None]
        y = torch.arange(self.H, device=rgb.device)[:, None]
        self.hi = (x + self.r + 1, x - self.l)
        self.vi = (y + self.d + 1, y - self.u)
        one = torch.ones_like(self.l)
        self.n1, self.n2 = self.vert(self.horz(one)), self.horz(self.vert(one))
        self.lmin = torch.minimum(torch.minimum(self.l, self.r), torch.minimum(self.u, self.d))

    def _range(self, v, dim, idx):
        pad = [0] * 4
        pad[2 * (1 - dim)] = 1
        c = torch.nn.functional.pad(v.cumsum(dim), pad)
        return c.gather(dim, idx[0]) - c.gather(dim, idx[1])

    def horz(self, v):
        return self._range(v, 1, self.hi)

    def vert(self, v):
        return self._range(v, 0, self.vi)


def _partner(ref, other, d, sign):
    """(sum of channel differences, Hamming distance, partner inside) at
    disparity d, the partner at x + sign d."""
    x = torch.arange(ref.W, device=ref.img.device) + sign * d
    inside = ((x >= 0) & (x < ref.W))[None].expand(ref.H, ref.W)
    x = x.clamp(0, ref.W - 1)
    s = (ref.img - other.img[:, x]).abs().sum(-1)
    h = _popcount(ref.code ^ other.code[:, x])
    return s, h, inside


def _f32(v):
    return v.float().double()


class _Costs:
    """The aggregated costs of one reference view, slice by slice."""

    def __init__(self, ref, other, sign, lam_ad=10.0, lam_c=40.0):
        self.ref, self.other, self.sign = ref, other, sign
        dev = ref.img.device
        k = torch.arange(L1 + 1, device=dev, dtype=torch.float64)
        e = torch.exp(-GAMMA / (k + float(torch.tensor(EPS))))
        self.alpha, self.beta = _f32(1 - e)[ref.lmin], _f32(e)[ref.lmin]
        s = torch.arange(766, device=dev, dtype=torch.float64)
        self.ta = _f32(-torch.expm1(-s / (3 * lam_ad)))
        self.tc = _f32(-torch.expm1(-s[:65] / lam_c))

    def slice(self, d):
        """Twice aggregated cost of disparity d: (as FP32, as FP64)."""
        ref = self.ref
        s, h, inside = _partner(ref, self.other, d, self.sign)
        q = (torch.round(self.alpha * self.ta[s] * 2.0 ** 20)
             + torch.round(self.beta * self.tc[h] * 2.0 ** 20)).long()
        q = torch.where(inside, q, torch.full_like(q, 1 << 20))
        a1 = (ref.vert(ref.horz(q)) + ref.n1 // 2) // ref.n1
        s2 = ref.horz(ref.vert(a1))
        return ((s2.float() / ref.n2.float()) * 2.0 ** -20,
                (s2.double() / ref.n2.double()) * 2.0 ** -20)


def _winner(costs, D, keep):
    """Smallest disparity of the least FP32 cost; with keep, all costs in FP64."""
    best, bd, vol = None, None, []
    for d in range(D):
        c32, c64 = costs.slice(d)
        if keep:
            vol.append(c64)
        if d == 0:
            best, bd = c32, torch.zeros_like(costs.ref.l)
        else:
            less = c32 < best
            best, bd = torch.where(less, c32, best), torch.where(less, d, bd)
    return bd, (torch.stack(vol) if keep else None)


def _offset(vol, d):
    """Parabola vertex offset at disparity map d."""
    D = vol.shape[0]
    at = lambda k: vol.gather(0, k.clamp(0, D - 1)[None])[0]
    m, c, p = at(d - 1), at(d), at(d + 1)
    den = (m - c) + (p - c)
    ok = (d > 0) & (d < D - 1) & (den > 0)
    off = ((m - p) / (2 * torch.where(ok, den, torch.ones_like(den)))).clamp(-0.5, 0.5)
    return torch.where(ok, off, torch.zeros_like(off))


def _vote(view, dv, D):
    """One pass of the region vote on a disparity map (-1: no vote)."""
    most, win = torch.zeros_like(view.l), torch.zeros_like(dv)
    for d in range(D):
        n = view.vert(view.horz((dv == d).long()))
        more = n > most
        most, win = torch.where(more, n, most), torch.where(more, d, win)
    return torch.where(dv >= 0, win, dv)


def _match(L, R, D, vote=0, volumes=False):
    """(disp, valid, dL, dR) of one pair and both views' costs (the right
    view's only if asked for)."""
    vl, vr = _View(L), _View(R)
    dL, vol = _winner(_Costs(vl, vr, -1), D, True)
    dR, volR = _winner(_Costs(vr, vl, 1), D, volumes)
    xr = torch.arange(vl.W, device=L.device)[None] - dL
    valid = (xr >= 0) & (dL == dR.gather(1, xr.clamp(min=0)))
    dv = torch.where(valid, dL, torch.full_like(dL, -1))
    for _ in range(vote):
        dv = _vote(vl, dv, D)
    at = dv.clamp(min=0)
    disp = torch.where(valid, at + _offset(vol, at), torch.zeros((), dtype=torch.float64,
                                                                 device=L.device))
    return disp, valid.to(torch.uint8), dL.to(torch.int16), dR.to(torch.int16), vol, volR


def _soft(case, s):
    """dhat, and for a training step the loss and its gradient."""
    B, D = case["B"], case["D"]
    theta = torch.tensor(THETA0, dtype=torch.float64, device=s["L"].device, requires_grad=True)
    nseen = s["nseen"] if "nseen" in s else s["seen"].sum()
    dhats, loss, grad = [], 0.0, torch.zeros_like(theta)
    for b in range(B):
        vl, vr = _View(s["L"][b]), _View(s["R"][b])
        al = 1 - torch.exp(-GAMMA / (vl.lmin.double() + float(torch.tensor(EPS))))
        vol = []
        with torch.set_grad_enabled(case["train"]):
            for d in range(D):
                sad, ham, inside = _partner(vl, vr, d, -1)
                c = (al * (1 - torch.exp(-(sad / 3.0) / theta[0]))
                     + (1 - al) * (1 - torch.exp(-ham / theta[1])))
                c = torch.where(inside, c, torch.ones_like(c))
                a1 = vl.vert(vl.horz(c)) / vl.n1
                vol.append(vl.horz(vl.vert(a1)) / vl.n2)
            w = torch.softmax(-torch.stack(vol) / theta[2], 0)
            k = torch.arange(D, device=w.device, dtype=torch.float64)[:, None, None]
            dhat = (w * k).sum(0)
            part = ((dhat - s["gt"][b].double()).abs() * s["seen"][b]).sum() / nseen
        if case["train"]:
            grad = grad + torch.autograd.grad(part, theta)[0]
            loss = loss + part.detach()
        dhats.append(dhat.detach())
    dhat = torch.stack(dhats)
    return dict(dhat=dhat, loss=loss, grad=grad.detach()) if case["train"] else dict(dhat=dhat)


def _densify(s):
    """Conjugate gradients on the normal equations, to the end of FP64."""
    Ds, Dp = s["Ds"].double(), s["Dpre"].double()
    lam_d, lam_s, lam_s2 = (float(torch.tensor(v)) for v in (0.8, 1.2, 0.02))
    sm, on = s["Mfuse"].double() * s["MI"].double(), s["Bdp"] != 0

    def edge(a, b):
        w = (1 - torch.minimum(sm[a], sm[b])).clamp(min=0)
        return 2 * lam_s * torch.where(on[a] ^ on[b], torch.zeros_like(w), w)

    n = slice(None)
    cr = edge((n, slice(0, -1)), (n, slice(1, None)))
    cd = edge((slice(0, -1), n), (slice(1, None), n))
    wd, wp = lam_d * (Ds > 0), lam_s2 * (Dp > 0)

    def add(y, v, w):
        y[:, :-1] += cr * v[:, w(0, -1)]
        y[:, 1:] += cr * v[:, w(1, 0)]
        y[:-1] += cd * v[w(0, -1)]
        y[1:] += cd * v[w(1, 0)]

    own = lambda lo, hi: slice(1, None) if lo else slice(0, -1)
    far = lambda lo, hi: slice(0, -1) if lo else slice(1, None)
    diag = wd + wp
    add(diag, torch.ones_like(diag), own)

    def mul(v):
        t = torch.zeros_like(v)
        add(t, v, far)
        return diag * v - t

    b = wd * Ds + wp * Dp
    inv = torch.where(diag > 0, 1 / torch.where(diag > 0, diag, torch.ones_like(diag)),
                      torch.zeros_like(diag))
    x, r = torch.zeros_like(b), b.clone()
    z = inv * r
    p, rz, bb = z.clone(), float((r * z).sum()), float((b * b).sum())
    for _ in range(400):
        if rz <= 0 or float((r * r).sum()) <= 1e-26 * bb:
            break
        q = mul(p)
        a = rz / float((p * q).sum())
        x += a * p
        r -= a * q
        z = inv * r
        new = float((r * z).sum())
        p = z + (new / rz) * p
        rz = new
    return x


def _contour(s):
    """(MI, Mn); the contour itself is a yes or no."""
    def terms(F):
        F = F.double()
        h, w = F.shape[:2]
        r = F.norm(dim=-1)
        gu, gv = torch.zeros_like(r), torch.zeros_like(r)
        gu[:, :-1] = (r[:, 1:] - r[:, :-1]).abs()
        gv[:-1] = (r[1:] - r[:-1]).abs()
        e = F / r.clamp(min=1e-300)[..., None]
        st = torch.round(e).long()
        ys = torch.arange(h, device=F.device)[:, None]
        xs = torch.arange(w, device=F.device)[None]
        at = lambda k: (F[(ys + k * st[..., 1]).clamp(0, h - 1),
                          (xs + k * st[..., 0]).clamp(0, w - 1)] * e).sum(-1)
        return torch.maximum(gu, gv), torch.where(r > 0, at(1) - at(-1), torch.zeros_like(r))

    mp, sp = terms(s["past"])
    mf, sf = terms(s["future"])
    fused = torch.where(sp > sf, mp, torch.where(sf > sp, mf, torch.maximum(mp, mf)))
    box = torch.nn.functional.avg_pool2d(fused[None, None], 5, 1, 2, count_include_pad=False)[0, 0]
    Mn = box / box.max() if float(box.max()) > 0 else box * 0
    Y = torch.nn.functional.pad(_grey(s["rgb"].long())[None, None].double(), (1, 1, 1, 1),
                                mode="replicate")[0, 0]
    H, W = s["rgb"].shape[:2]
    at = lambda dy, dx: Y[1 + dy:1 + dy + H, 1 + dx:1 + dx + W]
    gx = at(-1, 1) + 2 * at(0, 1) + at(1, 1) - at(-1, -1) - 2 * at(0, -1) - at(1, -1)
    gy = at(1, -1) + 2 * at(1, 0) + at(1, 1) - at(-1, -1) - 2 * at(-1, 0) - at(-1, 1)
    g2 = gx * gx + gy * gy
    return torch.sqrt(g2 / g2.max().clamp(min=1)), Mn


def _halved(img):
    v = img[:img.shape[0] // 2 * 2, :img.shape[1] // 2 * 2].long()
    return ((v[::2, ::2] + v[1::2, ::2] + v[::2, 1::2] + v[1::2, 1::2] + 2) >> 2).to(torch.uint8)


def exact(case, seed):
    """What run() returns for the inputs of this seed, in 64 bits.  Whole
    numbers follow the documented fixed-point contract; a winner is the least
    FP32 cost, as documented, and the offsets around it are FP64."""
    s, kind = _inputs(case, seed), case["kind"]
    if kind == "match":
        disp, valid = _match(s["L"], s["R"], case["D"], case["vote"])[:2]
        return dict(disp=disp, valid=valid)
    if kind == "half":
        disp, valid = _match(_halved(s["L"]), _halved(s["R"]), case["D"], case["vote"])[:2]
        disp = 2 * disp
        depth = torch.where(disp > 0, FB / torch.where(disp > 0, disp, torch.ones_like(disp)),
                            torch.zeros_like(disp))
        return dict(disp=disp, valid=valid, depth=depth)
    if kind == "staged":
        return dict(zip(("disp", "valid", "dL", "dR", "aggL", "aggR"),
                        _match(s["L"], s["R"], case["D"], volumes=True)))
    if kind == "batch":
        res = [_match(L, R, D) for L, R, (W, H, D) in zip(s["L"], s["R"], _batch_shapes(case))]
        return dict(disps=[r[0] for r in res], valids=[r[1] for r in res])
    if kind == "soft":
        return _soft(case, s)
    if kind == "densify":
        return dict(depth=_densify(s))
    MI, Mn = _contour(s)
    return dict(B=None, MI=MI, Mn=Mn)
