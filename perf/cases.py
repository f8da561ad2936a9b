"""The library's calls as programs make them, for timing: listed() and draw() name the sizes, prepare() makes
what a program holds before the call (inputs on the GPU, plans, weights), run() makes the call.

Kinds of case:
  me          motion estimation of one frame against its predecessor, as a video encoder does per frame
  pool        one pooling layer of a convolutional network (fp32)
  conv        one convolution layer (fp16), weights as they lie or packed once
  bottleneck  a residual block of three layers: 1x1 down, 3x3, 1x1 up with the block's input added
  dwsep       a depthwise-separable block: a depthwise layer, then a 1x1 layer
  corr        the correlation layer of an optical-flow network
  sep         a separable filter (Gaussian) over a batch of fp32 images
  bilateral   a bilateral filter over fp32 images
"""
import math

import torch

from paper_1911_03458_amd import binding as mb


# --------------------------------------------------------------------------
# sizes
# --------------------------------------------------------------------------
def listed():
    return [
        # the smallest call there is: a thumbnail, 64 blocks; latency and launches are all of it
        dict(name="me_64x64_b8_r4", kind="me", H=64, W=64, block=8, search=4),
        # a full-HD frame at its real height: the last row of 16x16 blocks reaches past the edge
        dict(name="me_1920x1080_b16_r32", kind="me", H=1080, W=1920, block=16, search=32),
        # the first pooling layer of a residual network, as an average
        dict(name="pool_avg_16x64x112x112", kind="pool", N=16, C=64, H=112, W=112, k=3, s=2, p=1, avg=True),
        # the first pooling layer of AlexNet: an odd width, no padding
        dict(name="pool_max_32x96x55x55", kind="pool", N=32, C=96, H=55, W=55, k=3, s=2, p=0, avg=False),
        # an ordinary 3x3 layer of a small serving batch
        dict(name="conv_8x64x56x56_k3", kind="conv", N=8, Cin=64, H=56, W=56, Cout=64, k=3, s=1, p=1, relu=True,
             packed=False),
        # the largest: a deep VGG-16 layer on a large batch, weights packed once as a server does
        dict(name="conv_64x256x56x56_k3_packed", kind="conv", N=64, Cin=256, H=56, W=56, Cout=256, k=3, s=1, p=1,
             relu=True, packed=True),
        # a network's first layer on three-channel images
        dict(name="conv_32x3x224x224_k7s2", kind="conv", N=32, Cin=3, H=224, W=224, Cout=64, k=7, s=2, p=3,
             relu=True, packed=False),
        # a late residual block: small images, many channels, three dependent launches
        dict(name="bottleneck_8x1024x14x14", kind="bottleneck", N=8, C=1024, M=256, H=14, W=14),
        # a block of a mobile network: the depthwise layer is bound by memory, the 1x1 layer follows at once
        dict(name="dwsep_32x32x64x64", kind="dwsep", N=32, C=32, H=64, W=64, Cout=64, k=3, s=1),
        # the correlation layer on one pair of feature maps
        dict(name="corr_1x256x64x64_r5_s2", kind="corr", N=1, C=256, H=64, W=64, R=5, sd=2),
        # a wide Gaussian over four full-HD planes
        dict(name="sep_4x1080x1920_k30", kind="sep", N=4, H=1080, W=1920, k=30),
        # denoising one full-HD plane
        dict(name="bilateral_1x1080x1920_k9", kind="bilateral", N=1, H=1080, W=1920, k=9),
    ]


def _log(rng, lo, hi):
    """A whole number of [lo, hi], spread over its logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _channels(rng, lo, hi):
    """Channel counts: mostly multiples of 8, as networks have them, some not."""
    c = _log(rng, lo, hi)
    return c if rng.random() < 0.15 else max(lo, c // 8 * 8)


def _drawn(rng, kind):
    if kind == "me":                       # frames are of even size; the block seldom divides them
        block = rng.choice((8, 16))
        return dict(kind=kind, H=2 * _log(rng, 24, 540), W=2 * _log(rng, 32, 960), block=block,
                    search=rng.choice((4, 8, 16) if block == 8 else (8, 16, 32)))
    if kind == "pool":
        H, W = _log(rng, 7, 147), _log(rng, 7, 147)
        k, s, p = rng.choice(((3, 2, 0), (3, 2, 1), (2, 2, 0), (3, 1, 1), (7, 1, 0)))
        if k == 7:
            H = W = 7                      # a network's last pooling layer
        return dict(kind=kind, N=_log(rng, 1, 32), C=_log(rng, 16, 1024), H=H, W=W, k=k, s=s, p=p,
                    avg=rng.random() < 0.5)
    if kind == "conv":
        relu, packed = rng.random() < 0.5, rng.random() < 0.5
        if rng.random() < 0.25:            # a first layer
            k, s = rng.choice(((3, 1), (3, 2), (7, 2), (11, 4)))
            return dict(kind=kind, N=_log(rng, 1, 32), Cin=rng.choice((1, 3, 3, 4)), H=_log(rng, 64, 260),
                        W=_log(rng, 64, 260), Cout=rng.choice((32, 48, 64, 96)), k=k, s=s, p=k // 2, relu=relu,
                        packed=False)
        k = rng.choice((1, 1, 3, 3, 3, 5))
        return dict(kind=kind, N=_log(rng, 1, 64), Cin=_channels(rng, 16, 1024), H=_log(rng, 7, 112),
                    W=_log(rng, 7, 112), Cout=_channels(rng, 16, 1024), k=k, s=rng.choice((1, 1, 1, 2)), p=k // 2,
                    relu=relu, packed=packed)
    if kind == "bottleneck":
        M = 8 * _log(rng, 4, 64)
        return dict(kind=kind, N=_log(rng, 1, 32), C=4 * M, M=M, H=_log(rng, 7, 56), W=_log(rng, 7, 56))
    if kind == "dwsep":
        C = 8 * _log(rng, 2, 64)
        return dict(kind=kind, N=_log(rng, 1, 32), C=C, H=_log(rng, 7, 112), W=_log(rng, 7, 112),
                    Cout=C * rng.choice((1, 2)), k=rng.choice((3, 3, 5)), s=rng.choice((1, 1, 2)))
    if kind == "corr":
        return dict(kind=kind, N=1, C=8 * _log(rng, 4, 32), H=_log(rng, 16, 64), W=_log(rng, 16, 64),
                    R=rng.choice((3, 4, 5)), sd=rng.choice((1, 1, 2)))
    if kind == "sep":
        return dict(kind=kind, N=_log(rng, 1, 4), H=_log(rng, 120, 1080), W=_log(rng, 160, 1920),
                    k=rng.randint(3, 31))
    return dict(kind="bilateral", N=1, H=_log(rng, 120, 1080), W=_log(rng, 160, 1920),
                k=2 * rng.randint(1, 6) + 1)


# A drawn case stays well below the largest listed one: operations of the kind (multiply-adds count two) and bytes.
_MOST = dict(me=4e9, pool=1e9, conv=16e9, bottleneck=16e9, dwsep=16e9, corr=1e8, sep=1e9, bilateral=2e9)


def draw(rng):
    kind = rng.choice(("me", "pool", "conv", "conv", "conv", "bottleneck", "dwsep", "corr", "sep", "bilateral"))
    while True:
        case = _drawn(rng, kind)
        w = work(case)
        if w["flops"] <= _MOST[kind] and w["bytes"] <= 80e6:
            return case


def _out(i, k, s, p):
    return (i + 2 * p - k) // s + 1


def work(case):
    """What one pass cannot do without: every input read once, every output written once; operations of the
    definition (a multiply-add counts two, an absolute difference and its addition two)."""
    c, kind = case, case["kind"]
    if kind == "me":
        blocks = -(-c["H"] // c["block"]) * -(-c["W"] // c["block"])
        return dict(bytes=2 * c["H"] * c["W"] + 12 * blocks,
                    flops=2 * blocks * c["block"] ** 2 * (2 * c["search"] + 1) ** 2)
    if kind == "pool":
        o = _out(c["H"], c["k"], c["s"], c["p"]) * _out(c["W"], c["k"], c["s"], c["p"])
        return dict(bytes=4 * c["N"] * c["C"] * (c["H"] * c["W"] + o), flops=c["N"] * c["C"] * o * c["k"] ** 2)
    if kind == "conv":
        o = c["N"] * _out(c["H"], c["k"], c["s"], c["p"]) * _out(c["W"], c["k"], c["s"], c["p"])
        taps = c["Cin"] * c["k"] ** 2
        return dict(bytes=2 * (c["N"] * c["Cin"] * c["H"] * c["W"] + c["Cout"] * taps + o * c["Cout"]),
                    flops=2 * o * c["Cout"] * taps)
    if kind == "bottleneck":
        px, macs = c["N"] * c["H"] * c["W"], 2 * c["C"] * c["M"] + 9 * c["M"] ** 2
        return dict(bytes=2 * (2 * px * c["C"] + macs), flops=2 * px * macs)
    if kind == "dwsep":
        o = c["N"] * _out(c["H"], c["k"], c["s"], c["k"] // 2) * _out(c["W"], c["k"], c["s"], c["k"] // 2)
        return dict(bytes=2 * (c["N"] * c["C"] * c["H"] * c["W"] + c["C"] * c["k"] ** 2 + c["C"] * c["Cout"]
                               + o * c["Cout"]),
                    flops=2 * o * c["C"] * (c["k"] ** 2 + c["Cout"]))
    if kind == "corr":
        o = c["N"] * c["H"] * c["W"] * (2 * c["R"] + 1) ** 2
        return dict(bytes=2 * (2 * c["N"] * c["C"] * c["H"] * c["W"] + o), flops=2 * o * c["C"])
    px = c["N"] * c["H"] * c["W"]
    if kind == "sep":
        return dict(bytes=8 * px, flops=4 * px * c["k"])
    return dict(bytes=8 * px, flops=8 * px * c["k"] ** 2)     # difference, square, exponential, two sums


def tolerance(case):
    """About four times what the same pass in 64 bits differs by, over the listed cases and forty drawn ones
    (intermediate fp16 tensors rounded where the layers round them)."""
    kind = case["kind"]
    if kind == "me" or (kind == "pool" and not case["avg"]):
        return "exact"
    if kind in ("pool", "sep", "bilateral"):       # fp32 sums: 9e-8 and 5e-7
        return {"rel": 4e-7, "max": 2e-6}
    if kind == "bottleneck":                       # three roundings to fp16 in a row: 1.1e-4 and 1e-3
        return {"rel": 4e-4, "max": 4e-3}
    # fp32 sums rounded to fp16, a unit in the last place here and there: 1.3e-5 and 1e-3 (dwsep 2.1e-3)
    return {"rel": 5e-5, "max": 8e-3 if kind == "dwsep" else 4e-3}


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _frames(case, g):
    """Two frames of a moving scene (uint8): detail at every scale, a camera pan, a few objects that move their own
    way, a flat region, and sensor noise in both frames."""
    H, W, R = case["H"], case["W"], case["search"]
    m = R + 8
    h, w = H + 2 * m, W + 2 * m
    scene = torch.full((h, w), 128.0, device="cuda")
    step, amp = 128, 40.0
    while step >= 2:
        coarse = torch.randn((1, 1, h // step + 2, w // step + 2), device="cuda", generator=g)
        scene += amp * torch.nn.functional.interpolate(coarse, size=(h, w), mode="bilinear")[0, 0]
        step, amp = step // 2, amp * 0.7
    scene[: h // 6] = 190.0                        # sky
    r = torch.rand(40, generator=g, device="cuda").tolist()          # (host values: where things are)

    def noise():
        return 1.5 * torch.randn((H, W), device="cuda", generator=g)

    def view(dy, dx):
        return scene[m + dy:m + dy + H, m + dx:m + dx + W]

    pan = (round((r[0] - 0.5) * R), round((r[1] - 0.5) * R))
    ref, cur = view(0, 0) + noise(), view(*pan) + noise()
    for i in range(6):
        y, x, dy, dx = (r[2 + 4 * i + j] for j in range(4))
        bh, bw = max(4, H // 5), max(4, W // 5)
        y, x = int(y * (H - bh)), int(x * (W - bw))
        moved = view(round((2 * dy - 1) * R), round((2 * dx - 1) * R))
        cur[y:y + bh, x:x + bw] = moved[y:y + bh, x:x + bw] + noise()[y:y + bh, x:x + bw]
    return tuple(t.round().clamp(0, 255).to(torch.uint8) for t in (cur, ref))


def _activations(shape, g):
    """What a clipped layer hands to the next one: half zeros."""
    return torch.randn(shape, device="cuda", generator=g).relu_().half()


def _weights(shape, g, gain=2.0):
    fan_in = math.prod(shape[1:])
    return (torch.randn(shape, device="cuda", generator=g) * math.sqrt(gain / fan_in)).half()


def _images(case, g):
    """fp32 images of 0..255: patches of a few grey levels and noise."""
    N, H, W = case["N"], case["H"], case["W"]
    coarse = torch.randint(0, 4, (N, 1, -(-H // 40), -(-W // 40)), device="cuda", generator=g).float() * 60 + 30
    x = coarse.repeat_interleave(40, 2).repeat_interleave(40, 3)[:, 0, :H, :W]
    return (x + 8 * torch.randn((N, H, W), device="cuda", generator=g)).clamp(0, 255).contiguous()


def _gauss(k, sigma, normalise):
    a = torch.arange(k, dtype=torch.float64) - k // 2
    t = torch.exp(-0.5 * (a / sigma) ** 2)
    return (t / t.sum() if normalise else t).float().cuda()


def prepare(case, seed):
    c, kind, g = case, case["kind"], _generator(seed)
    if kind == "me":
        cur, ref = _frames(c, g)
        return dict(kind=kind, plan=mb.merit_plan_sad(c["H"], c["W"], c["block"], c["search"]), cur=cur, ref=ref)
    if kind == "pool":
        return dict(kind=kind, plan=mb.merit_plan_pool2d(c["N"], c["C"], c["H"], c["W"], c["k"], c["k"], c["s"], c["s"],
                                                         c["p"], c["p"], c["avg"]),
                    x=torch.randn((c["N"], c["C"], c["H"], c["W"]), device="cuda", generator=g))
    if kind == "conv":
        make = mb.merit_plan_conv2d_relu if c["relu"] else mb.merit_plan_conv2d
        plan = make(c["N"], c["Cin"], c["H"], c["W"], c["Cout"], c["k"], c["k"], c["s"], c["s"], c["p"], c["p"])
        shape = (c["N"], c["Cin"], c["H"], c["W"])
        if c["Cin"] < 8:                           # pixels
            x = torch.rand(shape, device="cuda", generator=g).mul_(2).sub_(1).half()
        else:
            x = _activations(shape, g)
        state = dict(kind=kind, plan=plan, x=x, w=_weights((c["Cout"], c["Cin"], c["k"], c["k"]), g), packed=None)
        if c["packed"]:
            try:
                state["packed"] = mb.merit_conv2d_pack_weights(plan, state["w"])
            except mb.MeritError:                  # this layer's plan has no packed form
                pass
        return state
    if kind == "bottleneck":
        N, C, M, H, W = (c[k] for k in ("N", "C", "M", "H", "W"))
        return dict(kind=kind, x=_activations((N, C, H, W), g),
                    plans=(mb.merit_plan_conv2d_relu(N, C, H, W, M, 1, 1, 1, 1, 0, 0),
                           mb.merit_plan_conv2d_relu(N, M, H, W, M, 3, 3, 1, 1, 1, 1),
                           mb.merit_plan_conv2d_residual(N, M, H, W, C, 1, 1, 1, 1, 0, 0, relu=1)),
                    w=(_weights((M, C, 1, 1), g), _weights((M, M, 3, 3), g), _weights((C, M, 1, 1), g)))
    if kind == "dwsep":
        N, C, H, W, k, s = (c[n] for n in ("N", "C", "H", "W", "k", "s"))
        oh, ow = _out(H, k, s, k // 2), _out(W, k, s, k // 2)
        return dict(kind=kind, x=_activations((N, C, H, W), g),
                    plans=(mb.merit_plan_conv2d_depthwise(N, C, H, W, k, k, s, s, k // 2, k // 2),
                           mb.merit_plan_conv2d_relu(N, C, oh, ow, c["Cout"], 1, 1, 1, 1, 0, 0)),
                    w=(_weights((C, k, k), g), _weights((c["Cout"], C, 1, 1), g)))
    if kind == "corr":
        shape = (c["N"], c["C"], c["H"], c["W"])
        a = torch.randn(shape, device="cuda", generator=g)
        b = torch.roll(a, shifts=(2, -4), dims=(2, 3)) + 0.5 * torch.randn(shape, device="cuda", generator=g)
        return dict(kind=kind, plan=mb.merit_plan_correlation(c["N"], c["C"], c["H"], c["W"], c["R"], c["sd"]),
                    x1=(a / math.sqrt(c["C"])).half(), x2=b.half())
    k = c["k"]
    if kind == "sep":
        return dict(kind=kind, plan=mb.merit_plan_sepfilter(c["N"], c["H"], c["W"], k), x=_images(c, g),
                    kx=_gauss(k, k / 6, True), ky=_gauss(k, k / 4, True))
    return dict(kind=kind, plan=mb.merit_plan_bilateral(c["N"], c["H"], c["W"], k), x=_images(c, g),
                g=_gauss(k, max(k / 3, 0.5), False), norm=-1 / (2 * 25.0 ** 2))


# --------------------------------------------------------------------------
# the calls
# --------------------------------------------------------------------------
def run(state):
    s, kind = state, state["kind"]
    if kind == "me":
        return mb.merit_sad_search(s["plan"], s["cur"], s["ref"])
    if kind == "pool":
        return mb.merit_pool2d(s["plan"], s["x"])
    if kind == "conv":
        if s["packed"] is not None:
            return mb.merit_conv2d_packed(s["plan"], s["x"], s["packed"])
        return mb.merit_conv2d(s["plan"], s["x"], s["w"])
    if kind == "bottleneck":
        (p1, p2, p3), (w1, w2, w3) = s["plans"], s["w"]
        t = mb.merit_conv2d(p2, mb.merit_conv2d(p1, s["x"], w1), w2)
        return mb.merit_conv2d_residual(p3, t, w3, s["x"])
    if kind == "dwsep":
        (p1, p2), (w1, w2) = s["plans"], s["w"]
        return mb.merit_conv2d(p2, mb.merit_conv2d_depthwise(p1, s["x"], w1), w2)
    if kind == "corr":
        return mb.merit_correlation(s["plan"], s["x1"], s["x2"])
    if kind == "sep":
        return mb.merit_sepfilter(s["plan"], s["x"], s["kx"], s["ky"])
    return mb.merit_bilateral(s["plan"], s["x"], s["g"], s["g"], s["norm"])
