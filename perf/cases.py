"""The work a user of this library has it do, as cases to time and compare.

Every case is one call (or one chain of calls) of the public entry points on
seeded synthetic stereo scenes: textured regions of different mean lightness
and disparity over a textured background, the right image a z-buffered warp of
the left one. Kinds:

  sad          one frame's disparity search (``sad_disparity``)
  batch        many frames in one persistent launch (``BatchRunner.run``)
  front        the boundary list of one frame, cut to a fraction (``boundaries``)
  front_paper  the same in the paper's setting: K = 10, fill/remove, 4% rule
  reconstruct  dense disparity map from the listed pixels (``reconstruct``)
  blur         selective Gaussian blur by depth (``selective_blur``)
  chain        raw pair to blurred image (``pipeline.depth_blur``)

Lists come from the front end itself (``boundaries`` with fraction control),
as in serving and in the video benchmark; building them is not part of a pass.
"""
from __future__ import annotations

import math

import torch

import paper_2001_07809_amd as sbs
from paper_2001_07809_amd import pipeline

SERVE_CLASSES = (  # width, height, block, dmax, regions of the request classes
    (640, 480, 11, 31, 10),
    (1920, 1080, 21, 63, 20),
    (4096, 2304, 31, 127, 40),
)


def listed():
    return [
        # The smallest search: the Middlebury Tsukuba shape, grey. Launches and
        # latency are most of it.
        dict(name="sad_tsukuba_gray", kind="sad", W=384, H=288, C=1, block=15, dmax=15, regions=6, frac=0.18,
             shuffled=False),
        # A list that is not in raster order (a caller's own pixel list) on the
        # small serving class: the pixel-map path of the search.
        dict(name="sad_vga_rgb_shuffled", kind="sad", W=640, H=480, C=3, block=11, dmax=31, regions=10, frac=0.18,
             shuffled=True),
        # An ordinary still: full-size Middlebury shape, RGB, rows of 4170
        # bytes (not a multiple of 4).
        dict(name="sad_middlebury_rgb", kind="sad", W=1390, H=1110, C=3, block=21, dmax=63, regions=20, frac=0.18,
             shuffled=False),
        # One frame of the paper's video size, searched on its own.
        dict(name="sad_uhd_rgb", kind="sad", W=4096, H=2304, C=3, block=31, dmax=127, regions=40, frac=0.18,
             shuffled=False),
        # The benchmark's video step, 24 of its 250 frames: the throughput case.
        dict(name="batch_uhd_video", kind="batch", mix="same", W=4096, H=2304, C=3, block=31, dmax=127, regions=40,
             frames=24),
        # One group that the server admits: the three request classes, 5:3:2.
        dict(name="batch_serving_mix", kind="batch", mix="serving", W=4096, H=2304, C=3, block=31, dmax=127,
             regions=40, frames=10),
        # A raw request of the small serving class gets its list (launches and
        # latency count), and one frame of the video size does.
        dict(name="front_vga_rgb", kind="front", W=640, H=480, C=3, regions=10, frac=0.18),
        dict(name="front_uhd_rgb", kind="front", W=4096, H=2304, C=3, regions=40, frac=0.18),
        # The paper's own front end on a grey full-size Middlebury shape.
        dict(name="front_paper_middlebury", kind="front_paper", W=1390, H=1110, C=1, regions=60),
        # The two steps after the search at the video size.
        dict(name="reconstruct_uhd", kind="reconstruct", W=4096, H=2304, regions=40, dmax=127, frac=0.18,
             threshold=1),
        dict(name="blur_uhd_rgb", kind="blur", W=4096, H=2304, C=3, regions=40, dmax=127, sigma=2.0),
        # The whole method on a colour still, in the paper's Table 3 setting.
        dict(name="chain_middlebury_rgb", kind="chain", W=1390, H=1110, C=3, block=9, dmax=63, regions=60),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng):
    """A frame between 384x288 and 4096x2304, odd sizes among them."""
    W = min(4096, max(384, _log_int(rng, 384, 4096)))
    H = min(2304, max(288, int(W * rng.uniform(0.55, 0.78))))
    if rng.random() < 0.5:   # camera sizes are mostly multiples of 8
        W, H = W // 8 * 8, H // 8 * 8
    return W, H


def _search(rng, W):
    """Block and largest disparity of the workloads at about this width."""
    t = math.log(W / 384) / math.log(4096 / 384)
    block = 2 * int(round((9 + 22 * t + rng.uniform(-2, 6)) / 2)) + 1
    dmax = int(round(2 ** (4 + 3 * t + rng.uniform(-0.5, 0.5)))) - 1
    return min(31, max(9, block)), min(127, max(15, dmax))


def draw(rng):
    kind = rng.choice(["sad", "sad", "sad", "batch", "batch", "front", "front", "front_paper", "reconstruct", "blur",
                       "chain"])
    W, H = _size(rng)
    C = rng.choice([1, 3, 3])
    block, dmax = _search(rng, W)
    regions = rng.randint(6, 60)
    if kind == "sad":
        return dict(kind=kind, W=W, H=H, C=C, block=block, dmax=dmax, regions=regions, frac=rng.uniform(0.12, 0.24),
                    shuffled=rng.random() < 0.2)
    if kind == "batch":
        if rng.random() < 0.3:
            return dict(kind=kind, mix="serving", W=4096, H=2304, C=3, block=31, dmax=127, regions=40,
                        frames=rng.randint(3, 20))
        return dict(kind=kind, mix="same", W=W, H=H, C=C, block=block, dmax=dmax, regions=regions,
                    frames=_log_int(rng, 2, 24))
    if kind == "front":
        return dict(kind=kind, W=W, H=H, C=C, regions=regions, frac=rng.uniform(0.12, 0.24))
    if kind == "front_paper":
        return dict(kind=kind, W=W, H=H, C=C, regions=regions)
    if kind == "reconstruct":
        return dict(kind=kind, W=W, H=H, regions=regions, dmax=dmax, frac=rng.uniform(0.12, 0.24),
                    threshold=rng.choice([0, 1]))
    if kind == "blur":
        return dict(kind=kind, W=W, H=H, C=C, regions=regions, dmax=dmax, sigma=rng.choice([1.0, 1.5, 2.0, 3.0, 4.5]))
    return dict(kind="chain", W=W, H=H, C=C, block=9, dmax=dmax, regions=regions)


# ---------------------------------------------------------------------------
# Scenes

def _smoothed_noise(W, H, C, gen):
    """u8 noise under a 3x3 box, [H, W, C] float holding whole numbers."""
    n = torch.randint(0, 256, (C, 1, H, W), generator=gen, device="cuda", dtype=torch.int32).float()
    t = torch.nn.functional.avg_pool2d(n, 3, 1, 1, count_include_pad=False)
    return t.floor_().squeeze(1).permute(1, 2, 0)


def _scene(W, H, C, regions, dmax, seed):
    """Left and right u8 images ([H, W] or [H, W, 3]) and the disparity map."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    cpu = torch.Generator()
    cpu.manual_seed(seed)

    def uniform(lo, hi):   # whole number in [lo, hi]
        return int(torch.randint(lo, hi + 1, (1,), generator=cpu))

    disp = torch.zeros(H, W, dtype=torch.int32, device="cuda")
    mean = torch.full((H, W), 128.0, device="cuda")
    # regions behind first; background disparity 0
    for d in sorted(uniform(0, dmax) for _ in range(regions)):
        w, h = uniform(max(W // 16, 2), W // 4), uniform(max(H // 16, 2), H // 4)
        cx, cy, mu = uniform(0, W - 1), uniform(0, H - 1), uniform(30, 225)
        x0, x1, y0, y1 = max(cx - w // 2, 0), min(cx + w // 2, W), max(cy - h // 2, 0), min(cy + h // 2, H)
        if x1 <= x0 or y1 <= y0:
            continue
        dv, mv = disp[y0:y1, x0:x1], mean[y0:y1, x0:x1]
        if uniform(0, 1):   # ellipse
            yy = (torch.arange(y0, y1, device="cuda").float() - cy).div_(h / 2).square_()
            xx = (torch.arange(x0, x1, device="cuda").float() - cx).div_(w / 2).square_()
            inside = yy[:, None] + xx[None, :] <= 1.0
            dv.masked_fill_(inside, d)
            mv.masked_fill_(inside, float(mu))
        else:
            dv.fill_(d)
            mv.fill_(float(mu))
    left = _smoothed_noise(W, H, C, gen).sub_(128.0).div_(2.0).floor_().add_(mean[:, :, None]).clamp_(0, 255)
    left = left.to(torch.uint8)
    # z-buffered warp: the nearest (largest disparity) left pixel of each right pixel
    packed = torch.zeros(H, W, dtype=torch.int32, device="cuda")
    for c in range(C):
        packed |= left[:, :, c].to(torch.int32) << (8 * c)
    x = torch.arange(W, device="cuda")[None, :] - disp
    to = (torch.arange(H, device="cuda")[:, None] * W + x.clamp_min(0)).reshape(-1)
    key = torch.where(x >= 0, packed | (disp << 24), -1).reshape(-1)
    hit = torch.full((H * W,), -1, dtype=torch.int32, device="cuda")
    hit.scatter_reduce_(0, to, key, "amax")
    hit = hit.view(H, W)
    right = _smoothed_noise(W, H, C, gen).to(torch.uint8)
    for c in range(C):
        right[:, :, c] = torch.where(hit >= 0, ((hit >> (8 * c)) & 255).to(torch.uint8), right[:, :, c])
    if C == 1:
        left, right = left[:, :, 0], right[:, :, 0]
    return left.contiguous(), right.contiguous(), disp.to(torch.uint8)


def _search_inputs(W, H, C, block, dmax, regions, frac, seed):
    left, right, _ = _scene(W, H, C, regions, dmax, seed)
    idx = sbs.boundaries(left, K=4, frac=frac, seed=seed).clone()
    return left, right, idx, block, dmax


def _batch_frames(case, seed):
    """(W, H, block, dmax, regions, fraction, seed) of each frame of a batch."""
    out = []
    for t in range(case["frames"]):
        frac = 0.12 + 0.12 * ((0.618 * t + 0.3) % 1.0)   # spread over the workloads' 12-24%, alike for every seed
        if case["mix"] == "serving":
            k = (0, 1, 0, 2, 0, 1, 0, 2, 0, 1)[t % 10]
            W, H, block, dmax, regions = SERVE_CLASSES[k]
        else:
            W, H, block, dmax, regions = (case[k] for k in ("W", "H", "block", "dmax", "regions"))
        out.append((W, H, block, dmax, regions, frac, seed * 1000 + t))
    return out


# ---------------------------------------------------------------------------

def prepare(case, seed):
    kind, W, H = case["kind"], case["W"], case["H"]
    state = dict(case=case, seed=seed)
    if kind == "sad":
        f = _search_inputs(W, H, case["C"], case["block"], case["dmax"], case["regions"], case["frac"], seed)
        if case["shuffled"]:
            gen = torch.Generator(device="cuda")
            gen.manual_seed(seed)
            order = torch.randperm(f[2].numel(), generator=gen, device="cuda")
            f = (f[0], f[1], f[2][order].contiguous(), f[3], f[4])
        state["frame"] = f
    elif kind == "batch":
        frames = [_search_inputs(w, h, case["C"], b, d, r, frac, s)
                  for (w, h, b, d, r, frac, s) in _batch_frames(case, seed)]
        state["runner"] = sbs.BatchRunner(frames)
    elif kind in ("front", "front_paper", "chain"):
        left, right, _ = _scene(W, H, case["C"], case["regions"], case.get("dmax", 63), seed)
        state["left"], state["right"] = left, right
        if kind == "chain":
            state["params"] = pipeline.PaperParams(block=case["block"], dmax=case["dmax"], threshold=1,
                                                   ranges=((0, case["dmax"] // 2),))
    elif kind == "reconstruct":
        left, _, disp = _scene(W, H, 3, case["regions"], case["dmax"], seed)
        idx = sbs.boundaries(left, K=4, frac=case["frac"], seed=seed).clone()
        state["idx"], state["disp"] = idx, disp.view(-1)[idx.long()].contiguous()
    else:
        left, _, disp = _scene(W, H, case["C"], case["regions"], case["dmax"], seed)
        state["left"], state["depth"] = left, disp
    return state


def _record(t, n):
    """A list of data-dependent length as a fixed-size record (n entries, -1 or 255 past the end)."""
    return torch.nn.functional.pad(t, (0, n - t.numel()), value=255 if t.dtype == torch.uint8 else -1)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "sad":
        return sbs.sad_disparity(*state["frame"])
    if kind == "batch":
        runner = state["runner"]
        runner.run()
        return [runner.disp, runner.cost]
    if kind == "front":
        return sbs.boundaries(state["left"], K=4, mode=0, min_cc=50, frac=case["frac"], seed=state["seed"])
    if kind == "front_paper":
        return _record(sbs.boundaries(state["left"], K=10, mode=1), case["W"] * case["H"])
    if kind == "reconstruct":
        return sbs.reconstruct(state["idx"], state["disp"], case["W"], case["H"], case["threshold"])
    if kind == "blur":
        return sbs.selective_blur(state["left"], state["depth"], ((0, case["dmax"] // 2),), case["sigma"])
    out = pipeline.depth_blur(state["left"], state["right"], state["params"])
    for k in ("list", "disp", "cost"):
        out[k] = _record(out[k], case["W"] * case["H"])
    return out


def _search_work(W, H, C, dmax, n):
    # column sums: per image pixel and disparity one absolute difference for
    # the row entering the window and one for the row leaving it, one add and
    # one subtract along the row; one comparison per listed pixel and disparity
    return 2 * W * H * C + 9 * n, (4 * W * H + n) * (dmax + 1)


def work(case):
    kind, W, H, C = case["kind"], case["W"], case["H"], case.get("C", 1)
    N = W * H
    if kind == "sad":
        b, f = _search_work(W, H, C, case["dmax"], round(case["frac"] * N))
    elif kind == "batch":
        b = f = 0
        for (w, h, _, d, _, _, _) in _batch_frames(case, 1):
            fb, ff = _search_work(w, h, C, d, round(0.18 * w * h))   # fractions average 0.18
            b, f = b + fb, f + ff
    elif kind in ("front", "front_paper"):
        # image in, list out; about 40 operations per pixel: luminance, five
        # 3x3 steps (separable), the component merge
        b, f = N * C + 4 * round(case.get("frac", 0.18) * N), 40 * N
    elif kind == "reconstruct":
        b, f = 5 * round(case["frac"] * N) + N, 4 * N
    elif kind == "blur":
        b, f = N * C + N + 4 * N * C, 2 * 2 * (2 * math.ceil(3 * case["sigma"]) + 1) * C * N
    else:
        # a pair in; both lightness images, list, disparities, costs, depth and
        # the blurred image out; the paper's refinement keeps about 18%
        n = round(0.18 * N)
        b = 2 * N * C + 2 * N + 9 * n + N + 4 * N * C
        f = _search_work(W, H, 1, case["dmax"], n)[1] + 40 * N + 2 * 2 * 13 * C * N
    return {"bytes": b, "flops": f}


def exact(case, seed):
    """The blurred image in 64 bits. The other kinds return whole numbers."""
    if case["kind"] != "blur":
        return None
    s = prepare(case, seed)
    rad = math.ceil(3.0 * case["sigma"])
    g = torch.arange(-rad, rad + 1, device="cuda", dtype=torch.float64)
    g = torch.exp(-g * g / (2.0 * case["sigma"] ** 2))
    g /= g.sum()
    img = s["left"].double()
    H, W = case["H"], case["W"]
    x, y = torch.arange(W, device="cuda"), torch.arange(H, device="cuda")
    rows = sum(g[k + rad] * img[:, (x + k).clamp(0, W - 1)] for k in range(-rad, rad + 1))
    full = sum(g[k + rad] * rows[(y + k).clamp(0, H - 1)] for k in range(-rad, rad + 1))
    keep = s["depth"] <= case["dmax"] // 2   # the range starts at 0
    return torch.where(keep if img.dim() == 2 else keep[:, :, None], img, full)
