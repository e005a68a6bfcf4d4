"""Workloads of the SGM pipeline, for timing: what a program has the library
do through its public entry points (``SGM.compute``, ``Batch.compute`` and a
``Server`` request's submit and wait), from the smallest frame to the largest
served one.

``listed()`` gives fixed cases and ``draw(rng)`` more of the same ranges; a
case is a dict of plain values.  ``prepare(case, seed)`` makes device inputs
and the context, batch runner or server; ``run(state)`` makes one pass and
returns the whole disparity maps; ``work(case)`` says how many bytes and
operations a pass cannot do without.

Inputs are seeded synthetic stereo pairs made on the GPU: box-blurred noise
with some low-texture rectangles as the left view, a piecewise-constant
disparity field over a ramp, and the left view warped by it (nearer surfaces
occlude farther ones, holes filled with other texture), darkened and with
sensor noise, as the right view.
"""
from __future__ import annotations

import math
import random

import torch

from paper_1610_04121_amd.sgm import SGM, Batch, Server

# Sizes a camera or a benchmark in this repository has (synth.py): batches
# and served requests draw from these.
BATCH_SIZES = [(320, 240), (640, 480), (1242, 375), (1280, 720)]
SMALL_SIZES = [(160, 120), (200, 150), (240, 180), (320, 240)]
LARGEST_CELLS = 1920 * 1080 * 256 * 8  # cell-paths of the largest listed frame


def _single(name, w, h, d, paths, options, p1=7, p2=86):
    case = dict(kind="single", w=w, h=h, d=d, paths=paths, options=options, p1=p1, p2=p2)
    return dict(name=name, **case) if name else case


def listed():
    return [
        # the smallest call: a thumbnail or a region of interest; launches and
        # one short dependent chain are all there is
        _single("tiny_96x64_d32_p4", 96, 64, 32, 4, "median,lrcheck"),
        # a quarter-VGA preview without post-filters
        _single("small_320x240_d64_p4", 320, 240, 64, 4, ""),
        # the paper's own frame: 640x480, 128 levels, 4 paths
        _single("vga_640x480_d128_p4", 640, 480, 128, 4, "median,lrcheck"),
        # the paper's fastest setting: 2 paths, its center-symmetric census
        _single("vga_2path_csct", 640, 480, 128, 2, "csct,median,lrcheck"),
        # an odd crop with a range that is no power of two, for measuring
        # depth: 8 paths, sub-pixel output
        _single("ragged_451x377_d100_p8", 451, 377, 100, 8, "subpixel,median,lrcheck"),
        # a driving camera's frame at full quality
        _single("drive_1242x375_d128_p8", 1242, 375, 128, 8, "median,lrcheck"),
        # the strict left-right check (a second SGM on the right view)
        _single("vga_lr_full", 640, 480, 128, 4, "lr_full,median,lrcheck"),
        # HD with the penalty that adapts to intensity edges
        _single("hd_adaptive_1280x720_d64_p4", 1280, 720, 64, 4, "adaptive_p2,median,lrcheck"),
        # a large smoothness penalty: aggregated costs need 16 bits
        _single("vga_wide_penalty_p8", 640, 480, 128, 8, "median,lrcheck", 20, 250),
        # the largest served frame: full HD, 256 levels, 8 paths
        _single("fullhd_1920x1080_d256_p8", 1920, 1080, 256, 8, "median,lrcheck"),
        # an offline job: 64 mixed pairs in one batch call
        dict(name="batch64_mixed", kind="batch", pairs=64, mix=11, sizes="mixed"),
        # a burst of small requests to the server, submitted at once
        dict(name="served_burst16_small", kind="served", pairs=16, mix=12, sizes="small"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case: three in five are single frames, the others batches and
    served bursts of up to the listed ones' size."""
    kind = rng.choice(["single", "single", "single", "batch", "served"])
    mix = rng.randrange(1 << 20)
    if kind == "batch":
        return dict(kind=kind, pairs=_log_int(rng, 2, 56), mix=mix, sizes=rng.choice(["mixed", "mixed", "small"]))
    if kind == "served":
        return dict(kind=kind, pairs=_log_int(rng, 2, 32), mix=mix, sizes="small")
    while True:
        w, h = _log_int(rng, 48, 1920), _log_int(rng, 32, 1080)
        d, paths = _log_int(rng, 16, 256), rng.choice([2, 4, 4, 8, 8])
        if 0.4 <= w / h <= 4 and w * h * d * paths <= LARGEST_CELLS // 2:
            break
    options = rng.choice(["", "median", "median,lrcheck", "median,lrcheck", "csct,median,lrcheck",
                          "subpixel,median,lrcheck", "lr_full,median,lrcheck", "adaptive_p2,median,lrcheck"])
    p1, p2 = rng.choice([(7, 86), (7, 86), (7, 86), (10, 120), (20, 250)])
    return _single(None, w, h, d, paths, options, p1, p2)


def _pairs(case):
    """(w, h, d, paths, options) of each pair of a case."""
    if case["kind"] == "single":
        return [(case["w"], case["h"], case["d"], case["paths"], case["options"])]
    rng = random.Random(case["mix"])
    out = []
    for _ in range(case["pairs"]):
        if case["sizes"] == "small":
            w, h = rng.choice(SMALL_SIZES)
            out.append((w, h, rng.choice([32, 64]), 4, "median,lrcheck"))
        else:
            w, h = rng.choice(BATCH_SIZES)
            out.append((w, h, rng.choice([64, 128]), rng.choice([4, 8]), "median,lrcheck"))
    return out


def _flags(options):
    return {o: True for o in options.split(",") if o}


def _texture(w, h, gen):
    u = torch.randint(0, 256, (h + 2, w + 2), generator=gen, device="cuda", dtype=torch.int32)
    s = sum(u[j:j + h, i:i + w] for j in range(3) for i in range(3))
    return (s + 4) // 9


def _stereo_pair(w, h, d, gen, rng):
    """(left, right) u8 [h][w] of one random scene with disparities in [0, d)."""
    dev = "cuda"
    left = _texture(w, h, gen)
    for _ in range(3):  # low-texture rectangles
        rw, rh = max(1, w // rng.randint(5, 12)), max(1, h // rng.randint(5, 12))
        x, y = rng.randint(0, w - rw), rng.randint(0, h - rh)
        left[y:y + rh, x:x + rw] = 128 + torch.randint(-1, 2, (rh, rw), generator=gen, device=dev, dtype=torch.int32)
    ys = torch.arange(h, device=dev)[:, None]
    field = (ys * int(0.6 * d) // max(h, 1)).expand(h, w).clone()
    for _ in range(5):
        rw, rh = max(1, w // rng.randint(3, 9)), max(1, h // rng.randint(3, 8))
        x, y = rng.randint(0, w - rw), rng.randint(0, h - rh)
        field[y:y + rh, x:x + rw] = rng.randint(d // 8, max(d // 8, (d * 7) // 8))
    field = field.clamp(0, d - 1).long()
    # left pixel (x, y) lands on (x - disparity, y); the larger disparity wins
    xt = torch.arange(w, device=dev)[None, :] - field
    ok = xt >= 0
    flat = (ys * w + xt)[ok]
    key = field[ok] * 256 + left[ok].long()
    best = torch.full((h * w,), -1, device=dev, dtype=torch.int64)
    best.scatter_reduce_(0, flat, key, "amax")
    v = torch.where(best >= 0, best % 256, _texture(w, h, gen).long().reshape(-1)).reshape(h, w)
    noise = torch.randint(-3, 4, (h, w), generator=gen, device=dev) + torch.randint(-3, 4, (h, w), generator=gen, device=dev)
    right = (v * 9 // 10 + noise).clamp(0, 255).to(torch.uint8)
    return left.clamp(0, 255).to(torch.uint8).contiguous(), right.contiguous()


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    rng = random.Random(seed)
    pairs = []
    for w, h, d, paths, options in _pairs(case):
        left, right = _stereo_pair(w, h, d, gen, rng)
        pairs.append(dict(left=left, right=right, out=torch.empty((h, w), dtype=torch.uint16, device="cuda"),
                          max_disp=d, n_paths=paths, **_flags(options)))
    state = dict(kind=case["kind"], pairs=pairs)
    if case["kind"] == "single":
        state["handle"] = SGM(case["w"], case["h"], case["d"], P1=case["p1"], P2=case["p2"], n_paths=case["paths"],
                              **_flags(case["options"]))
    elif case["kind"] == "batch":
        state["handle"] = Batch()
    else:
        state["handle"] = Server(1 << 30)
        torch.cuda.synchronize()  # the server's streams do not follow torch's
    return state


def run(state):
    handle, pairs = state["handle"], state["pairs"]
    if state["kind"] == "single":
        return handle.compute(pairs[0]["left"], pairs[0]["right"], out=pairs[0]["out"])
    if state["kind"] == "batch":
        return handle.compute(pairs)
    tickets = [handle.submit(p) for p in pairs]
    for t in tickets:
        handle.wait(t)
    return [p["out"] for p in pairs]


def work(case):
    """Bytes: both images in, the disparity map out.  Operations (integer):
    per cell a 64-bit XOR and popcount, per cell and path the eight of Eq. 3
    (two P1 adds, four minima, the normalization, the cost add), and per cell
    the sum over the paths and two winner-take-all comparisons."""
    b = f = 0
    for w, h, d, paths, options in _pairs(case):
        sgms = 2 if "lr_full" in options else 1
        b += 4 * w * h
        f += sgms * w * h * d * (2 + 8 * paths + paths + 2)
    return {"bytes": b, "flops": f}


def exact(case, seed):
    """Every output is a map of whole numbers, which are compared as they are."""
    return None
