"""Slices walked in segments by several wavefronts (long slices of frames too
small to fill the device, 2 and 4 paths): every direction's L_r and the
disparities must be the ones of the whole walk, on images where the segments'
values meet after a few steps (a shifted copy), at once (flat) and never or
late (unrelated noise), with segments of one block, of many and none at the
end, and with the horizontal directions' checkpoints (the 64-, 128-level
frames above 72 Mi cell-paths)."""
import numpy as np
import pytest

import oracle
from paper_1610_04121_amd import SGM

pytestmark = pytest.mark.gpu


def _pair(kind, W, H):
    rng = np.random.default_rng(W * 1013 + H)
    if kind == "flat":
        return np.full((H, W), 90, np.uint8), np.full((H, W), 90, np.uint8)
    l = rng.integers(0, 256, (H, W), dtype=np.uint8)
    if kind == "noise":
        return l, rng.integers(0, 256, (H, W), dtype=np.uint8)
    return l, np.roll(l, -5, axis=1)


@pytest.mark.parametrize("kind", ["shifted", "noise", "flat"])
@pytest.mark.parametrize("P,adaptive,lanes", [(4, False, (0, 0)), (4, True, (16, 16)), (2, False, (64, 32)),
                                              (4, False, (32, 32))])
@pytest.mark.parametrize("W,H,D", [(160, 21, 40), (161, 8, 128), (255, 64, 100), (19, 177, 64), (5, 320, 128),
                                   (600, 3, 256), (330, 40, 200), (1, 200, 64), (500, 400, 64)])
def test_segments_per_direction(gpu, W, H, D, P, adaptive, lanes, kind):
    import torch
    l, r = _pair(kind, W, H)
    print(f"segments {W}x{H} D={D} P={P} adaptive={adaptive} lanes={lanes} {kind}", flush=True)
    s = SGM(W, H, D, 7, 86, P, adaptive_p2=adaptive)
    s.set_tuning(*lanes)
    tl, tr = torch.from_numpy(l).to(gpu), torch.from_numpy(r).to(gpu)
    mc = oracle.cost_volume(oracle.census(l), oracle.census(r), D, oracle.cmax_of())
    for k, (rx, ry) in enumerate(oracle.directions(P)):
        got = s.debug_stage(tl, tr, k).cpu().numpy()
        want = oracle.aggregate(mc, 7, 86, rx, ry, img=l) if adaptive else oracle.aggregate(mc, 7, 86, rx, ry)
        bad = np.argwhere(got != want)
        assert len(bad) == 0, f"L_r ({rx},{ry}): {len(bad)} cells differ, first {bad[:5].tolist()}"
    s.close()


@pytest.mark.parametrize("kind", ["shifted", "noise"])
@pytest.mark.parametrize("W,H,D,P,opts", [
    (320, 120, 64, 4, {}), (200, 90, 128, 2, dict(subpixel=True)), (400, 60, 100, 4, dict(lr_full=True)),
    (640, 230, 128, 4, {}), (1001, 299, 128, 4, {}), (8003, 37, 64, 4, {}), (41, 4700, 128, 4, dict(adaptive_p2=True)), (5001, 61, 128, 2, dict(lr_full=True)),
])
def test_segments_frames(gpu, W, H, D, P, opts, kind):
    import torch
    l, r = _pair(kind, W, H)
    print(f"segments, frame {W}x{H} D={D} P={P} {opts} {kind}", flush=True)
    s = SGM(W, H, D, 7, 86, P, lrcheck=True, **opts)
    got = s.compute(torch.from_numpy(l).to(gpu), torch.from_numpy(r).to(gpu)).cpu().numpy()
    s.close()
    want = oracle.sgm(l, r, D, 7, 86, P, lr=True, lr_full=opts.get("lr_full", False),
                      subpixel=opts.get("subpixel", False), adaptive=opts.get("adaptive_p2", False)).out
    assert (got == want).all(), f"{(got != want).sum()} pixels differ"
