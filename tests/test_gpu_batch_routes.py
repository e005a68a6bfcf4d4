"""The two ways a batch sums and takes winners: one winner-take-all launch over
whole planes up to a number of plane bytes, and the row kernel, one launch per
kernel variant (padded range, path count, plane type and sub-pixel option),
above.  The line is 12 MiB for one variant with 64 levels, 40 MiB with more, and
72 MiB more for each further variant.  Batches on both sides of it, with every
option; the row kernel's widths beside a pair that is large enough for it; and
the two pixel counts of the cost launch."""
import numpy as np
import pytest

import oracle
from paper_1610_04121_amd import sgm as api

pytestmark = pytest.mark.gpu

LARGE = 72 << 20  # above the line of one variant
WIDTHS = [1, 2, 7, 8, 9, 15, 16, 17, 31, 33, 63, 64, 65, 127, 130, 257, 530]


def _padded(D):
    return 64 if D <= 64 else 128 if D <= 128 else 256


def _pair(rng, W, H):
    return tuple(rng.integers(0, 256, (H, W), dtype=np.uint8) for _ in range(2))


def _item(gpu, l, r, D, P, **opts):
    import torch
    return dict(left=torch.from_numpy(l).to(gpu), right=torch.from_numpy(r).to(gpu),
                out=torch.empty(l.shape, dtype=torch.uint16, device=gpu), max_disp=D, n_paths=P, **opts)


def _want(l, r, D, P, P1, P2, opts):
    return oracle.sgm(l, r, D, P1, P2, P, median=opts.get("median", False), lr=opts.get("lrcheck", False),
                      lr_full=opts.get("lr_full", False), subpixel=opts.get("subpixel", False),
                      adaptive=opts.get("adaptive_p2", False), csct=opts.get("csct", False)).out


def _run(gpu, shapes, P1, P2, seed, compare=None):
    """shapes: (W, H, D, P, options); compares all of them, or the first `compare`."""
    rng = np.random.default_rng(seed)
    imgs = [_pair(rng, W, H) for W, H, *_ in shapes]
    b = api.Batch(P1=P1, P2=P2)
    got = [o.cpu().numpy() for o in b.compute([_item(gpu, l, r, D, P, **o) for (l, r), (_, _, D, P, o) in zip(imgs, shapes)])]
    b.close()
    for (W, H, D, P, o), (l, r), g in list(zip(shapes, imgs, got))[:compare]:
        n = int((g != _want(l, r, D, P, P1, P2, o)).sum())
        assert n == 0, f"{W}x{H} D={D} P={P} {o}: {n} pixels differ"


OPTIONS = [{}, dict(median=True, lrcheck=True), dict(subpixel=True, lrcheck=True), dict(lr_full=True, lrcheck=True),
           dict(adaptive_p2=True), dict(csct=True, median=True), dict(lr_full=True, lrcheck=True, subpixel=True)]


@pytest.mark.parametrize("P1,P2", [(7, 86), (3, 127), (3, 128), (20, 255), (20, 256), (300, 40)])
def test_small_mixed_batch(gpu, P1, P2):
    """Every range and path count with every option in one winner-take-all launch."""
    print(f"small mixed batch P1={P1} P2={P2}", flush=True)
    shapes = [(30 + 7 * i, 9 + i, D, P, OPTIONS[(i + k) % len(OPTIONS)])
              for i, D in enumerate((20, 64, 100, 128, 200, 256)) for k, P in enumerate((2, 4, 8))]
    _run(gpu, shapes, P1, P2, P2)


FULL = dict(lr_full=True, lrcheck=True)


@pytest.mark.parametrize("shapes,P2,mib", [
    ([(256, 192, 64, 4, dict(lrcheck=True))], 86, 12), ([(257, 192, 64, 4, dict(lrcheck=True))], 86, 12),  # at the line, past it
    ([(256, 160, 100, 4, FULL)], 86, 40), ([(257, 160, 100, 2, FULL)], 300, 40),
    ([(512, 256, 128, 4, {}), (512, 384, 50, 4, {})], 86, 112), ([(513, 256, 128, 4, {}), (512, 384, 50, 4, {})], 86, 112),
])
def test_line_between_the_routes(gpu, shapes, P2, mib):
    planes = sum(W * H * _padded(D) * P * (2 if P2 > 255 else 1) * (2 if o.get("lr_full") else 1) for W, H, D, P, o in shapes)
    assert 0 <= planes - (mib << 20) < 1 << 18
    print(f"line {shapes} P2={P2}: {planes - (mib << 20):+d} bytes", flush=True)
    _run(gpu, shapes, 7, P2, shapes[0][0])


@pytest.mark.parametrize("opts", [{}, dict(lrcheck=True, median=True), dict(lrcheck=True, subpixel=True),
                                  dict(lrcheck=True, lr_full=True, adaptive_p2=True)])
@pytest.mark.parametrize("P1,P2", [(7, 127), (7, 128), (20, 255), (10, 256)])
@pytest.mark.parametrize("D,P", [(40, 2), (64, 8), (100, 4), (128, 8), (140, 2), (256, 4), (250, 8)])
def test_row_kernel_widths_beside_a_large_pair(gpu, D, P, P1, P2, opts):
    print(f"row kernel D={D} P={P} P1={P1} P2={P2} {opts}", flush=True)
    W = 640
    large = (W, LARGE // (W * _padded(D) * P) + 1, D, P, opts)
    # (the large pair is there for the route; smaller tests cover its kind)
    _run(gpu, [(w, 3 + k % 4, D, P, opts) for k, w in enumerate(WIDTHS)] + [large], P1, P2, D + P, compare=len(WIDTHS))


@pytest.mark.parametrize("H", [1024, 1025])  # the last launch with 2 pixels a lane, the first with 8
def test_cost_launch_pixels(gpu, H):
    print(f"cost launch 32x{H}", flush=True)
    _run(gpu, [(32, H, 250, 2, dict(lrcheck=True))], 7, 86, H)
    _run(gpu, [(7, 5, 256, 2, {}), (65, 9, 60, 4, dict(lr_full=True, lrcheck=True)), (33, 4, 128, 2, {})], 7, 86, H)


def test_widest_pair_by_both_routes(gpu):
    """16000 columns with the right view: the keys of a row and the row
    kernel's penalty table together are 64 KiB of LDS."""
    for H, D in ((3, 128), (10, 256)):
        assert (16000 * H * _padded(D) * 2 > LARGE) == (H == 10)
        print(f"widest pair 16000x{H} D={D}", flush=True)
        _run(gpu, [(16000, H, D, 2, dict(lrcheck=True, median=True))], 7, 86, H)


def test_widest_frame_in_the_row_kernel(gpu):
    import torch
    W, H, D = 16000, 10, 256
    assert W * H * D * 2 > LARGE
    print(f"widest frame {W}x{H} D={D}", flush=True)
    l, r = _pair(np.random.default_rng(5), W, H)
    s = api.SGM(W, H, D, 7, 86, 2, lrcheck=True)
    got = s.compute(torch.from_numpy(l).to(gpu), torch.from_numpy(r).to(gpu)).cpu().numpy()
    s.close()
    assert (got == _want(l, r, D, 2, 7, 86, dict(lrcheck=True))).all()
