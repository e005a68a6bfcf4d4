"""The row kernel (both horizontal directions run again inside segments of 8
or 16 columns, the sum and the winner-take-all): widths on both sides of one
segment, of a wavefront's four (or two) and of a workgroup's, every padded
range, plane type (two values to a byte, one, 16 bits) and path count.  Batches
always take it, single frames above a size."""
import numpy as np
import pytest

import oracle
from paper_1610_04121_amd import SGM, sgm as api

pytestmark = pytest.mark.gpu

WIDTHS = [1, 2, 7, 8, 9, 15, 16, 17, 31, 33, 63, 64, 65, 127, 130, 257, 530]


def _pair(rng, W, H):
    return tuple(rng.integers(0, 256, (H, W), dtype=np.uint8) for _ in range(2))


@pytest.mark.parametrize("opts", [{}, dict(lrcheck=True, median=True), dict(lrcheck=True, subpixel=True),
                                  dict(lrcheck=True, lr_full=True, adaptive_p2=True)])
@pytest.mark.parametrize("P1,P2", [(7, 86), (20, 250), (10, 300)])
@pytest.mark.parametrize("D,P", [(40, 2), (64, 8), (100, 4), (128, 8), (140, 2), (256, 4), (250, 8)])
def test_row_kernel_widths(gpu, D, P, P1, P2, opts):
    import torch
    rng = np.random.default_rng(D * 131 + P * 17 + P2)
    print(f"row kernel D={D} P={P} P1={P1} P2={P2} {opts}", flush=True)
    b = api.Batch(P1=P1, P2=P2)
    items, imgs = [], []
    for k, W in enumerate(WIDTHS):
        H = 3 + k % 4
        l, r = _pair(rng, W, H)
        imgs.append((l, r))
        items.append(dict(left=torch.from_numpy(l).to(gpu), right=torch.from_numpy(r).to(gpu),
                          out=torch.empty((H, W), dtype=torch.uint16, device=gpu), max_disp=D, n_paths=P, **opts))
    got = [o.cpu().numpy() for o in b.compute(items)]
    b.close()
    for W, (l, r), g in zip(WIDTHS, imgs, got):
        want = oracle.sgm(l, r, D, P1, P2, P, median=opts.get("median", False), lr=opts.get("lrcheck", False),
                          lr_full=opts.get("lr_full", False), subpixel=opts.get("subpixel", False),
                          adaptive=opts.get("adaptive_p2", False)).out
        assert (g == want).all(), f"W={W}: {(g != want).sum()} pixels differ"


@pytest.mark.parametrize("W,H,D,P,opts", [
    (61, 650, 256, 8, dict(lrcheck=True)), (643, 235, 128, 4, dict(lrcheck=True, median=True)),
    (150, 1300, 200, 2, dict(subpixel=True, lrcheck=True)), (530, 150, 128, 8, dict(adaptive_p2=True, lrcheck=True)),
    (330, 470, 64, 8, dict(lr_full=True, lrcheck=True)),
])
def test_row_kernel_single_frame(gpu, W, H, D, P, opts):
    """Frames just above the size from which a context uses the row kernel."""
    import torch
    l, r = _pair(np.random.default_rng(W + H), W, H)
    assert W * H * (64 if D <= 64 else 128 if D <= 128 else 256) * P > 72 << 20
    print(f"row kernel, one frame {W}x{H} D={D} P={P} {opts}", flush=True)
    s = SGM(W, H, D, 7, 86, P, **opts)
    got = s.compute(torch.from_numpy(l).to(gpu), torch.from_numpy(r).to(gpu)).cpu().numpy()
    s.close()
    want = oracle.sgm(l, r, D, 7, 86, P, lr=True, median=opts.get("median", False), lr_full=opts.get("lr_full", False),
                      subpixel=opts.get("subpixel", False), adaptive=opts.get("adaptive_p2", False)).out
    assert (got == want).all(), f"{(got != want).sum()} pixels differ"
