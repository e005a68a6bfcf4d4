"""The right-to-left walk that stores checkpoints: it begins so that its blocks
end at multiples of a segment, with a lead-in of repeated first columns when
the width is no multiple of one, and the path starts after the lead-in.  With
16 levels per lane a block is 8 steps and a segment 16, so widths of 8 modulo
16 have a lead-in of one whole block.  Unrelated noise, on which a path
remembers its start for hundreds of columns."""
import numpy as np
import pytest

import oracle
from paper_1610_04121_amd import SGM, sgm as api

pytestmark = pytest.mark.gpu


def _pair(W, H):
    rng = np.random.default_rng(W * 131 + H)
    return tuple(rng.integers(0, 256, (H, W), dtype=np.uint8) for _ in range(2))


def _item(gpu, l, r, D, P, **opts):
    import torch
    return dict(left=torch.from_numpy(l).to(gpu), right=torch.from_numpy(r).to(gpu),
                out=torch.empty(l.shape, dtype=torch.uint16, device=gpu), max_disp=D, n_paths=P, **opts)


def _want(l, r, D, P, P1=7, P2=86, **opts):
    return oracle.sgm(l, r, D, P1, P2, P, lr=opts.get("lrcheck", False), lr_full=opts.get("lr_full", False),
                      adaptive=opts.get("adaptive_p2", False)).out


# every width modulo 16, on both sides of two blocks, and the class's larger ones
WIDTHS = [*range(24, 42), 56, 200, 600]


@pytest.mark.parametrize("opts", [{}, dict(adaptive_p2=True), dict(lrcheck=True, lr_full=True)])
@pytest.mark.parametrize("D,P,P2", [(130, 4, 86), (200, 8, 86), (256, 4, 86), (256, 4, 300), (100, 4, 86)])
def test_right_to_left_path_starts_in_a_batch(gpu, D, P, P2, opts):
    print(f"checkpoints, batch D={D} P={P} P2={P2} {opts}", flush=True)
    pairs = [_pair(W, 12 if W < 100 else 21) for W in WIDTHS]
    # a pair that makes the batch large enough for checkpoints
    pairs.append(_pair(640, (72 << 20) // (640 * (128 if D <= 128 else 256) * P) + 1))
    b = api.Batch(P1=7, P2=P2)
    b.set_tuning(16, 16)
    got = [o.cpu().numpy() for o in b.compute([_item(gpu, l, r, D, P, **opts) for l, r in pairs])]
    b.close()
    bad = [(l.shape[1], int((g != _want(l, r, D, P, P2=P2, **opts)).sum())) for (l, r), g in zip(pairs[:-1], got)]
    assert not any(n for _, n in bad), f"(width, pixels that differ): {[b for b in bad if b[1]]}"


@pytest.mark.parametrize("W,H,D,P,lanes,opts", [
    (1000, 600, 200, 4, (0, 0), {}),                        # the default shape
    (200, 371, 256, 4, (16, 16), {}), (88, 500, 256, 8, (16, 16), dict(adaptive_p2=True)),
    (8008, 10, 256, 4, (16, 16), {}), (2504, 31, 130, 4, (16, 16), dict(lrcheck=True, lr_full=True)),  # long slices, in segments
])
def test_right_to_left_path_starts_in_a_frame(gpu, W, H, D, P, lanes, opts):
    import torch
    assert W * H * 256 * P > 72 << 20
    print(f"checkpoints, frame {W}x{H} D={D} P={P} lanes={lanes} {opts}", flush=True)
    l, r = _pair(W, H)
    s = SGM(W, H, D, 7, 86, P, **opts)
    s.set_tuning(*lanes)
    got = s.compute(torch.from_numpy(l).to(gpu), torch.from_numpy(r).to(gpu)).cpu().numpy()
    s.close()
    n = int((got != _want(l, r, D, P, **opts)).sum())
    assert n == 0, f"{n} pixels differ"


def test_right_to_left_path_starts_in_a_batch_of_default_shape(gpu):
    """Enough wavefronts for 16 lanes without a tuning."""
    print("checkpoints, batch of the default shape", flush=True)
    W, H, D, P = 600, 480, 200, 8
    assert 2 * (H // 4) + 6 * (W // 4) > 1024
    l, r = _pair(W, H)
    b = api.Batch(P1=7, P2=86)
    got = b.compute([_item(gpu, l, r, D, P)])[0].cpu().numpy()
    b.close()
    n = int((got != _want(l, r, D, P)).sum())
    assert n == 0, f"{n} pixels differ"
