"""The cost volumes of both base images: widths on both sides of a unit (2 or 8
pixels per lane) of every padded range, match columns outside the image in the
first, middle and last levels of a lane, padded levels, and a volume larger
than the memory-side cache."""
import numpy as np
import pytest

import oracle
from paper_1610_04121_amd import SGM, sgm as api

pytestmark = pytest.mark.gpu


def _check(gpu, W, H, D, cw=9, ch=7, csct=False, lr_full=True):
    import torch
    rng = np.random.default_rng(W * 7919 + H * 31 + D)
    l, r = (rng.integers(0, 256, (H, W), dtype=np.uint8) for _ in range(2))
    print(f"cost {W}x{H} D={D} window {cw}x{ch} csct={csct}", flush=True)
    s = SGM(W, H, D, 7, 86, 2, census_w=cw, census_h=ch, csct=csct, lrcheck=lr_full, lr_full=lr_full)
    tl, tr = torch.from_numpy(l).to(gpu), torch.from_numpy(r).to(gpu)
    cl, cr = oracle.census(l, cw, ch, csct), oracle.census(r, cw, ch, csct)
    cmax = oracle.cmax_of(cw, ch, csct)
    maps = [(-1, oracle.cost_volume(cl, cr, D, cmax))]
    if lr_full:
        maps.append((-2, oracle.cost_volume_right(cr, cl, D, cmax)))
    for which, want in maps:
        got = s.debug_stage(tl, tr, which).cpu().numpy()
        bad = np.argwhere(got != want)
        assert len(bad) == 0, f"which={which}: {len(bad)} costs differ, first {bad[:5].tolist()}"
    s.close()


@pytest.mark.parametrize("H", [3, 1030])  # 2 and 8 pixels per lane
@pytest.mark.parametrize("W", [1, 8, 15, 33, 64, 65, 129, 150, 257])
@pytest.mark.parametrize("D", [1, 40, 64, 100, 128, 250, 256])
def test_cost_volumes(gpu, W, H, D):
    _check(gpu, W, H, D)


@pytest.mark.parametrize("W,H,D,cw,ch,csct", [(130, 9, 100, 5, 5, False), (75, 20, 64, 9, 7, True), (70, 30, 256, 3, 3, True)])
def test_cost_volumes_of_other_windows(gpu, W, H, D, cw, ch, csct):
    _check(gpu, W, H, D, cw, ch, csct)


def test_cost_volume_above_the_cache(gpu):
    assert 1055 * 1001 * 256 > 256 << 20
    _check(gpu, 1055, 1001, 250, lr_full=False)


def test_batch_above_the_cache(gpu):
    """Two units per wavefront and non-temporal stores in the batched launch."""
    import torch
    rng = np.random.default_rng(11)
    shapes = [(641, 430, 256, {}), (500, 401, 200, dict(lr_full=True)), (77, 1000, 128, {}), (900, 500, 250, {})]
    assert sum(W * H * 256 * (2 if o else 1) for W, H, D, o in shapes if D > 128) > 256 << 20
    b = api.Batch(P1=7, P2=86)
    items, pairs = [], []
    for W, H, D, o in shapes:
        l, r = (rng.integers(0, 256, (H, W), dtype=np.uint8) for _ in range(2))
        pairs.append((l, r))
        items.append(dict(left=torch.from_numpy(l).to(gpu), right=torch.from_numpy(r).to(gpu),
                          out=torch.empty((H, W), dtype=torch.uint16, device=gpu), max_disp=D, n_paths=2, lrcheck=True, **o))
    got = [o.cpu().numpy() for o in b.compute(items)]
    b.close()
    for (W, H, D, o), (l, r), g in zip(shapes, pairs, got):
        print(f"batch {W}x{H} D={D} {o}", flush=True)
        want = oracle.sgm(l, r, D, 7, 86, 2, lr=True, lr_full=bool(o)).out
        assert (g == want).all(), f"{W}x{H}: {(g != want).sum()} pixels differ"
