"""The plane types at their edges: bytes up to a penalty of 255, two of them
added in a byte up to 127, 16 bits above; the largest penalty is P2, or P1 when
it is the larger one and P2 adapts.  Per direction and as a whole, with stored
costs and (16-bit planes, every direction) with the costs computed from census
words."""
import numpy as np
import pytest

import oracle
from paper_1610_04121_amd import SGM

pytestmark = pytest.mark.gpu


def _pair(seed, W, H):
    rng = np.random.default_rng(seed)
    return tuple(rng.integers(0, 256, (H, W), dtype=np.uint8) for _ in range(2))


def _check(gpu, W, H, D, P, P1, P2, adaptive=False, fused=False, lanes=(0, 0)):
    import torch
    print(f"planes {W}x{H} D={D} P={P} P1={P1} P2={P2} adaptive={adaptive} fused={fused}", flush=True)
    l, r = _pair(W + H + P2 + P1, W, H)
    s = SGM(W, H, D, P1, P2, P, median=True, lrcheck=True, adaptive_p2=adaptive)
    s.set_tuning(*lanes, fused)
    tl, tr = torch.from_numpy(l).to(gpu), torch.from_numpy(r).to(gpu)
    mc = oracle.cost_volume(oracle.census(l), oracle.census(r), D, oracle.cmax_of())
    for k, (rx, ry) in enumerate(oracle.directions(P)):
        got = s.debug_stage(tl, tr, k).cpu().numpy()
        want = oracle.aggregate(mc, P1, P2, rx, ry, img=l) if adaptive else oracle.aggregate(mc, P1, P2, rx, ry)
        bad = np.argwhere(got != want)
        assert len(bad) == 0, f"L_r ({rx},{ry}): {len(bad)} cells differ, first {bad[:5].tolist()}"
    got = s.compute(tl, tr).cpu().numpy()
    s.close()
    assert (got == oracle.sgm(l, r, D, P1, P2, P, median=True, lr=True, adaptive=adaptive).out).all()


@pytest.mark.parametrize("P", [2, 4, 8])
@pytest.mark.parametrize("P1,P2,adaptive", [(7, 127, False), (7, 128, False), (7, 255, False), (7, 256, False),
                                            (127, 40, True), (128, 40, True), (255, 40, True), (256, 40, True)])
def test_penalties_at_the_edges_of_the_plane_types(gpu, P, P1, P2, adaptive):
    _check(gpu, 43, 37, 20, P, P1, P2, adaptive)


@pytest.mark.parametrize("D,P,P2", [(30, 4, 256), (70, 8, 300), (200, 4, 9000), (256, 8, 500), (128, 4, 255), (90, 8, 220)])
def test_census_computing_aggregation_past_byte_planes(gpu, D, P, P2):
    _check(gpu, 61, 41, D, P, 9, P2, fused=True)
    _check(gpu, 61, 41, D, P, 9, P2, fused=True, lanes=(32, 16))
