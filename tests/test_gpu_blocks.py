"""The blocks of an aggregation walk: a slice is walked in blocks of 8 or 16
steps, the inner ones with shared addresses and the ones at the slice's end or
(diagonals) around a border crossing in a general form.  Slice lengths and
widths here sit on both sides of one, two and three blocks."""
import numpy as np
import pytest

import oracle
from paper_1610_04121_amd import SGM

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("adaptive", [False, True])
@pytest.mark.parametrize("lanes", [(0, 0), (16, 16), (64, 32)])
@pytest.mark.parametrize("W,H,D", [
    (16, 33, 64), (17, 32, 40), (31, 47, 128), (33, 48, 130), (48, 15, 256), (64, 65, 100), (2, 50, 128),
    (3, 49, 20), (81, 31, 200), (1, 34, 70), (20, 97, 64),
])
def test_blocks_per_direction_parity(gpu, W, H, D, lanes, adaptive):
    import torch
    rng = np.random.default_rng(W * 1009 + H * 31 + D)
    l, r = (rng.integers(0, 256, (H, W), dtype=np.uint8) for _ in range(2))
    print(f"blocks {W}x{H} D={D} lanes={lanes} adaptive={adaptive}", flush=True)
    s = SGM(W, H, D, 7, 86, 8, adaptive_p2=adaptive)
    s.set_tuning(*lanes)
    tl, tr = torch.from_numpy(l).to(gpu), torch.from_numpy(r).to(gpu)
    mc = oracle.cost_volume(oracle.census(l), oracle.census(r), D, oracle.cmax_of())
    for k, (rx, ry) in enumerate(oracle.directions(8)):
        got = s.debug_stage(tl, tr, k).cpu().numpy()
        want = oracle.aggregate(mc, 7, 86, rx, ry, img=l) if adaptive else oracle.aggregate(mc, 7, 86, rx, ry)
        bad = np.argwhere(got != want)
        assert len(bad) == 0, f"L_r ({rx},{ry}): {len(bad)} cells differ, first {bad[:5].tolist()}"
    s.close()
