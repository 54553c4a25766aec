"""The motion cells of many tiles (more than 32,768: four tiles per lane), against
the oracle's labels: views of unlike sizes whose ends fall inside a work-group's 32
tiles, a tile count off every multiple, and motion in the last pixels of views."""
import numpy as np
import pytest
import torch

import synth
from test_gpu_flowmask import gpu_labels, oracle_labels

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiling", [(16, 16, 64), (8, 32, 64), (32, 8, 64)])
@pytest.mark.parametrize("views", [33, 41])
def test_motion_cells_of_many_tiles(views, tiling):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[gpu] motion cells of {views} views, tiling {tiling}", flush=True)
    sc = synth.random_scene(side=12, views=views, seed=views, lscale=(-3.0, 0.6))
    sc.cams = synth.ring_cameras(views, 4.0, 0, 0, sizes=[(640, 480), (17, 9), (801, 603)])
    sc.tiling = synth.Tiling(*tiling)
    rng = np.random.default_rng(views)
    masks = []
    for c in sc.cams:
        m = np.zeros((c.height, c.width), np.uint8)
        m[rng.integers(0, c.height, 40), rng.integers(0, c.width, 40)] = 1
        m[-1, -1] = 1
        masks.append(m.reshape(-1))
    masks = np.concatenate(masks)
    D, _, _ = gpu_labels(sc, masks)
    _, ref = oracle_labels(sc, masks)
    assert 0 < ref.sum() and np.array_equal(D, ref)
