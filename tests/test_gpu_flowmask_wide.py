"""Flow masking of Gaussians whose squares lie over many screen tiles: the motion
cells are then read eight tiles at a time.  Every tile shape, spans around six tiles
(where that begins) and around multiples of eight, set pixels that are few and single
(the last of a view, the last of the buffer), ragged views whose last tiles are cut.
Labels are integers and must equal the oracle's.  And without motion, large Gaussians
cost their projection and the cells under them, not a walk over every tile by a wave."""
import numpy as np
import pytest
import torch

import synth
from parity import atlas_tensor, renderer
from test_gpu_flowmask import gpu_labels, oracle_labels

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield


@pytest.mark.parametrize("few", [1, 6, 60])
@pytest.mark.parametrize("lscale", [-2.6, -1.8, -0.8])
@pytest.mark.parametrize("tiling", [(16, 16, 64), (8, 32, 64), (32, 8, 64)])
def test_squares_of_many_tiles(tiling, lscale, few):
    print(f"[gpu] flow mask wide {tiling} {lscale} {few}", flush=True)
    sc = synth.random_scene(side=24, sh_degree=0, views=2, width=301, height=237, seed=few, lscale=(lscale, 0.5),
                            tiling=synth.Tiling(*tiling))
    sc.cams[1].width, sc.cams[1].height = 261, 133
    n = [c.width * c.height for c in sc.cams]
    rng = np.random.default_rng(few + tiling[0])
    masks = np.zeros(sum(n), np.uint8)
    masks[rng.integers(0, sum(n), few)] = 1
    masks[n[0] - 1] = masks[-1] = 1
    D, _, _ = gpu_labels(sc, masks)
    _, ref = oracle_labels(sc, masks)
    assert np.array_equal(D, ref)


def test_large_gaussians_without_motion():
    """Every Gaussian over most of the screen: 4 views of 16,384 took as long without
    motion as with motion everywhere (a wave per Gaussian over all of its tiles), and
    takes a hundredth of that; an eighth is asked for."""
    sc = synth.random_scene(side=128, sh_degree=0, views=4, width=1024, height=768, seed=1, lscale=(-1.0, 0.5))
    r = renderer(sc)
    atlas = atlas_tensor(sc)
    times = []
    for value in (0, 1):
        masks = torch.full((r.n_pixels,), value, dtype=torch.uint8, device="cuda:0")
        best = 1e9
        for _ in range(4):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            dg, _ = r.flow_mask(atlas, masks)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        times.append(best)
    print(f"[gpu] flow mask without / with motion {times}", flush=True)
    assert times[0] <= times[1] / 8
    r.close()
