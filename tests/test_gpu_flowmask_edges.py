"""Flow masking where its bounds and mask reads can go wrong: view widths
around the 8-byte mask reads, squares around the 64-pixel limit of one lane's
scan, Gaussians near and behind the near plane and far outside the view, single
mask pixels (the last one of the buffer among them), and more Gaussians than one
work-group takes.  Labels are integers and must equal the oracle's."""
import numpy as np
import pytest
import torch

import synth
from test_gpu_flowmask import gpu_labels, oracle_labels

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield


def masks_of(sc, kind, rng):
    n = sum(c.width * c.height for c in sc.cams)
    m = np.zeros(n, np.uint8)
    if kind == "last":
        m[-1] = 1
    elif kind == "few":
        m[rng.integers(0, n, max(1, n // 400))] = 1
    else:
        m[:] = rng.random(n) < 0.3
    return m


@pytest.mark.parametrize("kind", ["last", "few", "many"])
@pytest.mark.parametrize("side,w,h,lscale,views,pos", [
    (20, 61, 45, -3.0, 2, ((-1, -1, -1), (1, 1, 1))),
    (20, 7, 9, -1.5, 1, ((-1, -1, -1), (1, 1, 1))),
    (24, 200, 150, -1.0, 2, ((-1, -1, -1), (1, 1, 1))),          # squares on both sides of 64 pixels
    (50, 128, 64, -4.5, 3, ((-1, -1, -1), (1, 1, 1))),           # 2,500 Gaussians: ten work-groups per view
    (24, 96, 80, -3.0, 0, ((-6, -6, -0.5), (6, 6, 1.0))),        # across the near plane and outside the view
])
def test_flow_mask_edges(side, w, h, lscale, views, pos, kind):
    print(f"[gpu] flow mask edges {side} {w}x{h} {lscale} {views} {kind}", flush=True)
    sc = synth.random_scene(side=side, sh_degree=0, views=views, width=w, height=h, seed=side + w,
                            lscale=(lscale, 0.6), pos=pos)
    masks = masks_of(sc, kind, np.random.default_rng(w))
    D, _, _ = gpu_labels(sc, masks)
    _, ref = oracle_labels(sc, masks)
    assert np.array_equal(D, ref)
    # without the test counter, Gaussians already labelled by an earlier view are passed over
    from parity import atlas_tensor, renderer
    r = renderer(sc)
    dg, _ = r.flow_mask(atlas_tensor(sc), torch.from_numpy(masks).to("cuda:0"))
    assert np.array_equal(dg.cpu().numpy().reshape(ref.shape), ref)
    r.close()
