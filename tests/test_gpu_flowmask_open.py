"""Flow masking of many work-groups (more than 4,096), where the Gaussians that no
earlier view has labelled are collected first: one Gaussian, part of a chunk, a
chunk and its neighbours, with few and with most Gaussians labelled, with and
without the test counter.  Labels are integers and must equal the oracle's."""
import numpy as np
import pytest
import torch

import synth
from parity import atlas_tensor, renderer
from test_gpu_flowmask import gpu_labels, oracle_labels

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("share", [0.0005, 0.2])
@pytest.mark.parametrize("n,views", [(1, 520), (300, 520), (768, 520), (2049, 520), (2500, 513)])
def test_unlabelled_gaussians_collected(n, views, share):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[gpu] flow mask of {n} Gaussians in {views} views, {share} of motion", flush=True)
    side = int(np.ceil(np.sqrt(n)))
    sc = synth.random_scene(side=side, views=views, width=24, height=16, seed=n, lscale=(-4.0, 0.6))
    occ = np.zeros_like(sc.occupancy)
    occ.reshape(-1)[:n] = 1
    sc.occupancy, sc.atlas = occ, sc.atlas * occ
    masks = (np.random.default_rng(n).random(views * 24 * 16) < share).astype(np.uint8)
    D, _, _ = gpu_labels(sc, masks)
    _, ref = oracle_labels(sc, masks)
    assert np.array_equal(D, ref)
    r = renderer(sc)
    for _ in range(2):
        dg, _ = r.flow_mask(atlas_tensor(sc), torch.from_numpy(masks).to("cuda:0"))
        assert np.array_equal(dg.cpu().numpy().reshape(ref.shape), ref)
    r.close()
