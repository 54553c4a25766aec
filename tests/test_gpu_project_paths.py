"""pg_project's launch paths against the oracle's FP64 projection: geometry and
colour in one thread or in waves of their own (more than 12 views of SH degree
2 or 3 per work-group), views in one loop or in chunks (few Gaussians), and
Gaussian counts around the 128 of a work-group.  The records are integers,
FP64 means and floats; check_records and check_tile_lists hold them bit for bit
(integers, means, lists) and to 1e-6 (floats)."""
import numpy as np
import pytest
import torch

import oracle
import synth
from parity import atlas_tensor, check_records, check_tile_lists, renderer, run_forward

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield


# side, SH degree, views per frame, frames, log-scale.  410^2 Gaussians are 1,314 work-groups: one loop over the
# views; below about 131,000 the views are dealt in chunks.
CASES = [(1, 3, 14, 1, -2.0), (11, 3, 3, 2, -3.0), (12, 2, 13, 1, -2.5), (23, 0, 7, 3, -3.0), (9, 1, 30, 1, -1.0),
         (410, 3, 14, 1, -5.5), (410, 2, 13, 1, -5.5), (410, 3, 2, 1, -5.5)]


@pytest.mark.parametrize("side,sh,views,frames,lscale", CASES)
def test_project_paths(side, sh, views, frames, lscale):
    print(f"[gpu] project side {side} sh {sh} {frames} x {views} views", flush=True)
    w, h = (64, 48) if side > 100 else (101, 77)
    sc = synth.random_scene(side=side, sh_degree=sh, views=views, width=w, height=h, seed=side + sh,
                            lscale=(lscale, 0.6), frames=frames)
    check = range(len(sc.cams)) if side < 100 else sorted({0, views // 2, views - 1})
    fw = oracle.Forward(sc, views=list(check))
    r = renderer(sc)
    run_forward(r, atlas_tensor(sc))
    bins, tsets, splats = r.bin_records(), r.tile_sets(), r.splat_records()
    keys, vals = r.sorted_instances()
    for v in check:
        valid, _ = check_records(fw, v, bins, tsets, splats, r.N)
        s, pr = splats[v * r.N:(v + 1) * r.N], fw.proj[v]
        np.testing.assert_allclose(s["conic"][valid], pr["conic"][valid], rtol=1e-6, atol=1e-9)
        np.testing.assert_allclose(s["opacity"][valid], pr["opacity"][valid], rtol=1e-6)
        np.testing.assert_allclose(s["color"][valid], pr["color"][valid], rtol=1e-6, atol=1e-7)
        assert np.array_equal(s["depth"][valid].view(np.uint32), pr["key"][valid])
        check_tile_lists(fw, v, keys, vals, r.sets[0].tile_base, r.N)
    if side < 100:
        vis = r.visible[:sc.frames * r.N].cpu().numpy().reshape(sc.frames, r.N)
        assert np.array_equal(vis, fw.visible())
    r.close()
