"""The emission of pg_bin_sort against a numpy sort of its inputs: windows of 64
sorted records that fit its staging buffer (608 instances), that end just beside
it, that do not fit, and that hold records keeping every tile of a rectangle
larger than 64 tiles.  Every output is an integer and must be equal."""
import numpy as np
import pytest
import torch

import synth
from parity import atlas_tensor, renderer, run_forward
from test_gpu_sort_paths import expected

pytestmark = pytest.mark.gpu

# n, views, log scale mean and spread, what the scene has to hold
CASES = [(5000, 2, (-5.0, 0.3), "short"), (6000, 1, (-3.3, 0.1), "edge"), (3000, 2, (-3.0, 0.4), "long"),
         (1500, 1, (-1.5, 0.8), "whole"), (4000, 2, (-4.0, 1.5), "mixed"), (1, 1, (-5.0, 0.1), "one")]


@pytest.mark.parametrize("n,views,scale,kind", CASES)
def test_emission_matches_numpy(n, views, scale, kind):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[gpu] emission {n} x {views} {kind}", flush=True)
    side = int(np.ceil(np.sqrt(n)))
    sc = synth.random_scene(side=side, views=views, width=640, height=480, seed=n % 1000, lscale=scale)
    occ = np.zeros_like(sc.occupancy)
    occ.reshape(-1)[:n] = 1
    sc.occupancy, sc.atlas = occ, sc.atlas * occ
    r = renderer(sc)
    run_forward(r, atlas_tensor(sc))
    tile, gv, _ = expected(r)
    bins, ts = r.bin_records(), r.tile_sets()
    nt = bins["n_tiles"].astype(np.int64)
    rec = np.flatnonzero(nt > 0)
    rec = rec[np.argsort(bins["key"][rec], kind="stable")]
    window = np.add.reduceat(nt[rec], np.arange(0, rec.size, 64))
    whole = (ts["mask"][rec] == 0).any()
    if kind == "edge":
        assert (np.abs(window - 608) < 64).any()
    assert (window > 608).any() == (kind in ("long", "whole", "mixed", "edge"))
    assert whole or kind not in ("whole", "mixed")
    keys, vals = r.sorted_instances()
    assert np.array_equal(keys.astype(np.int64), tile) and np.array_equal(vals, gv)
    r.close()
