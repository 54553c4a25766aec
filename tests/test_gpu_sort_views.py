"""pg_bin_sort with its views sorted apart, against a numpy sort of the projection's
bins and tile sets over all views: record counts on both sides of the limits of
that path (2^18 records, 2^17 where it saves a pass), runs that end on
and off the 1,024 records of a compaction group and the 4,096 pairs of a radix
work-group, views of two sizes, views that see nothing at either end, and depths
whose high digit is one value in all views, in some, or in none.  Every output is
an integer and must be equal."""
import numpy as np
import pytest
import torch

import synth
from parity import atlas_tensor, renderer, run_forward
from test_gpu_sort_paths import expected

pytestmark = pytest.mark.gpu

# records per view, views, sizes, camera distance, views that see nothing, views moved back
CASES = [(2048, 64, ((160, 120),), 8.0, (), (3,)),
         (2047, 64, ((160, 120),), 8.0, (), (3,)),
         (4096, 64, ((320, 240),), 8.0, (63,), (3,)),
         (4095, 64, ((320, 240),), 8.0, (63,), (3,)),
         (9000, 60, ((160, 120), (64, 48)), 4.0, (0, 7, 59), ()),
         (8192, 70, ((160, 120),), 8.0, (), (3, 4)),
         (8191, 64, ((160, 120),), 8.0, (), (3,)),
         (1024, 600, ((64, 48),), 20.0, (599,), (0,)),
         (1025, 520, ((64, 48), (48, 64)), 4.0, (1, 2), ()),
         (30000, 40, ((640, 480), (320, 240)), 8.0, (39,), (1,)),
         (240000, 9, ((320, 240),), 8.0, (4,), (5,)),
         (2100000, 2, ((64, 48),), 8.0, (), ())]


@pytest.mark.parametrize("n,views,sizes,radius,blind,back", CASES)
def test_views_sorted_apart_match_numpy(n, views, sizes, radius, blind, back):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[gpu] sort {n} x {views} views {sizes}", flush=True)
    side = int(np.ceil(np.sqrt(n)))
    sc = synth.random_scene(side=side, views=views, radius=radius, seed=n % 1000, lscale=(-5.0, 0.5))
    sc.cams = synth.ring_cameras(views, radius, 0, 0, sizes=list(sizes))
    for v, shift in [(v, -1000.0) for v in blind] + [(v, 16.0) for v in back]:
        sc.cams[v].t = np.asarray(sc.cams[v].t) + np.array([0.0, 0.0, shift])
    occ = np.zeros_like(sc.occupancy)
    occ.reshape(-1)[:n] = 1
    sc.occupancy, sc.atlas = occ, sc.atlas * occ
    r = renderer(sc, cap=1 << 23)
    for again in range(2):             # a second sort on the words the first one left
        run_forward(r, atlas_tensor(sc))
        tile, gv, first = expected(r)
        keys, vals = r.sorted_instances()
        assert keys.size == tile.size > 0
        assert np.array_equal(keys.astype(np.int64), tile) and np.array_equal(vals, gv)
        s = r.sets[0]
        assert np.array_equal(s.inst_first[:s.info.n_gv].cpu().numpy(), first)
        rg = s.ranges.cpu().numpy().reshape(-1, 2)[:s.info.n_tiles]
        count = np.bincount(tile, minlength=s.info.n_tiles)
        assert np.array_equal(rg[:, 1] - rg[:, 0], count)
        assert np.array_equal(rg[count > 0, 0], (np.cumsum(count) - count)[count > 0])
        assert r.check()
    r.close()
