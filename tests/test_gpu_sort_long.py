"""pg_bin_sort with more than 4,096 compaction groups and all views in one sort, against
the numpy sort of test_gpu_sort_paths.py: scans and clears are then launches of their
own, and the compaction counts no digits.  A table of one view is never sorted by
view, nor is one whose capacity is at most 2^18 instances (here most of 31 views see
nothing).  Every output is an integer and must be equal."""
import numpy as np
import pytest
import torch

import synth
from parity import atlas_tensor, renderer, run_forward
from test_gpu_sort_paths import expected

pytestmark = pytest.mark.gpu


def sorted_apart(records, views, cap):
    """The sort's rule at these sizes (at least 2^18 records: a saved pass is not asked for)."""
    return views > 1 and cap > 1 << 18 and records >= 1 << 18


@pytest.mark.parametrize("n,views,seeing,back,cap", [(4194305, 1, (0,), 0.0, 1 << 23), (4195328, 1, (0,), 40.0, 1 << 23),
                                                     (140000, 31, (3,), 0.0, 1 << 18)])
def test_one_sort_over_many_groups(n, views, seeing, back, cap):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[gpu] long sort {n} x {views} views capacity {cap}", flush=True)
    assert -(-n * views // 1024) > 4096 and not sorted_apart(n * views, views, cap)
    side = int(np.ceil(np.sqrt(n)))
    sc = synth.random_scene(side=side, views=views, width=64, height=48, radius=8.0, seed=n % 1000, lscale=(-5.0, 0.5))
    for v, cam in enumerate(sc.cams):      # blind views: everything behind the camera
        cam.t = np.asarray(cam.t) + np.array([0.0, 0.0, back if v in seeing else -1000.0])
    occ = np.zeros_like(sc.occupancy)
    occ.reshape(-1)[:n] = 1
    sc.occupancy, sc.atlas = occ, sc.atlas * occ
    r = renderer(sc, cap=cap)
    for again in range(2):                 # a second sort on the words the first one left
        run_forward(r, atlas_tensor(sc))
        s = r.sets[0]
        assert s.cap == cap                # not grown to another path
        tile, gv, first = expected(r)
        keys, vals = r.sorted_instances()
        assert keys.size == tile.size > 0
        assert np.array_equal(keys.astype(np.int64), tile) and np.array_equal(vals, gv)
        assert np.array_equal(s.inst_first[:s.info.n_gv].cpu().numpy(), first)
        rg = s.ranges.cpu().numpy().reshape(-1, 2)[:s.info.n_tiles]
        count = np.bincount(tile, minlength=s.info.n_tiles)
        assert np.array_equal(rg[:, 1] - rg[:, 0], count)
        assert np.array_equal(rg[count > 0, 0], (np.cumsum(count) - count)[count > 0])
    r.close()
