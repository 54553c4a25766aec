"""pg_bin_sort against a numpy sort of its own inputs (the projection's bins and
tile sets): record counts around the 1,024 and 4,096 pairs of a radix work-group
and the 1,024 records of a compaction group, capacities on both sides of the
limit of the small radix work-groups (2^18), and record counts past 4,096
compaction groups, where the scans and clears are launches of their own.  Every
output is an integer and must be equal."""
import numpy as np
import pytest
import torch

import synth
from parity import atlas_tensor, renderer, run_forward

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield


def expected(r):
    """(tile, gv) of every instance in sorted order, and inst_first."""
    bins, ts, s = r.bin_records(), r.tile_sets(), r.sets[0]
    nt = bins["n_tiles"].astype(np.int64)
    rec = np.flatnonzero(nt > 0)
    rec = rec[np.argsort(bins["key"][rec], kind="stable")]
    tx = np.array([-(-c.width // r.tiling.tile_w) for c in r.cams], np.int64)
    view = rec // r.N
    cnt = nt[rec]
    who = np.repeat(np.arange(rec.size), cnt)
    k = np.arange(cnt.sum()) - np.repeat(np.cumsum(cnt) - cnt, cnt)
    w = ts["width"][rec].astype(np.int64)
    mask = ts["mask"][rec]
    bit = k.copy()
    small = np.flatnonzero(mask[who] != 0)
    if small.size:                     # the k-th set bit of the mask
        bits = (mask[:, None] >> np.arange(64, dtype=np.uint64)) & np.uint64(1)
        order = np.argsort(1 - bits.astype(np.int8), axis=1, kind="stable")
        bit[small] = order[who[small], k[small]]
    tile = (np.asarray(s.tile_base)[view][who] + (ts["y_lo"][rec][who] + bit // w[who]) * tx[view][who]
            + ts["x_lo"][rec][who] + bit % w[who])
    o = np.argsort(tile, kind="stable")
    return tile[o], rec[who][o], np.cumsum(nt) - nt


CASES = [(1023, 1, 64, 48, None), (1024, 1, 64, 48, None), (1025, 1, 64, 48, None), (4097, 1, 320, 200, None),
         (3000, 3, 160, 120, None), (20000, 2, 320, 240, 1 << 18), (20000, 2, 320, 240, (1 << 18) + 1),
         (140000, 2, 640, 480, 1 << 20), (140000, 31, 64, 48, 1 << 23)]


@pytest.mark.parametrize("n,views,w,h,cap", CASES)
def test_sort_matches_numpy(n, views, w, h, cap):
    print(f"[gpu] sort {n} x {views} views {w}x{h} capacity {cap}", flush=True)
    side = int(np.ceil(np.sqrt(n)))
    sc = synth.random_scene(side=side, sh_degree=0, views=views, width=w, height=h, seed=n % 1000,
                            lscale=(-3.5 if n < 50000 else -5.0, 0.5))
    occ = np.zeros_like(sc.occupancy)
    occ.reshape(-1)[:n] = 1
    sc.occupancy, sc.atlas = occ, sc.atlas * occ
    r = renderer(sc, cap=cap)
    run_forward(r, atlas_tensor(sc))
    for again in range(2):             # a second sort on the words the first one left
        if again:
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
        assert int(s.n_inst[1]) >= 2 + again - 1 and r.check()
    r.close()
