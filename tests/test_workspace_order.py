"""Workspace sizes grow with the sizes asked for, so that one workspace sized for the
largest call serves every smaller one: instance capacities and record counts around
the limits of the sort's small radix work-groups (2^18 pairs) and of views sorted
apart (2^17 and 2^18 records), Gaussians around 32 per pixel of the pruning's map.
And the photometric loss's holds the sums of every strip its rule
of view sizes takes.  On the host, with the runtime's calls stood in for."""
from fake_hip import run

SORT = """
import numpy as np, synth
def sort_bytes(views, side, n, cap):
    v = abi.pg_views_create([synth.pinhole(np.eye(3), np.zeros(3), side, side)] * views, 1, n, 0, abi.make_tiling())
    b = C.c_size_t()
    assert lib.pg_sort_workspace_size(v, cap, C.byref(b)) == 0
    abi.pg_views_destroy(v)
    return b.value
K = 1 << 18
for views, side in ((1, 1024), (1, 2048), (3, 640), (16, 640), (50, 320)):
    for n in (1000, 20000, 1 << 17, 300000):
        caps = [0, 1, 1000, K // 2, K - 1, K, K + 1, K + 4096, 2 * K, 4 * K, 1 << 24]
        got = [sort_bytes(views, side, n, c) for c in caps]
        assert got == sorted(got), (views, side, n, got)
    for cap in (1000, K, K + 1, 1 << 20, 1 << 25):
        ns = sorted({x for q in (1 << 17, K) for x in (q // views - 1, q // views, q // views + 1)} | {1023, 1024, 400000})
        got = [sort_bytes(views, side, n, cap) for n in ns]
        assert got == sorted(got), (views, side, cap, got)
"""

PRUNE = """
for frames, M, N in ((1, 64, 32), (3, 200, 100), (2, 16, 8)):
    ns = sorted({max(x, 0) for p in (32 * M * N, 262144 // frames) for x in (p - 1, p, p + 1)} | {0, 1, 100, 90000, 400000})
    got = []
    for n in ns:
        b = C.c_size_t()
        assert lib.pg_uv_prune_workspace_size(n, frames, M, N, C.byref(b)) == 0
        got.append(b.value)
    assert got == sorted(got), (frames, M, N, got)
"""


def test_sort_workspace_grows_with_capacity_and_records(tmp_path):
    run(tmp_path, SORT)


def test_prune_workspace_grows_with_the_gaussians(tmp_path):
    run(tmp_path, PRUNE)


PHOTO = """
import math, random
import numpy as np, synth
from test_gpu_photo_rule import rows_of
rng = random.Random(1)
tables = [[(32, 32)] * 600, [(64, 64)] * 200, [(54, 16)] * 600, [(1, 17)] * 600, [(640, 480)] * 3, [(33, 33)] * 130]
for _ in range(300):
    size = lambda: (int(math.exp(rng.uniform(0, 7))), int(math.exp(rng.uniform(0, 7))))
    tables.append([size()] * rng.randint(1, 600) if rng.random() < 0.5 else [size() for _ in range(rng.randint(1, 200))])
heights = set()
for t in tables:
    cams = []
    for w, h in t:
        c = synth.pinhole(np.eye(3), np.zeros(3), w, h)
        cams.append(c)
    v = abi.pg_views_create(cams, 1, 10, 0, abi.make_tiling())
    b = C.c_size_t()
    assert lib.pg_photo_workspace_size(v, C.byref(b)) == 0
    rows = rows_of(t)
    heights.add(rows)
    sums = sum(-(-w // 54) * -(-h // rows) for w, h in t) if rows else sum(-(-w // 32) * -(-h // 32) for w, h in t)
    assert b.value >= 16 * sums, (t[:3], len(t), rows)
    abi.pg_views_destroy(v)
assert heights == {0, 16, 32, 64, 192}, heights
"""


def test_photo_workspace_holds_every_strip(tmp_path):
    run(tmp_path, PHOTO)
