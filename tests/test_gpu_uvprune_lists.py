"""UV pruning by pixel lists and its way over to the sorts: lists around the 512
entries that are ranked by comparison, all in one pixel beside sparse ones, equal
opacities, and Gaussian counts on both sides of the 32 per pixel up to which
lists are tried.  Pixels, ranks and flags are integers and must equal the oracle's."""
import numpy as np
import pytest
import torch

import synth
from test_gpu_uvprune import reference, run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield


@pytest.mark.parametrize("heavy", [0, 511, 512, 513, 2000])
@pytest.mark.parametrize("M,Nv", [(16, 8), (64, 32), (10, 6), (9, 7)])
def test_pixel_lists(heavy, M, Nv):
    print(f"[gpu] uv lists heavy {heavy} map {M}x{Nv}", flush=True)
    sc = synth.random_scene(side=45, sh_degree=0, views=1, width=16, height=16, seed=heavy + M, frames=2)   # 2,025 each
    for f in range(2):
        planes = sc.atlas[f].reshape(sc.C, -1)
        k = np.random.default_rng(f).permutation(planes.shape[1])[:heavy if f else heavy // 2]
        planes[0:3, k] = np.array([[0.7], [0.31], [0.11]], np.float32) * np.linspace(0.5, 1.5, k.size, dtype=np.float32)
        planes[10] = np.round(planes[10] * 4) / 4          # many equal opacities
    for K in (1, 7):
        got, ref = run(sc, M, Nv, K), reference(sc, M, Nv, K)
        for a, b, what in zip(got, ref, ("uv", "rank", "keep")):
            assert np.array_equal(a.astype(np.int64), b.astype(np.int64)), what
