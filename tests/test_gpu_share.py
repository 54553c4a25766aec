"""Compositing kernels of view tables with few tiles (four waves per tile)
against the one-wave kernels: the same view rendered alone and beside a large
empty view that takes the table past the few-tile limits.  List lengths sit at
the edges of the staged steps (64, 128 and 256), in one tile and over ragged
tiles, with and without early termination.

Every pixel runs the same operations in the same order in both, so images, T,
n_contrib and entries must agree bitwise.  The adjoint's per-pixel terms are
the same too; only the order in which up to 256 of them are added differs:
about 10 roundings on either side, 2 * 10 * 2^-24 of the sum of magnitudes,
and 1e-4 of the channel's norm leaves a factor of 80 for cancellation."""
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


def scene(n, w, h, lscale, lopac, seed):
    """n Gaussians around the optical axis of one camera."""
    sc = synth.random_scene(side=n, sh_degree=1, views=0, width=w, height=h, seed=seed, lscale=(lscale, 0.3),
                            pos=((-0.3, -0.3, 2.5), (0.3, 0.3, 3.5)), lopac=(lopac, 0.5))
    occ = np.zeros_like(sc.occupancy)
    occ.reshape(-1)[:n] = 1
    sc.occupancy = occ
    sc.atlas = sc.atlas * occ
    return sc


CASES = [(1, 16, 16, -0.5, -2.0), (64, 16, 16, -0.5, -4.0), (65, 16, 16, -0.5, -4.0), (129, 16, 16, -0.5, -4.0),
         (256, 16, 16, -0.5, -4.5), (257, 16, 16, -0.5, -4.5), (600, 16, 16, -0.5, -4.5), (600, 16, 16, -0.5, 4.0),
         (300, 61, 45, -2.5, 0.0), (900, 100, 37, -3.5, 1.5)]


@pytest.mark.parametrize("tiling", [(16, 16, 64), (8, 32, 128), (32, 8, 256)])
@pytest.mark.parametrize("n,w,h,lscale,lopac", CASES)
def test_few_tile_kernels_match_the_one_wave_kernels(n, w, h, lscale, lopac, tiling):
    print(f"[gpu] {n} Gaussians, {w}x{h}, opacity {lopac}, {tiling}", flush=True)
    sc = scene(n, w, h, lscale, lopac, seed=n)
    away = synth.pinhole(np.diag([1.0, -1.0, -1.0]), np.zeros(3), 1600, 1600)      # looks along -z: sees nothing
    few = renderer(sc, tiling=tiling)
    sc.cams = [sc.cams[0], away]
    many = renderer(sc, tiling=tiling)
    assert few.sets[0].info.n_tiles < 100 and many.sets[0].info.n_tiles > 10000
    atlas = atlas_tensor(sc)
    for r in (few, many):
        run_forward(r, atlas)
    px, nt = few.n_pixels, few.sets[0].info.n_tiles
    assert torch.equal(few.image, many.image[:3 * px])
    assert torch.equal(few.final_T, many.final_T[:px]) and torch.equal(few.n_contrib, many.n_contrib[:px])
    te, tm = few.sets[0].tile_entries[:nt], many.sets[0].tile_entries[:nt]
    assert torch.equal(te, tm) and int(te.sum()) > 0
    rf, rm = (r.sets[0].ranges[:2 * nt].view(-1, 2).cpu() for r in (few, many))
    for t in range(nt):
        c = int(te[t])
        assert torch.equal(few.sets[0].entries[int(rf[t, 0]):int(rf[t, 0]) + c],
                           many.sets[0].entries[int(rm[t, 0]):int(rm[t, 0]) + c])
    g = torch.randn(many.image.shape, device="cuda:0", generator=torch.Generator("cuda:0").manual_seed(n))
    few.backward(g[:3 * px].contiguous())
    many.backward(g)
    ngv = few.sets[0].info.n_gv
    a = few.sets[0].grad2d[:9 * ngv].view(9, ngv).double()
    b = many.sets[0].grad2d[:18 * ngv].view(9, 2, ngv)[:, 0].double()
    err = (a - b).norm(dim=1) / b.norm(dim=1).clamp_min(1e-30)
    print("[gpu] slot sums, relative per channel:", [f"{x:.1e}" for x in err.tolist()], flush=True)
    assert float(b.abs().max()) > 0 and float(err.max()) <= 1e-4
    for r in (few, many):
        r.close()
