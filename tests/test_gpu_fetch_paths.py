"""The fetch's gather and the fake quantiser where their splits can go wrong:
Gaussian counts around the 256 of a gather group and the 1,024 of a quantiser
group, row counts (frames x channels) that are no multiple of the 8 in flight,
enough Gaussians that the rows are not split, and channels left alone.  Copies
are exact; the quantiser's steps are single FP32 operations, which numpy repeats
bit for bit."""
import numpy as np
import pytest
import torch

from paper_2602_23040_amd import _abi as abi
from paper_2602_23040_amd.pipeline import Renderer
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield


@pytest.mark.parametrize("n,frames,sh", [(1, 1, 0), (255, 1, 3), (256, 2, 1), (257, 3, 2), (1023, 1, 0), (1024, 5, 3),
                                         (1025, 1, 3), (4099, 2, 0), (300001, 1, 1)])
def test_gather_and_quantiser(n, frames, sh):
    print(f"[gpu] fetch paths n {n} F {frames} sh {sh}", flush=True)
    side = int(np.ceil(np.sqrt(1.3 * n)))
    rng = np.random.default_rng(n)
    occ = np.zeros(side * side, np.uint8)
    texel = np.sort(rng.permutation(side * side)[:n])
    occ[texel] = 1
    occ = occ.reshape(side, side)
    C = synth.n_channels(sh)
    atlas = rng.standard_normal((frames, C, side, side)).astype(np.float32)
    cam = synth.pinhole(np.eye(3), np.zeros(3), 16, 16)
    cams = [synth.Camera(cam.R, cam.t, cam.fx, cam.fy, cam.cx, cam.cy, 16, 16, f) for f in range(frames)]
    ref = atlas.reshape(frames, C, -1)[:, :, texel]
    dev = torch.from_numpy(atlas.reshape(-1)).to("cuda:0")
    r = Renderer(occ, frames, sh, cams, device="cuda:0", inst_capacity=4096)
    r.fetch(dev)
    assert np.array_equal(r.params.cpu().numpy().reshape(ref.shape), ref)
    r.close()
    bits = [0 if c % 5 == 2 else (16 if c < 3 else 8) for c in range(C)]
    q = Renderer(occ, frames, sh, cams, device="cuda:0", inst_capacity=4096, quant_bits=bits)
    q.fetch(dev)
    exp = ref.copy()
    for c, b in enumerate(bits):
        if b:
            lo, hi = ref[:, c].min(), ref[:, c].max()
            levels = np.float32((1 << b) - 1)
            delta = np.float32((hi - lo) / levels)
            if delta > 0:
                k = np.clip(np.rint((ref[:, c] - lo) / delta), 0, levels).astype(np.float32)
                exp[:, c] = lo + k * delta
    assert np.array_equal(q.params.cpu().numpy().reshape(ref.shape), exp)
    codes = torch.full((frames * C * n,), 7, dtype=torch.uint16, device="cuda:0")
    abi.pg_atlas_fake_quant(q.params, q.n_gauss_dev, q.N, frames, C, bits, q.quant_range, codes, q.quant_partial)
    got = codes.cpu().numpy().reshape(ref.shape)
    left = [c for c, b in enumerate(bits) if b == 0]
    assert not got[:, left].any()
    q.close()
