"""Pixels that are not finite in the photometric loss's strip kernel: they spoil the
windows that hold them and no others.  Infinities and NaN stand in the image and
in the target, in rows of every kind (shifts are taken from every 16th row), at the
borders and inside; every cotangent that is finite in the FP64 restatement of
test_gpu_photo_strips.py has to match it under the gradient rule."""
import pytest
import torch

import synth
from parity import renderer
from test_gpu_photo_strips import reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
@pytest.mark.parametrize("where", ["image", "target"])
def test_bad_pixels_stay_in_their_windows(bad, where):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[gpu] photo pixels {bad} in {where}", flush=True)
    W, H = 1500, 1000         # more than 512 blocks: strips
    sc = synth.random_scene(side=2, views=1, width=8, height=8, seed=1)
    cam = sc.cams[0]
    sc.cams = [synth.Camera(cam.R, cam.t, 100.0, 100.0, W / 2, H / 2, W, H)]
    r = renderer(sc)
    gen = torch.Generator("cuda:0").manual_seed(3)
    target = torch.rand(3 * W * H, device="cuda:0", generator=gen)
    image = (target + 0.05 * torch.randn(target.shape, device="cuda:0", generator=gen)).clamp_(0, 1)
    planes = (image if where == "image" else target).view(3, H, W)
    for k in range(32):       # rows 25 k: all residues
        planes[k % 3, 25 * k, 34 * k + 3] = bad
    planes[0, H - 1, 0] = planes[1, 0, W - 1] = bad
    r.image.copy_(image)
    r.loss_photo(target, 0.2)
    _, G = reference(image, target, [(W, H)], 0.2)
    got, ok = r.dL_dimage.double(), torch.isfinite(G)
    assert 0.98 * G.numel() < int(ok.sum()) < G.numel()
    got, G = got[ok], G[ok]
    assert bool(torch.isfinite(got).all())
    assert float(((got - G).abs() / torch.clamp(G.abs(), min=float(0.01 * G.abs().max()))).max()) <= 1e-3
    r.close()
