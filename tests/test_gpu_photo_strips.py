"""The photometric loss's strip kernel (tables of more than 512 blocks of 32x32
pixels) against a torch FP64 restatement, under the rules of test_gpu_loss.py:
loss to 1e-5 relative, cotangent to the gradient rule.  View sizes lie around
the 54 columns of a strip, the 32, 64 and 192 rows it can have, and the 32 rows
between shifts of its base; images hold flat bright and black areas beside
texture."""
import numpy as np
import pytest
import torch

import synth
from parity import grad_compare, renderer

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    yield


def blur(v):
    k = torch.exp(-(torch.arange(11, dtype=torch.float64, device=v.device) - 5) ** 2 / 4.5)
    k = k / k.sum()
    H, W = v.shape[1:]
    v = torch.nn.functional.pad(v, (0, 0, 5, 5))
    v = sum(k[i] * v[:, i:i + H] for i in range(11))
    v = torch.nn.functional.pad(v, (5, 5))
    return sum(k[i] * v[:, :, i:i + W] for i in range(11))


def reference(image, target, sizes, lam):
    image, n, at, total = image.double().requires_grad_(True), image.numel(), 0, 0.0
    for w, h in sizes:
        x, y = (v[at:at + 3 * w * h].view(3, h, w) for v in (image, target.double()))
        mx, my = blur(x), blur(y)
        sx, sy, sxy = blur(x * x) - mx * mx, blur(y * y) - my * my, blur(x * y) - mx * my
        S = (2 * mx * my + 1e-4) * (2 * sxy + 9e-4) / ((mx * mx + my * my + 1e-4) * (sx + sy + 9e-4))
        part = ((1 - lam) * (x - y).abs().sum() + lam * (x.numel() - S.sum())) / n
        part.backward()
        total += float(part)
        at += 3 * w * h
    return total, image.grad


RAGGED = [(640, 480), (331, 257), (54, 33), (55, 64), (1, 1), (53, 700), (108, 31), (1024, 200), (5, 400)]


@pytest.mark.parametrize("lam", [0.0, 0.2, 1.0])
@pytest.mark.parametrize("sizes", [RAGGED, [(108, 832)] * 39 + [(109, 833), (61, 65)],
                                   [(108, 832)] * 105 + [(107, 191), (55, 193), (54, 1000)]],
                         ids=["32 rows", "64 rows", "192 rows"])
def test_strips_match_fp64(sizes, lam):
    print(f"[gpu] photo strips {len(sizes)} views, lambda {lam}", flush=True)
    sc = synth.random_scene(side=2, views=1, width=8, height=8, seed=1)
    cam = sc.cams[0]
    sc.cams = [synth.Camera(cam.R, cam.t, 100.0, 100.0, w / 2, h / 2, w, h) for w, h in sizes]
    r = renderer(sc)
    gen = torch.Generator("cuda:0").manual_seed(len(sizes))
    target = torch.cat([torch.nn.functional.interpolate(
        torch.rand((1, 3, h // 24 + 2, w // 24 + 2), device="cuda:0", generator=gen), (h, w), mode="bilinear").reshape(-1)
        for w, h in sizes])
    image = (target + 0.05 * torch.randn(target.shape, device="cuda:0", generator=gen)).clamp_(0, 1)
    at = 0
    for v, (w, h) in enumerate(sizes):          # a black and a flat bright band per view
        x, y = image[at:at + 3 * w * h].view(3, h, w), target[at:at + 3 * w * h].view(3, h, w)
        x[:, h // 3:h // 2], y[:, h // 3:h // 2] = 0.0, 0.0
        x[:, :, w // 2:2 * w // 3], y[:, :, w // 2:2 * w // 3] = 0.9, 0.9 if v % 2 else 0.8
        at += 3 * w * h
    r.image.copy_(image)
    loss = float(r.loss_photo(target, lam).item())
    ref, G = reference(image, target, sizes, lam)
    assert abs(loss - ref) <= 1e-5 * abs(ref)
    st = grad_compare(r.dL_dimage.cpu().numpy().reshape(1, 1, -1), G.cpu().numpy().reshape(1, 1, -1))
    print("[gpu]", st, flush=True)
    assert st["n_bad"] == 0 and st["worst_l2"] <= 1e-3, st
    r.close()
