"""The photometric loss's strip kernel on images far from their targets: flat
colours apart by a constant (a wrong colour, as at the start of a fit), plain and
under noise, colours above 1 among them.  There the variances are differences of
large moments unless x, y and x - y are all shifted first.

Against the FP64 restatement of test_gpu_photo_strips.py: the loss to 1e-5
relative, the cotangent to the gradient rule (1e-3 relative per element with a
floor of 1 % of the largest) plus the rounding that the sum of its three terms
cannot do without: they reach 2 |d| N1 / (D1 D2) <= 2 |d| / C2 and cancel, each
rounded some eight times (windows, partial maps)."""
import pytest
import torch

import synth
from parity import renderer
from test_gpu_photo_strips import reference

pytestmark = pytest.mark.gpu

SIZES = [(640, 480), (331, 257), (1024, 200), (54, 33), (5, 400), (1024, 768)]     # more than 512 blocks: strips


@pytest.mark.parametrize("lam", [0.2, 1.0])
@pytest.mark.parametrize("noise", [0.0, 0.01])
@pytest.mark.parametrize("x,y", [(0.2, 0.8), (0.1, 0.9), (0.8, 0.5), (2.0, 0.5), (10.0, 5.0)])
def test_constant_offsets_match_fp64(x, y, noise, lam):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[gpu] photo flat {x} / {y}, noise {noise}, lambda {lam}", flush=True)
    sc = synth.random_scene(side=2, views=1, width=8, height=8, seed=1)
    cam = sc.cams[0]
    sc.cams = [synth.Camera(cam.R, cam.t, 100.0, 100.0, w / 2, h / 2, w, h) for w, h in SIZES]
    r = renderer(sc)
    gen = torch.Generator("cuda:0").manual_seed(7)
    n = 3 * sum(w * h for w, h in SIZES)
    image, target = (c + noise * torch.randn(n, device="cuda:0", generator=gen) for c in (x, y))
    r.image.copy_(image)
    loss = float(r.loss_photo(target, lam).item())
    ref, G = reference(image, target, SIZES, lam)
    print(f"[gpu] {abs(loss - ref) / abs(ref):.1e}", flush=True)
    assert abs(loss - ref) <= 1e-5 * abs(ref)
    got = r.dL_dimage.double()
    rounding = lam / n * 8 * 2.0 ** -24 * 2 * (abs(x - y) + 10 * noise) / 9e-4
    err = (got - G).abs() - 1e-3 * torch.clamp(G.abs(), min=float(0.01 * G.abs().max())) - rounding
    assert float(err.max()) <= 0.0
    assert float((got - G).norm()) <= 1e-3 * float(G.norm()) + rounding * n ** 0.5
    r.close()
