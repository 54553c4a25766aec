"""UV pruning on both sides of the limits between pixel lists and sorts: one long list
(256 entries), the comparisons of many lists (128 a Gaussian as counted, 64 as
expected of an even map), the pixels of the map (2^22), and 2^18 Gaussians, each
with crowded pixels.  Pixels, ranks and
flags are integers and must equal the oracle's."""
import numpy as np
import pytest
import torch

import synth
from test_gpu_uvprune import reference, run

pytestmark = pytest.mark.gpu


# side of the atlas (two frames), map, crowded pixels, Gaussians in each
@pytest.mark.parametrize("side,M,Nv,pixels,each", [
    (45, 64, 32, 1, 255), (45, 64, 32, 1, 256), (45, 64, 32, 1, 257),
    (45, 64, 32, 10, 100), (45, 64, 32, 10, 160), (45, 64, 32, 10, 200),
    (45, 8, 4, 0, 0), (45, 11, 3, 0, 0), (45, 2048, 1024, 3, 70), (45, 2049, 1024, 3, 70),
    (362, 256, 128, 0, 0), (363, 256, 128, 0, 0), (363, 256, 128, 1, 250), (363, 256, 128, 40, 3000)])
def test_lists_and_sorts_agree_with_the_oracle(side, M, Nv, pixels, each):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print(f"[gpu] uv limits {side}^2 x 2 on {M}x{Nv}, {pixels} pixels of {each}", flush=True)
    sc = synth.random_scene(side=side, sh_degree=0, views=1, width=16, height=16, seed=side + M + each, frames=2)
    for f in range(2):
        planes = sc.atlas[f].reshape(sc.C, -1)
        k = np.random.default_rng(f).permutation(planes.shape[1])[:pixels * each]
        p = np.arange(k.size) % max(pixels, 1)              # pixel (p mod M, p / M + 1), its centre
        theta, phi = -np.pi + 2 * np.pi * (p % M + 0.5) / M, np.pi * (p // M + 1.5) / Nv
        planes[0:3, k] = np.stack([np.sin(phi) * np.cos(theta), np.sin(phi) * np.sin(theta), np.cos(phi)])
        planes[10] = np.round(planes[10] * 4) / 4           # many equal opacities
    for K in (1, 7):
        got, ref = run(sc, M, Nv, K), reference(sc, M, Nv, K)
        for a, b, what in zip(got, ref, ("uv", "rank", "keep")):
            assert np.array_equal(a.astype(np.int64), b.astype(np.int64)), what


@pytest.mark.parametrize("crowded", [1.0, 0.1])
def test_a_crowded_pixel_costs_no_more_than_the_sorts_do(crowded):
    """A count per Gaussian in one pixel took 11 ns each (0.4 M: 4.4 ms, a tenth of them
    0.5 ms), against some 0.08 ms for the same Gaussians spread evenly; 4 times the even map's
    time allows for the way from the lists to the sorts."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2602_23040_amd import _abi as abi
    print(f"[gpu] uv crowded {crowded}", flush=True)
    n, M, Nv, dev = 400000, 512, 256, "cuda:0"
    gen = torch.Generator(dev).manual_seed(1)
    ws = torch.empty(abi.pg_uv_prune_workspace_size(n, 1, M, Nv), dtype=torch.uint8, device=dev)
    count = torch.tensor([n], dtype=torch.int64, device=dev)
    uv, rank = (torch.empty(n, dtype=torch.int32, device=dev) for _ in range(2))
    keep = torch.empty(n, dtype=torch.uint8, device=dev)
    times = []
    for part in (0.0, crowded):
        params = torch.randn(14, n, device=dev, generator=gen)
        params[0:3, :int(part * n)] = torch.tensor([[0.5], [0.3], [0.1]], device=dev)
        best = 1e9
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            abi.pg_uv_prune(params, count, n, 1, 14, M, Nv, 4, None, uv, rank, keep, ws, ws.numel())
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b))
        times.append(best)
    print(f"[gpu] {times}", flush=True)
    assert times[1] <= 4 * times[0]
