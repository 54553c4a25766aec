"""Per-record sums of the gradient slots (the first pass of pg_project_bwd)
against FP64 sums of the same slots: records of one tile to hundreds, in the
few-record kernel (16 lanes per record, a wave for more than 256 tiles) and in
the streaming kernel (a thread per record, a wave for more than 64 tiles).

grad2d's colour channels are the sums themselves.  Adding at most a few
thousand floats in FP32 in any order is off by at most n 2^-24 of the sum of
magnitudes; the lanes' partial sums keep n near 300, so 2e-5 of the sum of
magnitudes bounds it."""
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


@pytest.mark.parametrize("side,views,w,h,lscale", [
    (1, 1, 640, 480, (0.0, 0.1)),          # one record over every tile
    (13, 2, 640, 480, (-2.5, 1.2)),        # 338 records: a few waves
    (40, 3, 640, 480, (-3.0, 1.0)),
    (170, 10, 320, 240, (-4.2, 1.2)),      # 289,000 records: the streaming kernel
])
def test_slot_sums(side, views, w, h, lscale):
    print(f"[gpu] slot sums side {side} {views} views {w}x{h}", flush=True)
    sc = synth.random_scene(side=side, sh_degree=0, views=views, width=w, height=h, seed=side, lscale=lscale,
                            lopac=(-2.0, 1.0))
    r = renderer(sc)
    run_forward(r, atlas_tensor(sc))
    g = torch.randn(r.image.shape, device="cuda:0", generator=torch.Generator("cuda:0").manual_seed(side))
    r.backward(g)
    s = r.sets[0]
    n, gen = (int(x) for x in s.n_inst.cpu())
    first = s.inst_first[:s.info.n_gv].cpu().numpy().astype(np.int64)
    nt = np.diff(np.append(first, n))
    slots = s.inst_grad[:10 * n].view(-1, 10).cpu().numpy()
    tagged = slots[:, 9].view(np.uint32) == np.uint32(gen)
    owner = np.repeat(np.arange(first.size), nt)[tagged]
    got = s.grad2d[:9 * first.size].view(9, -1).cpu().numpy().astype(np.float64)
    for ch in (6, 7, 8):
        x = slots[tagged, ch].astype(np.float64)
        ref = np.bincount(owner, x, first.size)
        mag = np.bincount(owner, np.abs(x), first.size)
        assert np.all(np.abs(got[ch] - ref) <= 2e-5 * mag + 1e-30)
    print(f"[gpu] most tiles of a record {int(nt.max())}, {int((nt > 64).sum())} above 64, "
          f"{int((nt > 256).sum())} above 256", flush=True)
    assert nt.max() > 256
    r.close()
