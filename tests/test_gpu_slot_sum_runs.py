"""The streaming kernel of the slot sums (more than 2^16 records) where long records,
short ones and ones without slots lie side by side, under the rule of
test_gpu_slot_sum.py: runs of long records over whole work-groups and their ends,
short ones between them, views that see only part of the Gaussians."""
import pytest
import torch

from test_gpu_slot_sum import test_slot_sums as check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("side,views,w,h,lscale", [
    (150, 3, 800, 600, (-2.9, 0.5)),       # about half above 64 tiles
    (150, 3, 800, 600, (-2.0, 0.5)),       # nearly all
    (257, 1, 640, 480, (-3.5, 0.8)),       # some
    (150, 3, 640, 480, (-1.0, 3.0)),       # every length
])
def test_runs_of_long_records(side, views, w, h, lscale):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    check(side, views, w, h, lscale)
