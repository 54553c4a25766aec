"""The photometric loss by strips of 16, 32, 64 and 192 rows, whichever its rule of view
sizes takes, against FP64 under the rules of test_gpu_photo_strips.py.  The rule is
stated here as well, so that each table is known to take its height."""
import pytest
import torch

from test_gpu_photo_strips import RAGGED, test_strips_match_fp64 as check

pytestmark = pytest.mark.gpu


def rows_of(sizes):
    def count(c, r):
        return [-(-w // c) * -(-h // r) for w, h in sizes]

    def time(rows, ns):
        steps, n = [min(rows, h) + 20 for _, h in sizes], count(54, rows)
        return max(1e-3 * ns * sum(a * b for a, b in zip(n, steps)), (60 + 0.034 * sum(n)) * max(steps) / 52)

    times = {192: time(192, 1.72), 64: time(64, 1.62), 32: time(32, 1.75), 16: time(16, 1.75)}
    return min(times, key=times.get) if sum(count(32, 32)) > 512 else 0


@pytest.mark.parametrize("lam", [0.0, 0.2, 1.0])
@pytest.mark.parametrize("rows,sizes", [
    (16, RAGGED), (16, [(640, 480), (641, 481), (53, 17), (55, 15)]), (32, RAGGED + [(1024, 768)]),
    (32, [(110, 110)] * 99 + [(53, 140)]), (64, [(400, 300)] * 19 + [(640, 65), (55, 700)]),
    (192, [(108, 760)] * 160 + [(107, 191), (55, 193), (54, 1000), (500, 385)])],
    ids=["16 rows", "16 rows even", "32 rows", "32 rows small", "64 rows", "192 rows"])
def test_each_height_matches_fp64(rows, sizes, lam):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    assert rows_of(sizes) == rows
    check(sizes, lam)
