"""The kept-line list at the sizes where its kernels change (16 flags a lane, 16384 a tile,
eight tiles), against the keep flags; the filter's and the peak library's samples on windows
about the origin and off it, with line lengths that leave chunks of four part full."""
import numpy as np
import pytest
import torch

import paper_1511_01157_amd as M
from oracle.lines import line_filter_mirror32, line_peaks_mirror32
from tests.helpers import note

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def problem(n, centre, size, seed=5):
    rng = np.random.default_rng(seed)
    amap = (1.0 + rng.random(size[::-1])).astype(np.float32)
    window = (*centre, 1.5, 1.5 * size[1] / size[0], *size)
    lines = np.stack([rng.uniform(-0.9, 0.9, n), rng.uniform(0, 2 * np.pi, n), rng.uniform(-0.1, 0.1, n)], 1)
    return amap, window, lines


@pytest.mark.parametrize("n", [1, 15, 16, 17, 1023, 16384, 16385, 131072, 131073])
def test_kept_list_is_the_set_flags_in_order(n):
    amap, window, lines = problem(n, (0.0, 0.0), (8, 8))
    note(f"kept list n={n}")
    best, keep, kept = M.line_filter(torch.from_numpy(amap).to(DEV), window, torch.from_numpy(lines).to(DEV), 1.9)
    assert torch.equal(kept, keep.nonzero()[:, 0])
    assert torch.equal(keep.bool(), best >= np.float32(1.9))


@pytest.mark.parametrize("centre", [(0.0, 0.0), (0.3, -0.2)])
@pytest.mark.parametrize("size", [(2, 2), (44, 46), (46, 46), (90, 64), (182, 180)])
def test_samples_bitwise_equal_to_the_mirror(centre, size):
    amap, window, lines = problem(37, centre, size)
    note(f"line samples {centre} {size}")
    d, L = torch.from_numpy(amap).to(DEV), torch.from_numpy(lines).to(DEV)
    ob, ok = line_filter_mirror32(amap, window, lines, 1.5)
    best, keep, _ = M.line_filter(d, window, L, 1.5)
    assert np.array_equal(best.cpu().numpy(), ob) and np.array_equal(keep.cpu().numpy().astype(bool), ok)
    for h in (0.0, 0.3):
        cnt, ptau, pA, ob = line_peaks_mirror32(amap, window, lines, h, 5)
        g = M.line_peaks(d, window, L, 1.5, min_peaks=2, hysteresis=h, max_peaks=5)
        for x, y in zip(g, (ob, cnt, ptau, pA, (ob >= np.float32(1.5)) & (cnt >= 2))):
            assert np.array_equal(x.cpu().numpy().astype(y.dtype), y, equal_nan=y.dtype.kind == "f")
