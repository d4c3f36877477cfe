"""Ray shooting over the forms of its kernel: small and large tiles, tiles skipped because
no ray can reach the window, the short and the IEEE division, ragged ends.  Counts are
integers, so every comparison with the binary32 mirror is exact."""
import numpy as np
import pytest
import torch

import paper_1511_01157_amd as M
from oracle.rays import rayshoot_mirror32_c
from tests.helpers import note

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = {
    # large tiles (at least 4 rays a pixel side, over 2048 tiles), ragged, off the axis
    "large_off_axis": (0.9, 0.03, (0.11, -0.07, 5.0, 4.4, 5002, 4210), (0.05, 0.02, 1.9, 1.7, 300, 270)),
    "large_mirror": (1.1, 0.02, (0.0, 0.0, 6.0, 6.0, 7170, 5122), (0.2, 0.0, 2.0, 2.2, 310, 250)),
    # a window that only the deflected rays of a few tiles reach
    "window_aside": (1.3, 0.2, (0.0, 0.0, 8.0, 8.0, 2050, 2046), (2.6, 1.9, 0.5, 0.4, 64, 48)),
    # a coarse lattice: boxes beyond the LDS histogram count ray by ray
    "coarse": (0.8, 0.01, (0.0, 0.01, 4.0, 4.0, 640, 600), (0.0, 0.0, 3.0, 3.0, 1024, 1000)),
    # a row on the lens axis and a ray on the lens: the IEEE division, non-finite rays
    "ray_on_lens": (1.0, 0.0, (2.0 ** -9, 2.0 ** -9, 4.0, 4.0, 1024, 1024), (0.0, 0.0, 2.0, 2.0, 128, 128)),
    "row_on_axis": (1.2, 0.5, (0.0, 2.0 ** -10, 4.0, 4.0, 2048, 2048), (0.0, 0.0, 2.0, 2.0, 256, 256)),
}


@pytest.mark.parametrize("name", CASES)
def test_counts_and_statistics_exact(name):
    s, q, rays, window = CASES[name]
    note(f"ray tiles {name}")
    counts = torch.empty((window[5], window[4]), dtype=torch.int32, device=DEV)
    stats = torch.zeros(3, dtype=torch.int64, device=DEV)
    M.rayshoot(s, q, rays, window, counts, stats=stats)
    o, ost = rayshoot_mirror32_c(s, q, rays, window, nthreads=8)
    assert np.array_equal(counts.cpu().numpy().view(np.uint32), o)
    assert dict(zip(("out", "nonfinite", "zero_axis"), stats.tolist())) == ost
    assert o.sum() > 0
    if name == "ray_on_lens":
        assert ost["nonfinite"] > 0
