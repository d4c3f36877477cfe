"""Ray statistics where tiles are skipped unseen: rays whose offset from the window overflows
binary32 are non-finite in the kernel's arithmetic, however far from the window their tile lies."""
import numpy as np
import pytest
import torch

import paper_1511_01157_amd as M
from oracle.rays import rayshoot_mirror32_c
from tests.helpers import note

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = {
    "all_but_the_centre": (1.0, 0.1, (0.0, 0.0, 1e36, 1e36, 512, 512), (0.0, 0.0, 1e-3, 1e-3, 64, 64)),
    "columns_only": (1.0, 0.1, (0.0, 0.0, 1e30, 4.0, 512, 512), (0.0, 0.0, 1e-9, 1e-9, 64, 64)),
    "rows_only": (1.0, 0.0, (0.0, 1.0, 4.0, 1e32, 500, 514), (0.0, 0.0, 1e-7, 1e-7, 64, 66)),
    # far beyond the window and still finite: outside
    "finite_rows": (1.0, 0.0, (0.0, 1.0, 4.0, 1e32, 500, 514), (0.0, 0.0, 1e-7, 2.0, 64, 66)),
    "finite": (1.0, 0.1, (0.0, 0.0, 1e36, 1e36, 512, 512), (0.0, 0.0, 2.0, 2.0, 64, 64)),
}


@pytest.mark.parametrize("name", CASES)
def test_overflowing_rays_count_as_nonfinite(name):
    s, q, rays, window = CASES[name]
    note(f"ray statistics {name}")
    counts = torch.empty((window[5], window[4]), dtype=torch.int32, device=DEV)
    stats = torch.zeros(3, dtype=torch.int64, device=DEV)
    M.rayshoot(s, q, rays, window, counts, stats=stats)
    o, ost = rayshoot_mirror32_c(s, q, rays, window, nthreads=8)
    assert np.array_equal(counts.cpu().numpy().view(np.uint32), o)
    assert dict(zip(("out", "nonfinite", "zero_axis"), stats.tolist())) == ost
    assert (ost["nonfinite"] > 0) == (not name.startswith("finite"))
