"""Ray shooting at its edges.  Statistics where tiles are skipped unseen: rays whose offset from the window overflows
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


# windows of a few columns or rows: a tile's box of bins is narrow; 16 and 17 columns about the line
# between the two ways through it
@pytest.mark.parametrize("nx,ny", [(2, 8192), (8192, 2), (16, 3000), (18, 3000), (3000, 34), (6, 6)])
@pytest.mark.parametrize("cy", [0.0, 0.01])
def test_narrow_windows_count_exactly(nx, ny, cy):
    s, q, rays, window = 0.8, 0.01, (0.0, cy, 4.0, 4.0, 1500, 1400), (0.0, 0.0, 2.0, 2.0, nx, ny)
    note(f"ray statistics narrow window {nx} x {ny} cy={cy}")
    counts = torch.empty((ny, nx), dtype=torch.int32, device=DEV)
    stats = torch.zeros(3, dtype=torch.int64, device=DEV)
    M.rayshoot(s, q, rays, window, counts, stats=stats)
    o, ost = rayshoot_mirror32_c(s, q, rays, window, nthreads=8)
    assert np.array_equal(counts.cpu().numpy().view(np.uint32), o) and o.sum() > 0
    assert dict(zip(("out", "nonfinite", "zero_axis"), stats.tolist())) == ost


# lattices of about a ray a pixel: both sides of the line to the coarse form (1.5 to 2 rays a pixel
# side), on and off the lens axis, with a row on it (the IEEE division), ragged tiles
@pytest.mark.parametrize("rays_per_pixel", [0.4, 0.75, 1.0, 1.4, 1.9, 2.1])
@pytest.mark.parametrize("s,q,cx,cy,rows", [(0.9, 0.01, 0.0, 0.0, 1026), (1.3, 0.2, 0.1, 0.05, 1000), (1.2, 0.5, 0.0, 2.0 ** -9, 1024)])
def test_coarse_lattices_count_exactly(rays_per_pixel, s, q, cx, cy, rows):
    n = int(500 / rays_per_pixel) // 2 * 2
    rays, window = (cx, cy, 4.0, 4.0, 1000, rows), (2 * cx, 0.0, 2.0, 2.0, n, n - 2)
    note(f"ray statistics coarse {rays_per_pixel} s={s}")
    counts = torch.empty((n - 2, n), dtype=torch.int32, device=DEV)
    stats = torch.zeros(3, dtype=torch.int64, device=DEV)
    M.rayshoot(s, q, rays, window, counts, stats=stats)
    o, ost = rayshoot_mirror32_c(s, q, rays, window, nthreads=8)
    assert np.array_equal(counts.cpu().numpy().view(np.uint32), o) and o.sum() > 0
    assert dict(zip(("out", "nonfinite", "zero_axis"), stats.tolist())) == ost
