"""Convolution at the sizes where its kernels change: transforms of every power-of-two height
and width (one wide pass, two, narrow remainders, columns that do not fill a workgroup), and
direct stencils of unequal half-widths on maps that do not fill a tile."""
import numpy as np
import pytest
import torch

import paper_1511_01157_amd as M
from oracle.maps import normalize_convolve_exact64
from oracle.profiles import ld_pixel_weights
from tests.helpers import note

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def problem(mx, my, dx, dy, seed):
    rng = np.random.default_rng(seed)
    counts = rng.integers(0, 4000, (my, mx)).astype(np.int32)
    win = (0.0, 0.0, mx * dx, my * dy, mx, my)
    rays = (0.0, 0.0, 2 * mx * dx, 2 * my * dy, 30 * mx, 30 * my)
    s64 = float(np.float32(rays[2] / rays[4])) * float(np.float32(rays[3] / rays[5])) / ((win[2] / mx) * (win[3] / my))
    return counts, win, rays, s64


@pytest.mark.parametrize("mx,my", [(4, 4), (20, 12), (30, 26), (18, 60), (100, 120), (250, 250), (12, 500), (500, 12),
                                   (26, 1000), (1000, 26), (12, 2000), (2000, 12), (10, 4000), (4000, 10), (300, 700)])
def test_transform_heights_and_widths(mx, my):
    dx, dy = 0.011, 0.013
    counts, win, rays, s64 = problem(mx, my, dx, dy, mx + my)
    rhos = [0.021, 0.034, 0.015]
    note(f"stack transform {mx} x {my}")
    got = M.convolve_stack(torch.from_numpy(counts).to(DEV), rays, win, rhos, 0.4, fft_min_taps=1)
    for k, rho in enumerate(rhos):
        ref = normalize_convolve_exact64(counts, s64, ld_pixel_weights(rho, win[2] / mx, win[3] / my, 0.4))
        g = got[k].cpu().numpy().astype(np.float64)
        # rounded once from FP64: within one unit in the last place, and the transform's error
        ulp = np.spacing(ref.astype(np.float32)).astype(np.float64)
        assert np.all(np.abs(g - ref) <= ulp + 1e-13 * ref.max()), rho


@pytest.mark.parametrize("mx,my", [(2, 2), (6, 4), (64, 32), (66, 34), (62, 30), (130, 100)])
@pytest.mark.parametrize("rx,ry", [(2, 1), (1, 2), (3, 3), (4, 9), (15, 2), (2, 15), (15, 15)])
def test_direct_stencils(mx, my, rx, ry):
    rho = 0.05
    dx, dy = rho / (rx - 0.4), rho / (ry - 0.4)
    counts, win, rays, s64 = problem(mx, my, dx, dy, 100 * rx + ry)
    note(f"direct stencil {mx} x {my}, {rx} x {ry}")
    for gamma in (0.0, 0.53):
        got = M.convolve_stack(torch.from_numpy(counts).to(DEV), rays, win, [rho], gamma, fft_min_taps=2**31 - 1)[0]
        w = ld_pixel_weights(rho, win[2] / mx, win[3] / my, gamma)
        ref = normalize_convolve_exact64(counts, s64, w)
        # rounded weights, products, the sequential sum of n terms, rounded scale, last product
        tol = (np.count_nonzero(w) + 3) * 2.0**-24
        g = got.cpu().numpy().astype(np.float64)
        assert np.all(np.abs(g - ref) <= tol * ref + 1e-12 * ref.max())
