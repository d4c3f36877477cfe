"""Bounds of the nodes inside the source, on grids whose columns leave a wavefront part full or
alone and whose radial nodes end within a look of eight: each cut decides the next grid, so the
magnification of many cuts matches the oracle's only if every one is the oracle's."""
import numpy as np
import pytest
import torch

import paper_1511_01157_amd as M
from oracle.caustics import caustic_points
from oracle.fsmag import FsOptions, fs_magnification
from tests.helpers import note

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n_r,n_theta", [(6, 63), (7, 64), (8, 65), (9, 8), (15, 127), (16, 257), (33, 40), (257, 300)])
@pytest.mark.parametrize("gamma", [0.0, 0.53])
def test_cut_grids_match_the_oracle(n_r, n_theta, gamma):
    s, q, rho = 1.2, 0.3, 0.02
    cc = np.asarray(caustic_points(s, q, 2048)).reshape(-1)
    cc = cc[np.isfinite(cc)]
    rng = np.random.default_rng(n_r)
    z = cc[rng.integers(0, len(cc), 6)] + rho * (rng.normal(0, 0.8, 6) + 1j * rng.normal(0, 0.8, 6))
    kw = dict(n_b=64, n_side=32, n_grow=20, n_r=n_r, n_theta=n_theta, n_shrink=4)
    note(f"fs boxes {n_r} x {n_theta} gamma {gamma}")
    A, nreg = M.fs_magnification(s, q, torch.from_numpy(np.stack([z.real, z.imag], 1).copy()).to(DEV), rho, gamma, **kw)
    A, nreg = A.cpu().numpy(), nreg.cpu().numpy()
    for k, zk in enumerate(z):
        oA, d = fs_magnification(zk, rho, gamma, s, q, opt=FsOptions(**kw), details=True)
        assert nreg[k] == (-1 if d["point_source"] else len(d["regions"])), k
        assert abs(A[k] - oA) <= 1e-8 * abs(oA), (k, A[k], oA)
    assert (nreg > 0).sum() >= 3
