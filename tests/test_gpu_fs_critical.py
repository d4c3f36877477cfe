"""The critical curve of the finite-source magnification, solved on the GPU, through what
it decides: sources just inside and just outside `near` rho of the nearest caustic point at
the same phases take the image-centred and the point-source branch."""
import numpy as np
import pytest
import torch

import paper_1511_01157_amd as M
from oracle.lens import lens_setup
from tests.helpers import note

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def caustic_at_phases(s, q, n):
    """Caustic images of the critical points at n phases (numpy's companion matrices)."""
    m1, m2, x1, x2 = lens_setup(s, q)
    out = []
    for k in range(n):
        e = np.exp(-2j * np.pi * k / n)
        a = np.polymul([1.0, -x1], [1.0, -x1])
        b = np.polymul([1.0, -x2], [1.0, -x2])
        c = np.polysub(np.polyadd(m1 * b, m2 * a), e * np.polymul(a, b))
        z = np.roots(c)
        out.append(z - m1 / (z.conj() - x1) - m2 / (z.conj() - x2))
    return np.concatenate(out)


# close, resonant and wide topologies, equal masses, a planet; phase counts that leave the
# last wavefront of four-lane groups part full
@pytest.mark.parametrize("s,q,n_crit", [(0.6, 1.0, 16), (1.0, 0.3, 1024), (2.5, 1.0, 257), (0.8, 1e-5, 1000),
                                        (1.3, 1e-3, 4099)])
def test_branch_follows_the_distance_to_the_caustic(s, q, n_crit):
    note(f"fs critical points s={s} q={q} n_crit={n_crit}")
    caus = caustic_at_phases(s, q, n_crit)
    rng = np.random.default_rng(3)
    rho, near = 1e-3, 10.0
    z = caus[rng.integers(0, len(caus), 24)] + near * rho * rng.uniform(0.5, 1.5, 24) * np.exp(2j * np.pi * rng.uniform(0, 1, 24))
    # move each source along the line to its nearest point until it is 1e-6 inside / outside
    at = caus[np.abs(z[:, None] - caus[None, :]).argmin(1)]
    for side in (1 - 1e-6, 1 + 1e-6):
        zz = at + (z - at) * (near * rho * side / np.abs(z - at))
        dist = np.abs(zz[:, None] - caus[None, :]).min(1)
        zt = torch.from_numpy(np.stack([zz.real, zz.imag], 1)).to(DEV)
        _, nreg = M.fs_magnification(s, q, zt, rho, n_crit=n_crit, n_b=16, n_r=16, n_theta=16, n_side=8, near=near)
        far = nreg.cpu().numpy() == -1
        assert np.array_equal(far, dist > near * rho)
