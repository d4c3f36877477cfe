"""The two forms of a call's preparation (light-curve points kept in registers or read twice): the
same bits for the same event whichever form its call takes."""
import numpy as np
import pytest
import torch

import paper_1511_01157_amd as M
from tests.helpers import note

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def batch(rng, lens):
    return [dict(tt=np.sort(rng.uniform(-30, 30, n)).astype(np.float32), F=2 + rng.standard_normal(n),
                 w=rng.uniform(50, 150, n), t_ref=rng.uniform(-2, 2)) for n in lens]


def run(maps, evs, P):
    r = M.search(maps, M.LightCurveBatch.from_events(evs, DEV), M.list_trajectories(P, shared=True), "batched", fs=True, fb=True)
    return [r[k].view(torch.int64) for k in ("chi2", "fs", "fb")]


def rows(rng, n):
    return torch.from_numpy(np.stack([rng.normal(0, 3, n), rng.uniform(0, 0.6, n), rng.uniform(8, 40, n),
                                      rng.uniform(0, 6.28, n)], 1)).to(DEV)


@pytest.mark.parametrize("n_events", [2047, 2048, 2049])
def test_many_events_equal_few(n_events):
    rng = np.random.default_rng(n_events)
    lens = rng.integers(3, 40, n_events)
    lens[[0, 5, 100, -1]] = [257, 4095, 4097, 4096]
    evs = batch(rng, lens)
    maps = [(torch.from_numpy((1 + 3 * rng.random((60, 70))).astype(np.float32)).to(DEV), (0.0, 0.0, 2.0, 1.7, 70, 60))]
    P = rows(rng, 7)
    note(f"prep forms {n_events} events")
    all_ = run(maps, evs, P)
    for a, b in ((0, 200), (n_events - 3, n_events)):
        for x, y in zip(all_, run(maps, evs[a:b], P)):
            assert torch.equal(x[a:b], y)


# cells in all just below and at 2^22
@pytest.mark.parametrize("ny", [2046, 2048, 2050])
def test_large_maps_equal_small(ny):
    rng = np.random.default_rng(ny)
    small = (torch.from_numpy((1 + 3 * rng.random((6, 10))).astype(np.float32)).to(DEV), (0.0, 0.0, 2.0, 1.7, 10, 6))
    large = (torch.from_numpy((1 + 3 * rng.random((ny, 2048))).astype(np.float32)).to(DEV), (0.0, 0.0, 2.0, 1.7, 2048, ny))
    evs = batch(rng, [3, 300, 5000])
    P = rows(rng, 50)
    note(f"prep forms 2048 x {ny}")
    both = run([small, large], evs, P)
    for x, y, z in zip(both, run([small], evs, P), run([large], evs, P)):
        assert torch.equal(x[:, :1], y) and torch.equal(x[:, 1:], z)
