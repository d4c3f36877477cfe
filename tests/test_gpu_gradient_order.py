"""Gradients of more candidates than are evaluated in their own order: the same bits as those of
the pieces that are, also without allocation, about the count at which the line lies, for one
map and several, with events and maps out of range and parameters that are not finite."""
import numpy as np
import pytest
import torch

import paper_1511_01157_amd as M
from tests.helpers import note

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n,n_maps,n_events", [(2048, 2, 3), (2049, 2, 3), (2049, 1, 1), (2049, 1, 3),
                                               (9001, 3, 1100), (40003, 3, 3)])
def test_ordered_gradient_equals_pieces(n, n_maps, n_events):
    rng = np.random.default_rng(n + n_events)
    maps = [(torch.from_numpy((1 + 3 * rng.random((70, 62))).astype(np.float32)).to(DEV), (0.0, 0.0, 1.8, 1.5, 62, 70))
            for _ in range(n_maps)]
    evs = []
    for k in range(n_events):
        npts = (5, 130, 300)[k % 3] if n_events < 10 else 3 + k % 5
        tt = np.sort(rng.uniform(-30, 30, npts)).astype(np.float32)
        evs.append(dict(tt=tt, F=2 + rng.standard_normal(npts), w=rng.uniform(50, 150, npts), t_ref=rng.uniform(-1, 1)))
    lcs = M.LightCurveBatch.from_events(evs, DEV)
    P = np.stack([rng.normal(0, 3, n), rng.uniform(0, 0.6, n), rng.uniform(8, 40, n), rng.uniform(0, 6.28, n)], 1)
    P[7, 0], P[8, 2], P[9, 3], P[n - 1, 1] = np.nan, 0.0, np.inf, 1e300
    ev, mi = rng.integers(0, n_events, n).astype(np.int32), rng.integers(0, n_maps, n).astype(np.int32)
    ev[3], mi[5], ev[31], mi[n - 2] = n_events, -1, -2, n_maps
    P, ev, mi = (torch.from_numpy(x).to(DEV) for x in (P, ev, mi))
    note(f"gradient order {n} {n_maps} {n_events}")
    parts = [M.chi2_grad(maps, lcs, P[i:i + 1024].contiguous(), ev[i:i + 1024].contiguous(), mi[i:i + 1024].contiguous())
             for i in range(0, n, 1024)]
    want = [torch.cat(x) for x in zip(*parts)]
    for noalloc in (False, True):
        for _ in range(2):
            got = M.chi2_grad(maps, lcs, P, ev, mi, noalloc=noalloc)
            for a, b in zip(got, want):
                assert torch.equal(a.view(torch.int64), b.view(torch.int64)), noalloc
