"""The allocation-free gradient with metadata of sizes about that up to which it goes by value,
and far beyond: the same bits as the ordinary entry point, also captured."""
import numpy as np
import pytest
import torch

import paper_1511_01157_amd as M
from tests.helpers import note

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# 16 bytes an event, 104 a map, 512 of rounding: 14336 bytes lie near 850 events
@pytest.mark.parametrize("n_events", [1, 830, 840, 850, 860, 880, 900, 30000])
def test_noalloc_equals_the_ordinary_gradient(n_events):
    rng = np.random.default_rng(n_events)
    n = 4 * n_events
    lcs = M.LightCurveBatch(torch.from_numpy(np.sort(rng.uniform(-30, 30, (n_events, 4)).astype(np.float32), 1).ravel()).to(DEV),
                            torch.from_numpy(2 + rng.standard_normal(n)).to(DEV), torch.from_numpy(rng.uniform(50, 150, n)).to(DEV),
                            np.arange(0, n + 1, 4), rng.uniform(-1, 1, n_events))
    maps = [(torch.from_numpy((1 + 3 * rng.random((40, 60))).astype(np.float32)).to(DEV), (0.0, 0.0, 2.0, 1.7, 60, 40))]
    P = torch.from_numpy(np.stack([rng.normal(0, 3, 64), rng.uniform(0, 0.6, 64), rng.uniform(8, 40, 64),
                                   rng.uniform(0, 6.28, 64)], 1)).to(DEV)
    ev = torch.from_numpy(rng.integers(0, n_events, 64).astype(np.int32)).to(DEV)
    ev[0] = n_events - 1
    mi = torch.zeros(64, dtype=torch.int32, device=DEV)
    note(f"noalloc metadata of {n_events} events")
    want = M.chi2_grad(maps, lcs, P, ev, mi)
    s = torch.cuda.Stream(device=DEV)
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        got = M.chi2_grad(maps, lcs, P, ev, mi, noalloc=True)
        for a, b in zip(got, want):
            assert torch.equal(a.view(torch.int64), b.view(torch.int64))
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            got = M.chi2_grad(maps, lcs, P, ev, mi, noalloc=True)
        for rep in range(3):
            for x in got:
                x.zero_()
            g.replay()
            s.synchronize()
            for a, b in zip(got, want):
                assert torch.equal(a.view(torch.int64), b.view(torch.int64)), rep
