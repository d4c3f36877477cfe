"""Refinements of counts about those from which a workgroup takes four candidates (fewer where the
mean light curve has at most 1024 points): the same bits as those of a few at a time, with a
last workgroup that is not full, events of very different lengths and rows out of range."""
import numpy as np
import pytest
import torch

import paper_1511_01157_amd as M
from tests.helpers import note

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n,longest", [(6143, 700), (6144, 700), (6145, 700), (6147, 700),
                                       (16383, 3000), (16384, 3000), (16387, 3000)])
@pytest.mark.parametrize("steps,history", [(0, 8), (9, 2)])
def test_many_equal_few(n, longest, steps, history):
    rng = np.random.default_rng(n + steps)
    maps = [(torch.from_numpy((1 + 3 * rng.random((90, 96))).astype(np.float32)).to(DEV), (0.0, 0.0, 1.6, 1.5, 96, 90))
            for _ in range(2)]
    evs = []
    for npts in (5, 130, longest):
        tt = np.sort(rng.uniform(-30, 30, npts)).astype(np.float32)
        evs.append(dict(tt=tt, F=2 + rng.standard_normal(npts), w=rng.uniform(50, 150, npts), t_ref=0.0))
    lcs = M.LightCurveBatch.from_events(evs, DEV)
    P = np.stack([rng.normal(0, 3, n), rng.uniform(0, 0.6, n), rng.uniform(8, 40, n), rng.uniform(0, 6.28, n)], 1)
    ev, mi = rng.integers(0, 3, n).astype(np.int32), rng.integers(0, 2, n).astype(np.int32)
    ev[3], mi[5], ev[31], mi[n - 1] = 3, -1, -2, 2  # out of range
    dP, de, dm = (torch.from_numpy(x).to(DEV) for x in (P, ev, mi))
    note(f"refine counts {n} {longest} {steps} {history}")
    got = M.refine(maps, lcs, dP, de, dm, steps=steps, history=history)
    for i in range(0, n, 2500):
        want = M.refine(maps, lcs, dP[i:i + 2500].contiguous(), de[i:i + 2500].contiguous(),
                        dm[i:i + 2500].contiguous(), steps=steps, history=history)
        for a, b in zip(got, want):
            assert torch.equal(a[i:i + 2500].contiguous().view(torch.int64), b.view(torch.int64)), i
