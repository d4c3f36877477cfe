"""Every item of a batched search is scored once however the workgroups are dealt to the XCDs: counts
of trajectories about the lines between the deals (chunks that change places, chunks that do not,
chunks at their largest), ragged ends, shared and separate lists; against the plain mode."""
import numpy as np
import pytest
import torch

import paper_1511_01157_amd as M
from tests.helpers import note

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n", [4080, 4089, 4096, 4103, 9001, 32767, 32768, 32776, 40001])
@pytest.mark.parametrize("shared", [True, False])
def test_batched_equals_plain(n, shared):
    rng = np.random.default_rng(n)
    evs = [dict(tt=np.sort(rng.uniform(-30, 30, k)).astype(np.float32), F=2 + rng.standard_normal(k),
                w=rng.uniform(50, 150, k), t_ref=rng.uniform(-2, 2)) for k in (3, 70, 300)]
    lcs = M.LightCurveBatch.from_events(evs, DEV)
    maps = [(torch.from_numpy((1 + 3 * rng.random((50, 64))).astype(np.float32)).to(DEV), (cx, 0.0, 2.0, 1.7, 64, 50))
            for cx in (0.0, 0.1, 0.0)]
    P = np.stack([rng.normal(0, 4, 3 * n), rng.uniform(-1, 1, 3 * n), rng.uniform(5, 60, 3 * n), rng.uniform(-7, 7, 3 * n)], 1)
    P = torch.from_numpy(P[:n] if shared else P.reshape(3, n, 4)).to(DEV).contiguous()
    tr = M.list_trajectories(P, shared=shared)
    note(f"search deals {n} shared {shared}")
    out = {k: torch.full((3, 3, n), -7.0, dtype=torch.float64, device=DEV) for k in ("chi2", "fs", "fb")}
    b = M.search(maps, lcs, tr, "batched", fs=True, fb=True, out=dict(out))
    p = M.search(maps, lcs, tr, "plain", fs=True, fb=True)
    for k in out:
        assert torch.equal(p[k].view(torch.int64), b[k].view(torch.int64)), k
