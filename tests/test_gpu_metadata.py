"""Host metadata of a call (offsets, map table, grid axes) on its way to the device: sizes about
one launch's worth of it and about the size from which it is copied; calls in a captured graph,
replayed after other calls have put theirs."""
import numpy as np
import pytest
import torch

import paper_1511_01157_amd as M
from tests.helpers import note

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def problem(seed, npts=90):
    rng = np.random.default_rng(seed)
    amap = torch.from_numpy((1 + 3 * rng.random((50, 60))).astype(np.float32)).to(DEV)
    tt = np.sort(rng.uniform(-30, 30, npts)).astype(np.float32)
    ev = dict(tt=tt, F=2 + rng.standard_normal(npts), w=rng.uniform(50, 150, npts), t_ref=float(seed))
    return rng, [(amap, (0.0, 0.0, 2.0, 1.7, 60, 50))], M.LightCurveBatch.from_events([ev], DEV)


@pytest.mark.parametrize("n", [1, 420, 430, 431, 432, 433, 440, 1770, 1775, 1776, 1777, 1780, 4000])
def test_grid_axes_of_any_length_match_their_list(n):
    rng, maps, lcs = problem(n)
    u0 = rng.uniform(0, 0.8, n)
    note(f"metadata axes {n}")
    grid = M.grid_trajectories(u0, [0.7], [1.5], [20.0])
    rows = np.stack([np.full(n, 1.5), u0, np.full(n, 20.0), np.full(n, 0.7)], 1)
    lst = M.list_trajectories(torch.from_numpy(rows).to(DEV), shared=True)
    for mode in ("plain", "batched"):
        a = M.search(maps, lcs, grid, mode, fs=True, best=True, top_k=5)
        b = M.search(maps, lcs, lst, mode, fs=True, best=True, top_k=5)
        for k in a:
            assert torch.equal(a[k].view(torch.int64), b[k].view(torch.int64)), k
    cand, _, _ = M.candidates_from_topk(grid, a["topk_idx"], 1)
    want = rows[a["topk_idx"].cpu().numpy()[0].clip(0)]
    assert np.array_equal(cand.cpu().numpy().reshape(want.shape), want)


@pytest.mark.parametrize("noalloc", [False, True])
def test_captured_calls_bring_their_metadata(noalloc):
    _, maps, lcs = problem(3)
    rng, other_maps, other = problem(4)
    P = torch.from_numpy(np.stack([rng.normal(3, 2, 40), rng.uniform(0, 0.6, 40), rng.uniform(8, 40, 40),
                                   rng.uniform(0, 6.28, 40)], 1)).to(DEV)
    z = torch.zeros(40, dtype=torch.int32, device=DEV)
    tr = M.list_trajectories(P, shared=True)
    s = torch.cuda.Stream(device=DEV)
    note(f"metadata capture noalloc={noalloc}")

    def calls(m, l):
        r = M.search(m, l, tr, "batched", best=True, top_k=7)
        c = M.chi2_grad(m, l, P, z, z, noalloc=noalloc)
        return [r["chi2"], r["best_idx"], r["topk_idx"], *c]

    with torch.cuda.stream(s):
        want = [x.clone() for x in calls(maps, lcs)]
        calls(other_maps, other)  # the last metadata put before the capture is another's
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            got = calls(maps, lcs)
        for rep in range(3):
            alone = [x.clone() for x in calls(other_maps, other)]
            assert not torch.equal(alone[0], want[0])
            for x in got:
                x.zero_()
            g.replay()
            s.synchronize()
            for a, b in zip(got, want):
                assert torch.equal(a, b), rep
            # eager calls after it, on what the replay replaced and on what it put
            for a, b in zip(calls(other_maps, other), alone):
                assert torch.equal(a, b), rep
            g.replay()
            for a, b in zip(calls(maps, lcs), want):
                assert torch.equal(a, b), rep
