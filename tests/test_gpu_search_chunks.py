"""The search's chunks of 64 points: light curves about the lengths where the forms change
(whole chunks, the first classified length, the 64-chunk segment), trajectories on the map,
off it, crossing its edge, times out of order, windows about the origin and off it.  Every
form computes the same binary32 samples, so plain and all batched shapes agree bit for bit,
and with the oracle's mirror within FP64 rounding of the sums."""
import json

import numpy as np
import pytest
import torch

import paper_1511_01157_amd as M
from oracle.search import search_mirror32
from tests.helpers import note, rel_err

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TU_SHAPES = {"tu4": 18, "tu2": 20, "tu1": 22, "tu4_items": 12}


def problem(npts, centre, order):
    rng = np.random.default_rng(npts)
    n = 96
    amap = (1.0 + 3.0 * rng.random((n, n - 14))).astype(np.float32)
    window = (*centre, 2.0, 1.7, n - 14, n)
    tt = np.sort(rng.uniform(-40.0, 40.0, npts)).astype(np.float32)
    if order == "reversed":
        tt = tt[::-1].copy()
    elif order == "shuffled":
        tt = rng.permutation(tt)
    F = 2.0 + rng.standard_normal(npts)
    ev = dict(tt=tt, F=F, w=rng.uniform(50.0, 150.0, npts), t_ref=0.0)
    k = 40
    # on the map throughout (slow), crossing it (fast), beside it throughout (u0 large)
    tE = np.concatenate([rng.uniform(60, 200, k), rng.uniform(4, 30, k), rng.uniform(5, 100, k + 3)])
    u0 = np.concatenate([rng.uniform(0, 0.3, k), rng.uniform(0, 0.6, k), rng.uniform(1.5, 4.0, k + 3)])
    P = np.stack([rng.uniform(-8, 8, len(tE)), u0, tE, rng.uniform(0, 2 * np.pi, len(tE))], 1)
    return amap, window, ev, P[rng.permutation(len(P))]


@pytest.mark.parametrize("npts,centre,order", [
    (3, (0.0, 0.0), "sorted"), (63, (0.0, 0.0), "sorted"), (255, (0.0, 0.0), "sorted"), (256, (0.0, 0.0), "sorted"),
    (257, (0.1, -0.05), "sorted"), (640, (0.0, 0.0), "sorted"), (1001, (0.0, 0.0), "reversed"),
    (1001, (0.0, 0.0), "shuffled"), (4096, (0.0, 0.0), "sorted"), (4097, (0.0, 0.2), "sorted"),
    (8300, (0.0, 0.0), "sorted")])
def test_every_shape_matches_the_mirror(npts, centre, order, tmp_path):
    amap, window, ev, P = problem(npts, centre, order)
    note(f"search chunks {npts} {centre} {order}")
    maps = [(torch.from_numpy(amap).to(DEV), window)]
    lcs = M.LightCurveBatch.from_events([ev], DEV)
    tr = M.list_trajectories(torch.from_numpy(P).to(DEV), shared=True)
    chi2, Fs, Fb, _ = search_mirror32(amap, window, ev["tt"], ev["F"], ev["w"], P, 0.0)
    ref = M.search(maps, lcs, tr, "plain", fs=True, fb=True)
    assert rel_err(ref["chi2"].cpu().numpy()[0, 0], chi2).max() < 1e-9
    path = tmp_path / "tune.json"
    M.autotune(maps, lcs, tr, cache_path=str(path))
    cls = list(json.loads(path.read_text()))[0]
    for name, shape in TU_SHAPES.items():
        path.write_text(json.dumps({cls: shape}))
        s = torch.cuda.Stream(device=DEV)
        c = M.Context.bound(s)
        assert M.autotune_load(str(path), ctx=c) == 1
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            r = M.search(maps, lcs, tr, "batched", fs=True, fb=True, ctx=c)
        s.synchronize()
        for k in ("chi2", "fs", "fb"):
            assert torch.equal(r[k], ref[k]), (name, k)


@pytest.mark.parametrize("shape", [(1, 1, 1, 1), (3, 5, 7, 2), (2, 9, 1, 6), (5, 1, 11, 1)])
def test_product_grids_of_any_axes(shape):
    """The scoring order of a grid puts t0 fastest; outputs stay in the index order."""
    amap, window, ev, _ = problem(700, (0.0, 0.0), "sorted")
    rng = np.random.default_rng(sum(shape))
    u0, al, t0, tE = (np.sort(rng.uniform(lo, hi, n)) for n, (lo, hi) in
                      zip(shape, [(0, 0.8), (0, 6.2), (-8, 8), (5, 90)]))
    note(f"search grid {shape}")
    maps = [(torch.from_numpy(amap).to(DEV), window)]
    lcs = M.LightCurveBatch.from_events([ev], DEV)
    P = np.stack([g.ravel() for g in np.meshgrid(u0, al, t0, tE, indexing="ij")], 1)[:, [2, 0, 3, 1]]
    chi2, _, _, _ = search_mirror32(amap, window, ev["tt"], ev["F"], ev["w"], np.ascontiguousarray(P), 0.0)
    tr = M.grid_trajectories(u0, al, t0, tE)
    a, b = M.search(maps, lcs, tr, "batched"), M.search(maps, lcs, tr, "plain")
    assert torch.equal(a["chi2"], b["chi2"])
    assert rel_err(a["chi2"].cpu().numpy()[0, 0], chi2).max() < 1e-9
