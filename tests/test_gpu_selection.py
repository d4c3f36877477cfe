"""Best and top-k selection against the order of the scores themselves: segments about the
length that one workgroup sorts, lists about the sizes of the sort, scores that are equal in
more places than the list holds (trajectories repeated), NaN scores, more asked than there is."""
import numpy as np
import pytest
import torch

import paper_1511_01157_amd as M
from tests.helpers import note

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def problem(n, distinct, nan, n_maps, n_events):
    rng = np.random.default_rng(n + distinct)
    maps = [(torch.from_numpy((1 + 3 * rng.random((40, 40))).astype(np.float32)).to(DEV), (0.0, 0.0, 2.0, 2.0, 40, 40))
            for _ in range(n_maps)]
    evs = []
    for _ in range(n_events):
        tt = np.sort(rng.uniform(-30, 30, 70)).astype(np.float32)
        evs.append(dict(tt=tt, F=2 + rng.standard_normal(70), w=rng.uniform(50, 150, 70), t_ref=0.0))
    P = np.stack([rng.uniform(-5, 5, n), rng.uniform(0, 0.8, n), rng.uniform(5, 80, n), rng.uniform(0, 6.28, n)], 1)
    P[distinct:] = P[rng.integers(0, max(1, distinct // 50), n - distinct)]  # a few of them again and again
    P = P[rng.permutation(n)]
    P[rng.choice(n, nan, replace=False), 0] = np.nan
    return maps, M.LightCurveBatch.from_events(evs, DEV), M.list_trajectories(torch.from_numpy(P).to(DEV), shared=True)


@pytest.mark.parametrize("n,distinct,nan,n_maps,n_events,ks", [
    (1, 1, 0, 1, 1, (1, 5)), (2, 2, 1, 1, 1, (1, 3)), (65, 65, 3, 1, 2, (1, 64, 65, 66)),
    (1023, 1000, 0, 1, 1, (16, 1023)), (1025, 1025, 900, 1, 1, (200, 1025, 4096)),
    (4096, 3, 0, 2, 2, (1, 4096)), (4097, 4097, 0, 2, 2, (1, 256, 257, 511, 512, 4096)),
    (8192, 8000, 5, 1, 1, (4096,)), (8193, 8193, 8100, 1, 1, (64, 4096)), (8193, 1, 0, 1, 1, (1, 4096)),
    (30000, 60, 0, 1, 1, (1, 64, 4095, 4096)), (30000, 2000, 10, 3, 2, (16, 2500, 4096)),
    (700, 650, 3, 1, 9, (1, 64, 900)), (5000, 2600, 9, 2, 9, (300, 4096)),
    (150001, 150001, 0, 1, 1, (64, 4096)), (150001, 120, 0, 2, 1, (100, 4096))])
def test_selection_matches_the_order_of_the_scores(n, distinct, nan, n_maps, n_events, ks):
    maps, lcs, tr = problem(n, distinct, nan, n_maps, n_events)
    for k in ks:
        note(f"selection {n} {distinct} {nan} {n_maps} {n_events} k {k}")
        for mode in ("plain", "batched", "batched"):
            r = M.search(maps, lcs, tr, mode, best=True, top_k=k)
            g = r["chi2"].cpu().numpy()
            for e in range(n_events):
                for m in range(n_maps):
                    i = np.lexsort((np.arange(n), g[e, m]))[0]
                    assert int(r["best_idx"][e, m]) == i
                    assert np.array_equal(r["best_chi2"][e, m].cpu().numpy(), g[e, m, i], equal_nan=True)
                flat = g[e].reshape(-1)
                order = np.lexsort((np.arange(len(flat)), flat))[:k]
                want = np.full(k, -1)
                want[:len(order)] = order
                assert np.array_equal(r["topk_idx"][e].cpu().numpy(), want)
                vals = np.full(k, np.nan)
                vals[:len(order)] = flat[order]
                assert np.array_equal(r["topk_chi2"][e].cpu().numpy(), vals, equal_nan=True)
