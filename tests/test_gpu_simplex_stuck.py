"""Simplices that a shrink no longer moves end with the result and the counts of the run to
max_iter: starts that give no chi-square (NaN), and vertices one unit in the last place
apart at absolute dates, across a step of the binary32 samples."""
import numpy as np
import pytest
import torch

import paper_1511_01157_amd as M
import workloads as W
from oracle.simplex import line_simplex
from tests.helpers import note

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def setup(amap):
    win = W.config("tiny")["window"]
    ev = dict(W.load_lightcurve("tiny"))
    shift = 2456000.0
    ev["t_ref"] = ev["t_ref"] + shift
    rng = np.random.default_rng(8)
    n = 400
    phi = rng.uniform(0, 2 * np.pi, n)
    lines = np.stack([rng.uniform(0, 0.3, n), phi, 0.05 * np.cos(phi)], 1)
    start = np.stack([shift + 0.4 * rng.standard_normal(n), 20.0 * np.exp(0.05 * rng.standard_normal(n))], 1)
    start[3] = np.nan
    start[7, 1] = np.nan

    def run(max_iter, ftol):
        res = M.line_simplex([(torch.from_numpy(np.ascontiguousarray(amap)).to(DEV), win)],
                             M.LightCurveBatch.from_events([ev], DEV), torch.from_numpy(lines).to(DEV),
                             torch.from_numpy(start).to(DEV), max_iter=max_iter, ftol=ftol)
        return [x.cpu().numpy()[:, 0] for x in res]
    return run, ev, win, lines, start


@pytest.mark.parametrize("max_iter", [0, 1, 70])
def test_stuck_simplices_match_the_oracle(tiny_oracle_map, max_iter):
    _, _, amap = tiny_oracle_map
    run, ev, win, lines, start = setup(amap)
    note(f"stuck simplices max_iter={max_iter}")
    chi2, t0, tE, it, ne = run(max_iter, 1e-10)
    for k in (3, 7):
        assert chi2[k] == np.inf and it[k] == max_iter and ne[k] == 3 + 4 * max_iter
    args = (ev["tt"], ev["F"], ev["w"], ev["t_ref"])
    for k in [k for k in np.flatnonzero(it == max_iter) if k not in (3, 7)][:4]:
        o = line_simplex(amap, win, *args, lines[k], start[k], (2.0, 0.2), max_iter, 1e-10)
        assert o[3] == it[k] and o[4] == ne[k]
        assert abs(o[2] / chi2[k] - 1) < 1e-9


def test_one_more_iteration_adds_its_four_evaluations(tiny_oracle_map):
    """With ftol 0 a simplex stops only on equal values: those that reach max_iter are stuck,
    and one iteration more changes nothing but the counts."""
    _, _, amap = tiny_oracle_map
    run = setup(amap)[0]
    note("stuck simplices, ftol 0")
    a, b = run(600, 0.0), run(601, 0.0)
    stuck = (a[3] == 600) & (b[3] == 601)
    assert stuck.sum() >= 2 and np.array_equal(stuck, a[3] == 600)
    for x, y in zip(a[:3], b[:3]):
        assert np.array_equal(x, y, equal_nan=True)
    assert np.array_equal(b[4] - a[4], np.where(stuck, 4, 0))
