"""All rounds of a refinement in one launch: equal, bit for bit, to the rounds launched one by
one (state kept in between) and to the candidates in another order, for history rings that
wrap, none or many rounds, counts about the one from which an order is laid, events of very
different lengths, rows out of range; and to the oracle's state machine for short histories."""
import numpy as np
import pytest
import torch

import paper_1511_01157_amd as M
import workloads as W
from oracle.lbfgs import LbfgsOptions, refine as oracle_refine
from tests.helpers import note, rel_err

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def bits(*xs):
    return [x.view(torch.int64) for x in xs]


@pytest.mark.parametrize("n,steps,history", [(1, 7, 8), (33, 0, 8), (33, 30, 1), (40, 60, 3), (64, 40, 16),
                                             (2048, 12, 8), (2049, 12, 8), (2600, 20, 5), (32767, 6, 8),
                                             (32769, 6, 8), (32770, 9, 2), (32771, 0, 8)])
def test_one_launch_equals_round_by_round(n, steps, history):
    rng = np.random.default_rng(n + steps)
    maps = [(torch.from_numpy((1 + 3 * rng.random((90, 96))).astype(np.float32)).to(DEV), (0.0, 0.0, 1.6, 1.5, 96, 90))
            for _ in range(2)]
    evs = []
    for npts in (5, 130, 700):
        tt = np.sort(rng.uniform(-30, 30, npts)).astype(np.float32)
        evs.append(dict(tt=tt, F=2 + rng.standard_normal(npts), w=rng.uniform(50, 150, npts), t_ref=0.0))
    lcs = M.LightCurveBatch.from_events(evs, DEV)
    P = np.stack([rng.normal(0, 3, n), rng.uniform(0, 0.6, n), rng.uniform(8, 40, n), rng.uniform(0, 6.28, n)], 1)
    ev, mi = rng.integers(0, 3, n).astype(np.int32), rng.integers(0, 2, n).astype(np.int32)
    if n > 32:
        ev[3], mi[5], ev[31] = 3, -1, -2  # out of range
    dP, de, dm = torch.from_numpy(P).to(DEV), torch.from_numpy(ev).to(DEV), torch.from_numpy(mi).to(DEV)
    note(f"refine rounds {n} {steps} {history}")
    one = M.refine(maps, lcs, dP, de, dm, steps=steps, history=history)
    perm = torch.from_numpy(rng.permutation(n)).to(DEV)
    other = M.refine(maps, lcs, dP[perm].contiguous(), de[perm], dm[perm], steps=steps, history=history)
    for a, b in zip(bits(*one), bits(*other)):
        assert torch.equal(a[perm], b)
    ctx = M.Context.get(0)
    ctx.set_timing([M.KERNEL_GRADIENT])
    try:
        many = M.refine(maps, lcs, dP, de, dm, steps=steps, history=history)
        torch.cuda.synchronize()
    finally:
        ctx.set_timing([])
    assert ctx.kernel_time(M.KERNEL_GRADIENT, reset=True)[1] == steps + 1
    for a, b in zip(bits(*one), bits(*many)):
        assert torch.equal(a, b)
    bad = np.zeros(n, bool)
    if n > 32:
        bad[[3, 5, 31]] = True
    chi2, chi2_0 = one[1].cpu().numpy(), one[2].cpu().numpy()
    assert np.isnan(chi2[bad]).all() and np.all(chi2[~bad] <= chi2_0[~bad])


@pytest.mark.parametrize("history", [1, 3])
def test_short_histories_follow_the_oracle(tiny_oracle_map, history):
    c = W.config("tiny")
    ev = W.load_lightcurve("tiny")
    n, tr = 24, ev["truth"]
    rng = np.random.default_rng(history)
    P = np.array([tr["t0"], tr["u0"], tr["tE"], tr["alpha"]]) + rng.normal(0, 1, (n, 4)) * np.array([0.5, 0.01, 1.0, 0.02])
    amap = np.ascontiguousarray(tiny_oracle_map[2], np.float32)
    z = torch.zeros(n, dtype=torch.int32, device=DEV)
    note(f"refine oracle history {history}")
    _, chi2, chi2_0 = M.refine([(torch.from_numpy(amap).to(DEV), c["window"])], M.LightCurveBatch.from_events([ev], DEV),
                               torch.from_numpy(P).to(DEV), z, z, steps=30, history=history)
    _, oc, o0 = oracle_refine(tiny_oracle_map[2], c["window"], ev["tt"], ev["F"], ev["w"], ev["t_ref"], P,
                              LbfgsOptions(steps=30, history=history))
    assert rel_err(chi2_0.cpu().numpy(), o0).max() < 1e-10
    # the same machine but for binary32 roundings that an FP64 rounding of a sum flipped
    assert (rel_err(chi2.cpu().numpy(), oc) < 1e-6).mean() >= 0.9


def test_many_candidates_on_large_maps_equal_few():
    """Rounds as launches of their own (many candidates, maps beyond the last-level cache)
    against the same candidates a few at a time."""
    g = torch.Generator(device=DEV).manual_seed(3)
    maps = [(1 + 3 * torch.rand((2048, 2048), generator=g, device=DEV), (0.0, 0.0, 1.6, 1.6, 2048, 2048)) for _ in range(5)]
    rng = np.random.default_rng(8)
    evs = []
    for npts in (40, 300):
        tt = np.sort(rng.uniform(-30, 30, npts)).astype(np.float32)
        evs.append(dict(tt=tt, F=2 + rng.standard_normal(npts), w=rng.uniform(50, 150, npts), t_ref=0.0))
    lcs = M.LightCurveBatch.from_events(evs, DEV)
    n = 32801
    P = np.stack([rng.normal(0, 3, n), rng.uniform(0, 0.6, n), rng.uniform(8, 40, n), rng.uniform(0, 6.28, n)], 1)
    dP = torch.from_numpy(P).to(DEV)
    ev, mi = rng.integers(0, 2, n).astype(np.int32), rng.integers(0, 5, n).astype(np.int32)
    ev[7], mi[n - 1] = 2, 5  # out of range
    de, dm = torch.from_numpy(ev).to(DEV), torch.from_numpy(mi).to(DEV)
    note("refine many candidates on large maps")
    got = M.refine(maps, lcs, dP, de, dm, steps=12, history=3)
    for i0 in (0, 16000, n - 900):
        sl = slice(i0, i0 + 900)
        want = M.refine(maps, lcs, dP[sl].contiguous(), de[sl], dm[sl], steps=12, history=3)
        for a, b in zip(bits(*got), bits(*want)):
            assert torch.equal(a[sl], b)
