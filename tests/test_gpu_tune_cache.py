"""Autotune caches of other versions of the shape table: taken without an error, kept by a merge,
and never used for a shape (their indices mean other shapes, tuned on other kernels)."""
import json

import numpy as np
import pytest
import torch

import paper_1511_01157_amd as M
from tests.helpers import note

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def test_cache_of_another_version(tmp_path):
    rng = np.random.default_rng(2)
    ev = dict(tt=np.sort(rng.uniform(-30, 30, 300)).astype(np.float32), F=2 + rng.standard_normal(300),
              w=rng.uniform(50, 150, 300), t_ref=0.0)
    lcs = M.LightCurveBatch.from_events([ev], DEV)
    maps = [(torch.from_numpy((1 + 3 * rng.random((40, 60))).astype(np.float32)).to(DEV), (0.0, 0.0, 2.0, 1.7, 60, 40))]
    tr = M.grid_trajectories(np.linspace(0, 0.5, 8), [0.3, 1.0], [0.5], [20.0])
    path = tmp_path / "tune.json"
    note("autotune cache of another version")
    best = M.autotune(maps, lcs, tr, cache_path=str(path))
    (cls, index), = json.loads(path.read_text()).items()
    assert index == best and cls.startswith("gfx950|v4|")
    old = cls.replace("|v4|", "|v3|")
    path.write_text(json.dumps({old: 11}))
    c = M.Context.bound(torch.cuda.current_stream())
    assert M.autotune_load(str(path), ctx=c) == 1
    want, got = M.search(maps, lcs, tr, "batched", top_k=4), M.search(maps, lcs, tr, "batched", top_k=4, ctx=c)
    for k in want:
        assert torch.equal(want[k], got[k])
    best = M.autotune(maps, lcs, tr, cache_path=str(path))
    assert json.loads(path.read_text()) == {old: 11, cls: best}
