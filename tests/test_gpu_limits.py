"""Sizes that an entry point refuses, whatever path the call would take."""
import ctypes

import numpy as np
import pytest
import torch

import paper_1511_01157_amd as M
from paper_1511_01157_amd import _abi
from tests.helpers import note

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n", [1 << 31, (1 << 31) + 5, 1 << 40])
@pytest.mark.parametrize("n_maps", [1, 2])  # one group of candidates needs no order, two do
def test_more_candidates_than_an_order_holds(n, n_maps):
    rng = np.random.default_rng(0)
    ev = dict(tt=np.arange(5, dtype=np.float32), F=rng.random(5), w=np.ones(5), t_ref=0.0)
    lcs = M.LightCurveBatch.from_events([ev], DEV)
    amap = torch.ones((8, 8), device=DEV)
    views = M._map_views([(amap, (0.0, 0.0, 2.0, 2.0, 8, 8))] * n_maps)
    buf = torch.zeros(64, dtype=torch.float64, device=DEV)
    p = ctypes.c_void_p(buf.data_ptr())
    c = M.Context.get(0)
    note(f"limits: {n} candidates on {n_maps} maps")
    opts = M.LbfgsOpts(2, 8, 4, 0, 1e-4, 0.5)
    lca = lcs.abi()
    assert c.lib.morse_chi2_grad(c.handle, views, n_maps, ctypes.byref(lca), n, p, p, p, p, p, p, p) == _abi.MORSE_ERANGE
    assert c.lib.morse_chi2_grad_noalloc(c.handle, views, n_maps, ctypes.byref(lca), n, p, p, p, p, p, p, p) == _abi.MORSE_ERANGE
    assert c.lib.morse_refine(c.handle, views, n_maps, ctypes.byref(lca), n, p, p, p, ctypes.byref(opts), p, p) == _abi.MORSE_ERANGE
    torch.cuda.synchronize()
    assert not bool(buf.any())
