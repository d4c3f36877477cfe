"""Calls under the caller's own graph captures: what is refused leaves the context and the capture
as they were; what is captured replays with its own inputs and results whatever the context did
in between."""
import numpy as np
import pytest
import torch

import paper_1511_01157_amd as M
from tests.helpers import note

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def test_refused_finite_source_call_leaves_no_trace():
    """The critical curve kept in a context is that of the last call that ran, not of a captured
    call that was refused; the capture that refused it goes on."""
    s = torch.cuda.Stream(device=DEV)
    z = torch.from_numpy(np.random.default_rng(0).normal(0, 0.05, (200, 2))).to(DEV)
    x = torch.zeros(8, device=DEV)
    lens_a, lens_b = (1.0, 0.1), (0.7, 0.4)
    note("graphs: refused finite-source call")
    with torch.cuda.stream(s):
        c, fresh = M.Context.bound(s), M.Context.bound(s)
        want = M.fs_magnification(*lens_b, z, 0.01, ctx=fresh)[0].clone()
        M.fs_magnification(*lens_a, z, 0.01, ctx=c)
        s.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            x += 1
            with pytest.raises(M.MorseError):
                M.fs_magnification(*lens_b, z, 0.01, ctx=c)
        got = M.fs_magnification(*lens_b, z, 0.01, ctx=c)[0]
        assert torch.equal(got, want)
        for rep in range(3):
            g.replay()
            s.synchronize()
            assert torch.equal(x, torch.full_like(x, rep + 1.0))
