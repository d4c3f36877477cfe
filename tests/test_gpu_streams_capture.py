"""A map built under capture through a context bound to a stream that joins the capture, or to the
captured stream while another one is current: nothing is waited for while the graph is recorded, and every replay gives the map."""
import pytest
import torch

import paper_1511_01157_amd as M
from tests.helpers import note

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("forked", [True, False])
def test_map_captured_through_a_bound_context(forked):
    s, side = torch.cuda.Stream(device=DEV), torch.cuda.Stream(device=DEV)
    c = M.Context.bound(side)
    call = (1.0, 0.1, (0.0, 0.0, 4.0, 4.0, 1024, 1024), (0.0, 0.0, 2.0, 2.0, 256, 256), 0.02)
    want = M.build_map(*call, device=DEV).clone()
    out = torch.zeros_like(want)
    M.build_map(*call, out=out, ctx=c)  # workspace and taps are there
    torch.cuda.synchronize()
    note(f"streams: map captured through a bound context, forked {forked}")
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s if forked else side):
        if forked:
            side.wait_stream(s)
            M.build_map(*call, out=out, ctx=c)
            s.wait_stream(side)
        else:
            with torch.cuda.stream(s):
                M.build_map(*call, out=out, ctx=c)
        got = out * 1.0
    for _ in range(3):
        out.zero_()
        got.zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, want)
