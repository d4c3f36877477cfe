"""Contexts on another stream than torch's current one."""
import pytest
import torch

import paper_1511_01157_amd as M
from tests.helpers import note

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("with_counts", [False, True])
def test_map_is_whole_when_the_call_returns_to_another_stream(with_counts):
    """A map built through a context bound to a busy stream can be read on the current stream."""
    s = torch.cuda.Stream(device=DEV)
    c = M.Context.bound(s)
    call = (1.0, 0.1, (0.0, 0.0, 4.0, 4.0, 4096, 4096), (0.0, 0.0, 2.0, 2.0, 512, 512), 0.01)
    want = M.build_map(*call, device=DEV).clone()
    counts = torch.zeros((512, 512), dtype=torch.int32, device=DEV) if with_counts else None
    out = torch.zeros_like(want)
    big = torch.randn(8192, 8192, device=DEV)
    tmp = torch.empty_like(big)
    M.build_map(*call, out=torch.empty_like(out), ctx=c)  # workspace and taps are there
    torch.cuda.synchronize()
    note(f"streams: map on a bound context, counts {with_counts}")
    with torch.cuda.stream(s):
        for _ in range(5):
            torch.mm(big, big, out=tmp)
    got = M.build_map(*call, out=out, counts=counts, ctx=c).clone()
    assert torch.equal(got, want)
    torch.cuda.synchronize()
