"""The single-lens magnification (uu + 2) / sqrt(uu (uu + 4)) of a sample off the map, uu = zx^2 + zy^2:
its short form takes the hardware's reciprocal square root and two corrections by residuals, and
has to give the bits of the correctly rounded root and quotient.  Every binary32 uu of its range
[2^-22, 2^12) and two binades beyond either end, through the line filter: a line passing (zx, zy)
in a window so small that all its samples are that point, none on the map.  The reference rounds
the FP64 root and quotient of binary32 values once, which is the correct rounding (53 bits are
more than twice 24 and two)."""
import math

import pytest
import torch

import paper_1511_01157_amd as M
from tests.helpers import note

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def point_with_square(uu):
    """Binary32 (x, y) with fl(fl(x x) + fl(y y)) = uu, or next to it."""
    y = uu.double().sqrt().float()
    y = torch.where(y * y > uu, torch.nextafter(y, torch.zeros_like(y)), y)
    return (uu.double() - (y * y).double()).sqrt().float(), y


@pytest.mark.parametrize("exponent", range(-24, 14))
def test_every_value_of_a_binade(exponent):
    note(f"single-lens magnification, uu in [2^{exponent}, 2^{exponent + 1})")
    first = (exponent + 127) << 23
    uu = torch.arange(first, first + (1 << 23), dtype=torch.int32, device=DEV).view(torch.float32)
    x, y = point_with_square(uu)
    xx, yy = x * x, y * y
    got_uu = xx + yy
    assert (got_uu == uu).float().mean() > 0.99
    lines = torch.zeros((uu.numel(), 3), dtype=torch.float64, device=DEV)
    lines[:, 0] = torch.hypot(x.double(), y.double())  # x = -u0 sin a, y = u0 cos a
    lines[:, 1] = torch.atan2(-x.double(), y.double())
    amap = torch.full((2, 2), 7.0, device=DEV)
    best, _, _ = M.line_filter(amap, (0.0, 0.0, 1e-30, 1e-30, 2, 2), lines, 1.0)
    p, d = got_uu + 2.0, got_uu * (got_uu + 4.0)
    want = (p.double() / d.double().sqrt().float().double()).float()
    assert torch.equal(best.view(torch.int32), want.view(torch.int32))
    assert math.isclose(float(best[0]), (2.0 ** exponent + 2) / math.sqrt(2.0 ** exponent * (2.0 ** exponent + 4)), rel_tol=1e-6)
